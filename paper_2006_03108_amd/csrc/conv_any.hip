// Local convolution (Sec. 4, "Conv" and "[dConv]*" steps) of any channel count, kernel width, stride and dilation on
// the matrix cores: the layers whose shapes the patch kernels (conv_mfma.hip, conv_small.hip) do not take, for
// instance three input channels, or 7 x 7 kernels.  fp32 tensors are multiplied as three bf16 planes (split_bf16.h),
// bf16 tensors as they are; accumulation in fp32.
//
// Both kernels are one product C[row][col] = sum_k A[row][k] B[k][col] with 256 (or 64) rows and 32 NT columns per
// workgroup.  The values of a stage are gathered straight from the tensor, split and written to LDS as MFMA operand
// pieces (8 k of one row).
//   corr_any_kernel: rows are output positions, columns output channels, k = (tap, channel) with the channel fastest and
//     without padding (three channels of 49 taps are 147 k, not 49 x 8).  Data gradient: one class of the cells of dx^
//     per residue modulo the stride, all classes in one launch; a tap whose output does not exist reads as zero.
//     256 rows, 32 k per stage: wave w multiplies rows 64 w ... + 63 (2 x NT MFMA tiles).  64 rows, 128 k per stage, for
//     layers with too few positions to fill the chip: every wave multiplies all rows for its 32 k, and the four partial
//     tiles are added through LDS, in wave order.
//     Channel counts that are multiples of 4: neighbouring lanes load neighbouring pieces of 4 channels (with a lane per
//     row the 64 lanes of a load touch 64 lines, and the chip then loads 15 bytes per clock and compute unit: data
//     gradient of 8 x 224 x 224, 3 -> 32 channels, 7 x 7: 156 us).
//     Other counts: forward the channels of the taps along dimension 2 lie one behind the other in memory, a run; k is then
//     (tap of the other dimensions, place in the run), each run in octets of its own, what lies behind its end made zero.  Data
//     gradient, or taps that are dilated: a run is the channels of one tap.  Neighbouring lanes load neighbouring octets, 16 bytes
//     at a time whatever the alignment (bf16: the five words that hold them), where every element was a load that touched a line
//     for each row.  us of the kernel, element by element / by runs: forward 3 -> 32, 7 x 7, stride 2, 8 x 224 x 224 25.5 / 23.5;
//     43 -> 1, 5^3, 5 x 22 x 20 x 34 499 / 284; bf16 9 -> 2, 7 x 7, 2 x 252 x 325 54 / 23; back with 29 channels, 5^3, 2 x 31 x 29 x
//     35 437 / 247.  Not for runs of less than 8, nor where their ends make more than 1.3 times the stages (2 -> 24, 5^3 67 / 81),
//     nor for less than half a stage (1 -> 45, 5 taps 27 / 30), or a whole one back (30 channels, one tap, bf16 91 / 101).  bf16 quads
//     are 8 bytes: runs of 16 and more, of whole quads, go by octets too (60 -> 8, 5^3, 4 x 39 x 49 x 30 499 / 362), but not 4 -> 44,
//     3^3, 72 x 85 x 77, whose runs of 12 end in half an octet, 21 / 24.
//     In those a lane per row, and the offset of a k, the same for all lanes, goes into the scalar offset of the load.
//   wgrad_any_kernel: rows are k, columns output channels, the sum runs over output positions; the offset that all
//     lanes share is that of the position.  Every (worker, chunk of positions) writes a partial, which also holds the
//     chunk's part of db^.  256 rows and 32 positions per stage, or 64 rows and 128 positions (a layer of few channels and
//     taps has less than 64 rows, and a thread fetches 32 values a stage either way), where the waves take 32 positions
//     each and their partial tiles are added through LDS, in wave order.  us, 256 and 64 rows: 4 -> 16, 5 taps, 15 x 76551: 187 and 62; 9 -> 27,
//     5 taps, 2 x 184717: 65 and 25; bf16 20 -> 4, 3 taps, 7 x 455875: 415 and 127.
// Offsets that the lanes share are computed by the lanes, one each, and read out with v_readlane.
// fp32: the hi * hi products have an accumulator of their own, see gemm_split.hip.
#include <algorithm>
#include <type_traits>

#include "buffer.h"
#include "common.h"
#include "conv_any.h"
#include "conv_mfma.h"
#include "profile.h"
#include "split_bf16.h"
#include "weight_job.h"

namespace distdl {

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));


struct WgradAnyArgs {
  int32_t n_b, ci, co;
  int32_t k[3], s[3], dil[3];
  int32_t nchunks, ntm, ntn;  // position chunks per worker, row tiles, column tiles
  int32_t rows;               // taps * ci
  int64_t slot;
};

template <bool BF16>
__device__ inline float load1(__amdgpu_buffer_rsrc_t rs, uint32_t vo, uint32_t so) {
  if constexpr (BF16) return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rs, vo, so, 0) << 16);
  else return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, vo, so, 0));
}
template <bool BF16>
__device__ inline void load4(float* v, __amdgpu_buffer_rsrc_t rs, uint32_t vo, uint32_t so) {
  if constexpr (BF16) {
    const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(rs, vo, so, 0);
    v[0] = __uint_as_float(t[0] << 16), v[1] = __uint_as_float(t[0] & 0xffff0000u);
    v[2] = __uint_as_float(t[1] << 16), v[3] = __uint_as_float(t[1] & 0xffff0000u);
  } else {
    const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rs, vo, so, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(t[e]);
  }
}

// One dimension of a launch: the taps that take part and the input coordinate of the first one for output position q,
// in0 + q * step, and from one to the next, + dt.
struct DimAny {
  int32_t nt, tf, ts;      // taps tf, tf + ts, ...
  int32_t step, in0, dt;   // input coordinate of tap i at position q: in0 + q * step + i * dt
  int32_t nq, in_ext, out_ext, out0, ostep;
};
// (d is a template argument: indexed at run time the geometry would lie in scratch memory, and what is read from there counts
// as different in every lane, the buffers' descriptors too)
template <int d>
__device__ __forceinline__ DimAny dim_any(const WorkerDev& wd, const AnyArgs& a, int par) {
  DimAny g;
  if (a.mode == 0) {
    g.nt = a.k[d], g.tf = 0, g.ts = 1;
    g.step = a.s[d], g.in0 = wd.origin[d], g.dt = a.dil[d];
    g.nq = g.out_ext = wd.out[d], g.in_ext = wd.buf[d], g.out0 = 0, g.ostep = 1;
  } else {
    const int s = a.s[d], op = wd.origin[d] + par, first = op % s;  // first buffer cell of the class
    class_taps(a.k[d], s, a.dil[d], par, g.nt, g.tf, g.ts);
    // cell first + s q is origin + par + s (q - op / s): tap t reads dy[(q - op / s) - (t dil - par) / s]
    g.step = 1, g.in0 = -(op / s) - (g.tf * a.dil[d] - par) / s, g.dt = -(g.ts * a.dil[d] / s);
    g.nq = first < wd.buf[d] ? (wd.buf[d] - 1 - first) / s + 1 : 0;
    g.in_ext = wd.out[d], g.out_ext = wd.buf[d], g.out0 = first, g.ostep = s;
  }
  return g;
}

// What a thread gathers: octets of a row element by element, quads of channels, octets of runs (see above)
enum { kByOne = 0, kByQuad = 1, kByRun = 2 };
// k without padding, or the octets of a tap or run on their own
constexpr bool flat_k(int mode, int by) { return by == kByQuad || (mode == 0 && by == kByOne); }

// ROWS rows x KS octets of k per stage: 1024 pieces of A
constexpr int octets_of(int ROWS) { return 1024 / ROWS; }
// a little more than the planes, so that the pieces that eight neighbouring lanes write fall into different banks
constexpr uint32_t a_pitch(int ROWS, bool bf16) { return planes_of(bf16) * ROWS * 16 + (ROWS == 256 ? 32 : 16); }
constexpr uint32_t b_pitch(int NT, bool bf16) { return planes_of(bf16) * 32 * NT * 16 + 16; }
constexpr int any_lds(int ROWS, int NT, bool bf16) {
  const int stage = octets_of(ROWS) * (int)(a_pitch(ROWS, bf16) + b_pitch(NT, bf16));
  // (64 rows: four partial tiles at the end); the outputs of the rows, the word that asks for fp32 products
  return std::max(stage, ROWS == 64 ? 4 * 64 * 32 * NT * 4 : 0) + ROWS * 4 + 16;
}
// n / d for n, d < 2^22 through the reciprocal
__device__ inline int div_by(int n, int d, float rcp) {
  int q = (int)((float)n * rcp);
  q -= q * d > n;
  q += (q + 1) * d <= n;
  return q;
}

// the products of two 16-k slices, smallest first; la, lb: this wave's first row and octet
template <int ROWS, int NT, bool BF16>
__device__ inline void multiply_stage(floatx16 (&acc)[2][NT], floatx16 (&low)[2][NT], const char* la, const char* lb, int lane) {
  union Frag {
    u32x4 u;
    bf16x8 v;
  };
  constexpr int PL = planes_of(BF16);
  const int h = lane >> 5, ml = lane & 31;
#pragma unroll
  for (int sl = 0; sl < 2; ++sl) {
    Frag fa[PL][2], fb[PL][NT];
#pragma unroll
    for (int p = 0; p < PL; ++p) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
        fa[p][t].u = *(const u32x4*)(la + (2 * sl + h) * a_pitch(ROWS, BF16) + (p * ROWS + 32 * t + ml) * 16);
#pragma unroll
      for (int t = 0; t < NT; ++t)
        fb[p][t].u = *(const u32x4*)(lb + (2 * sl + h) * b_pitch(NT, BF16) + (p * 32 * NT + 32 * t + ml) * 16);
    }
    auto mm = [&](floatx16 (&c)[2][NT], int pa, int pb) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          c[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[pa][i].v, fb[pb][j].v, c[i][j], 0, 0, 0);
    };
    if constexpr (!BF16) {
      mm(low, 2, 0);
      mm(low, 0, 2);
      mm(low, 1, 1);
      mm(low, 1, 0);
      mm(low, 0, 1);
    }
    mm(acc, 0, 0);
  }
}
template <int ROWS, int NT>
__device__ inline void multiply_stage_halves(floatx16 (&acc)[2][NT], const char* la, const char* lb, int lane) {
  const int h = lane >> 5, ml = lane & 31;
#pragma unroll
  for (int sl = 0; sl < 2; ++sl) {
    Eight a[2], b[NT];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const char* const at = la + (2 * sl + h) * a_pitch(ROWS, false) + (32 * t + ml) * 16;
      a[t] = join_halves(*(const u32x4*)at, *(const u32x4*)(at + ROWS * 16));
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const char* const at = lb + (2 * sl + h) * b_pitch(NT, false) + (32 * t + ml) * 16;
      b[t] = join_halves(*(const u32x4*)at, *(const u32x4*)(at + 32 * NT * 16));
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = multiply_fp32(a[i], b[j], acc[i][j]);
  }
}
template <int NT, bool BF16>
struct Sums {
  floatx16 acc[2][NT], low[2][NT];
  __device__ inline void zero() {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
        for (int e = 0; e < 16; ++e) acc[i][j][e] = low[i][j][e] = 0.f;
  }
  // the sums of split operands; false if one of them is not finite
  __device__ inline bool finish() {
    float seen = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        acc[i][j] += low[i][j];
#pragma unroll
        for (int e = 0; e < 16; ++e) seen = note_not_finite(acc[i][j][e] *= kUnsplit, seen);
      }
    return !any_not_finite(seen);
  }
};

// Data gradient, output element (position, channel) term by term: only those taps whose output exists (in the product of a
// tile the others are zeros, which do not cancel a weight that is not finite).  A NaN ends it.
__device__ inline float corr_direct(const AnyArgs& a, const DimAny& g0, const DimAny& g1, const DimAny& g2, const float* in, int q0,
                                   int q1, int q2, int n, int ch) {
  float sum = 0.f;
  for (int i0 = 0; i0 < g0.nt; ++i0)
    for (int i1 = 0; i1 < g1.nt; ++i1)
      for (int i2 = 0; i2 < g2.nt; ++i2) {
        const int c0 = g0.in0 + q0 * g0.step + i0 * g0.dt, c1 = g1.in0 + q1 * g1.step + i1 * g1.dt,
                  c2 = g2.in0 + q2 * g2.step + i2 * g2.dt;
        if (c0 < 0 || c0 >= g0.in_ext || c1 < 0 || c1 >= g1.in_ext || c2 < 0 || c2 >= g2.in_ext) continue;
        const int tap = ((g0.tf + i0 * g0.ts) * a.k[1] + g1.tf + i1 * g1.ts) * a.k[2] + g2.tf + i2 * g2.ts;
        const float* x = in + ((((size_t)n * g0.in_ext + c0) * g1.in_ext + c1) * g2.in_ext + c2) * a.kc;
        for (int c = 0; c < a.kc; ++c) sum = fmaf(x[c], ((const float*)a.w)[((size_t)c * a.ci + ch) * a.taps + tap], sum);
        if (sum != sum) return sum;
      }
  return sum;
}

template <int ROWS, int NT, bool BF16, int MODE, int BY>
__global__ __launch_bounds__(256, 2) void corr_any_kernel(const WorkerDev* __restrict__ workers, void* const* in_bufs,
                                                          void* const* out_bufs, AnyArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr uint32_t ES = BF16 ? 2 : 4;
  constexpr int PL = planes_of(BF16), KS = octets_of(ROWS);
  constexpr bool VEC = BY != kByOne, RUNS = BY == kByRun;  // neighbouring lanes take neighbouring k of a row
  constexpr bool FLAT = flat_k(MODE, BY);                  // k without padding; else the octets of a run, or a tap, are its own
  // consecutive tiles share input rows and stay on one XCD (one L2)
  const uint32_t nblk = gridDim.x, r = (blockIdx.x & 7u) * (nblk >> 3) + (blockIdx.x >> 3);
  const uint32_t worker = r / a.tiles_max;
  int tile = (int)(r - worker * a.tiles_max);
  if (worker >= (uint32_t)a.n_workers) return;
  const WorkerDev wd = workers[worker];
  const int cls = (int)blockIdx.y;
  const int c12 = a.s[1] * a.s[2];
  const DimAny g0 = dim_any<0>(wd, a, MODE == 0 ? 0 : cls / c12), g1 = dim_any<1>(wd, a, MODE == 0 ? 0 : cls / a.s[2] % a.s[1]),
               g2 = dim_any<2>(wd, a, MODE == 0 ? 0 : cls % a.s[2]);
  const int ntile = tile % a.ntn;
  tile /= a.ntn;
  const int64_t total = (int64_t)a.n_b * g0.nq * g1.nq * g2.nq;
  if ((int64_t)tile * ROWS >= total) return;
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, ml = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t sc1 = (uint32_t)g2.in_ext * a.kc, sc0 = (uint32_t)g1.in_ext * sc1, scn = (uint32_t)g0.in_ext * sc0;
  const uint32_t so1 = (uint32_t)g2.out_ext * a.nc, so0 = (uint32_t)g1.out_ext * so1, son = (uint32_t)g0.out_ext * so0;
  // (bf16 runs are loaded as whole words: the first and the last may hold a value that is not the tensor's)
  const uint32_t skew = BF16 && RUNS ? (uint32_t)(uintptr_t)in_bufs[worker] & 2u : 0u;
  const uint32_t in_bytes = (uint32_t)a.n_b * scn * ES + skew;
  const __amdgpu_buffer_rsrc_t rin = rsrc_of((const char*)in_bufs[worker] - skew, BF16 && RUNS ? (in_bytes + 3u) & ~3u : in_bytes);
  const __amdgpu_buffer_rsrc_t rout = rsrc_of(out_bufs[worker], (uint32_t)a.n_b * son * ES);

  // a row's sample and position; false: beyond the last
  auto position = [&](int row, int& n, int& q0, int& q1, int& q2) {
    const int64_t pos = (int64_t)tile * ROWS + row;
    if (pos >= total) return false;
    uint32_t t = (uint32_t)pos;  // (fewer than 2^31 positions: the tensors are < 2 GiB)
    q2 = (int)(t % (uint32_t)g2.nq); t /= (uint32_t)g2.nq;
    q1 = (int)(t % (uint32_t)g1.nq); t /= (uint32_t)g1.nq;
    q0 = (int)(t % (uint32_t)g0.nq);
    n = (int)(t / (uint32_t)g0.nq);
    return true;
  };
  // The rows this thread gathers: VEC (octets of runs too): octet tid % KS of row tid / KS + i * (256 / KS); else row tid % ROWS, whose octets
  // (wave of the row) + (256 / ROWS) * o it takes.
  constexpr int NR = VEC ? 4 : 1;
  uint32_t base[NR];
  int p0[NR], p1[NR], p2[NR];  // input coordinates of tap 0 (data gradient: they may lie outside)
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int row = VEC ? tid / KS + i * (256 / KS) : tid % ROWS;
    int n, q0, q1, q2;
    base[i] = kOob;
    p0[i] = -0x40000000, p1[i] = p2[i] = 0;  // no tap of such a row is in range
    if (position(row, n, q0, q1, q2)) {
      p0[i] = g0.in0 + q0 * g0.step, p1[i] = g1.in0 + q1 * g1.step, p2[i] = g2.in0 + q2 * g2.step;
      base[i] = ((uint32_t)n * scn + (uint32_t)p0[i] * sc0 + (uint32_t)p1[i] * sc1 + (uint32_t)p2[i] * a.kc) * ES;
    }
  }
  char* const la = smem;
  char* const lb = smem + KS * a_pitch(ROWS, BF16);
  uint32_t* const row_out = (uint32_t*)(smem + any_lds(ROWS, NT, BF16) - ROWS * 4 - 16);  // byte offset of a row's outputs
  if (tid < ROWS) {
    int n, q0, q1, q2;
    row_out[tid] = position(tid, n, q0, q1, q2)
                       ? ((uint32_t)n * son + (uint32_t)(g0.out0 + q0 * g0.ostep) * so0 + (uint32_t)(g1.out0 + q1 * g1.ostep) * so1 +
                          (uint32_t)(g2.out0 + q2 * g2.ostep) * a.nc) * ES
                       : kOob;
  }

  const int n2 = RUNS ? g2.nt / a.run : g2.nt, ntaps = g0.nt * g1.nt * n2, len = RUNS ? a.run * a.kc : a.kc, noct = (len + 7) / 8;
  const int K = FLAT ? ntaps * a.kc : ntaps * noct * 8;
  const int stages = (K + 8 * KS - 1) / (8 * KS);
  const int octs = (K + 8 * kOctPad - 1) / (8 * kOctPad) * kOctPad;
  const float rc = 1.0f / (float)(FLAT ? a.kc : noct), r2 = 1.0f / (float)max(n2, 1), r1 = 1.0f / (float)max(g1.nt, 1);
  const __amdgpu_buffer_rsrc_t rw = rsrc_of(a.wt + ((size_t)a.woff[cls] * a.ntn + (size_t)ntile * octs) * (PL * 32 * NT),
                                            (uint32_t)octs * (PL * 32 * NT) * 16u);
  // index of a tap -> what its input coordinates add to those of tap 0
  auto steps_of = [&](int tap, int& d0, int& d1, int& d2) {
    const int t01 = div_by(tap, max(n2, 1), r2), t0 = div_by(t01, max(g1.nt, 1), r1);
    d2 = (tap - t01 * n2) * g2.dt, d1 = (t01 - t0 * g1.nt) * g1.dt, d0 = t0 * g0.dt;
  };

  float v[4][8];
  uint32_t word[4][5], shift[4];  // bf16 runs: the words that hold an octet, and where it starts in the first
  constexpr int BP = KS * PL * 32 * NT, BPT = (BP + 255) / 256;  // weight pieces of a stage
  u32x4 wp[BPT];
  int left = 0;  // BY RUN: of the octet that is loaded, the elements in its run
  auto load_stage = [&](int st, bool weights) {
    if constexpr (RUNS) {
      const int oct = st * KS + tid % KS, tap = div_by(oct, noct, rc), c = (oct - tap * noct) * 8;
      int d0, d1, d2;
      steps_of(tap, d0, d1, d2);
      const uint32_t add = ((uint32_t)d0 * sc0 + (uint32_t)d1 * sc1 + (uint32_t)d2 * (uint32_t)a.kc + (uint32_t)c) * ES;
      if (tap >= ntaps) d0 = -0x20000000;
      left = len - c;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        bool ok;
        if constexpr (MODE == 0) ok = tap < ntaps && base[i] != kOob;
        else ok = (uint32_t)(p0[i] + d0) < (uint32_t)g0.in_ext && (uint32_t)(p1[i] + d1) < (uint32_t)g1.in_ext &&
                  (uint32_t)(p2[i] + d2) < (uint32_t)g2.in_ext;
        const uint32_t off = ok ? base[i] + add + skew : kOob;
        if constexpr (BF16) {
          const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rin, off & ~3u, 0, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) word[i][e] = t[e];
          word[i][4] = __builtin_amdgcn_raw_buffer_load_b32(rin, (off & ~3u) + 16, 0, 0);
          shift[i] = (off & 2u) * 8u;
        } else {
          load4<BF16>(&v[i][0], rin, off, 0);
          load4<BF16>(&v[i][4], rin, off + 16, 0);
        }
      }
    } else if constexpr (VEC) {
      // two groups of four channels, each within one tap
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int k = (st * KS + tid % KS) * 8 + 4 * j, tap = div_by(k, a.kc, rc), c = k - tap * a.kc;
        int d0, d1, d2;
        steps_of(tap, d0, d1, d2);
        const uint32_t add = ((uint32_t)d0 * sc0 + (uint32_t)d1 * sc1 + (uint32_t)d2 * (uint32_t)a.kc + (uint32_t)c) * ES;
        if (k >= K) d0 = -0x20000000;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          bool ok;
          if constexpr (MODE == 0) ok = k < K && base[i] != kOob;
          else ok = (uint32_t)(p0[i] + d0) < (uint32_t)g0.in_ext && (uint32_t)(p1[i] + d1) < (uint32_t)g1.in_ext &&
                    (uint32_t)(p2[i] + d2) < (uint32_t)g2.in_ext;
          load4<BF16>(&v[i][4 * j], rin, ok ? base[i] + add : kOob, 0);
        }
      }
    } else if constexpr (MODE == 0) {
      // lane l works out where element l % 8 of this wave's octet l / 8 lies
      const int k = (st * KS + (ROWS == 256 ? 0 : wave) + (256 / ROWS) * ((lane & 31) >> 3)) * 8 + (lane & 7);
      const int tap = div_by(k, a.kc, rc);
      int d0, d1, d2;
      steps_of(tap, d0, d1, d2);
      const uint32_t ko = k < K ? ((uint32_t)d0 * sc0 + (uint32_t)d1 * sc1 + (uint32_t)d2 * (uint32_t)a.kc + (uint32_t)(k - tap * a.kc)) * ES : kOob;
#pragma unroll
      for (int o = 0; o < 4; ++o)
#pragma unroll
        for (int e = 0; e < 8; ++e) v[o][e] = load1<BF16>(rin, base[0], __builtin_amdgcn_readlane(ko, 8 * o + e));
    } else {
      // lane l works out octet l % 4 of this wave's: its tap's steps and first channel
      const int oct = st * KS + (ROWS == 256 ? 0 : wave) + (256 / ROWS) * (lane & 3);
      const int tap = div_by(oct, noct, rc), c8 = (oct - tap * noct) * 8;
      int d0, d1, d2;
      steps_of(tap, d0, d1, d2);
      if (tap >= ntaps) d0 = -0x20000000;
#pragma unroll
      for (int o = 0; o < 4; ++o) {
        const int e0 = __builtin_amdgcn_readlane(d0, o), e1 = __builtin_amdgcn_readlane(d1, o),
                  e2 = __builtin_amdgcn_readlane(d2, o), c0 = __builtin_amdgcn_readlane(c8, o);
        const bool ok = (uint32_t)(p0[0] + e0) < (uint32_t)g0.in_ext && (uint32_t)(p1[0] + e1) < (uint32_t)g1.in_ext &&
                        (uint32_t)(p2[0] + e2) < (uint32_t)g2.in_ext;
        const uint32_t vo = base[0] + ((uint32_t)e0 * sc0 + (uint32_t)e1 * sc1 + (uint32_t)e2 * (uint32_t)a.kc + (uint32_t)c0) * ES;
#pragma unroll
        for (int e = 0; e < 8; ++e)  // channels beyond kc (the same for all lanes) read as zero
          v[o][e] = load1<BF16>(rin, ok ? vo + e * ES : kOob, c0 + e < a.kc ? 0u : kOob);
      }
    }
    if (!weights) return;
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      const int piece = tid + i * 256;
      wp[i] = __builtin_amdgcn_raw_buffer_load_b128(rw, piece < BP ? piece * 16u : kOob, (uint32_t)st * (BP * 16u), 0);
    }
  };
  auto write_octets = [&](auto raw) {
    if constexpr (RUNS && BF16) {
      uint32_t keep[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) keep[e] = left >= 2 * e + 2 ? ~0u : left == 2 * e + 1 ? 0xffffu : 0u;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        u32x4 t;
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = __builtin_amdgcn_alignbit(word[i][e + 1], word[i][e], shift[i]) & keep[e];
        *(u32x4*)(la + tid % KS * a_pitch(ROWS, BF16) + (tid / KS + i * (256 / KS)) * 16) = t;
      }
      return;
    }
    if (RUNS && (len & 7) != 0) {  // (what lies behind a run is another cell's)
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i][e] = e < left ? v[i][e] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int oct = VEC ? tid % KS : tid / ROWS + (256 / ROWS) * i, row = VEC ? tid / KS + i * (256 / KS) : tid % ROWS;
      put_octet<BF16, decltype(raw)::value>(la + oct * a_pitch(ROWS, BF16) + row * 16, ROWS * 16, v[i]);
    }
  };
  auto write_stage = [&]() {
    write_octets(std::false_type{});
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      const int piece = tid + i * 256;  // [octet][plane][column]
      if (piece < BP) *(u32x4*)(lb + (piece / (PL * 32 * NT)) * b_pitch(NT, BF16) + piece % (PL * 32 * NT) * 16) = wp[i];
    }
  };

  Sums<NT, BF16> sums;
  const char* const wa = la + (ROWS == 256 ? wave * 64 * 16 : wave * 4 * a_pitch(ROWS, BF16));
  const char* const wb = lb + (ROWS == 256 ? 0 : wave * 4 * b_pitch(NT, BF16));
  // set if a sum of the tile is not finite; if a weight is not
  int* const redo = (int*)(smem + any_lds(ROWS, NT, BF16) - 16);
  if (!BF16 && tid == 0) redo[0] = redo[1] = 0;
  sums.zero();
  if (stages > 0) load_stage(0, true);
  for (int st = 0; st < stages; ++st) {
    write_stage();
    __syncthreads();
    if (st + 1 < stages) load_stage(st + 1, true);  // in flight while this stage multiplies
    multiply_stage<ROWS, NT, BF16>(sums.acc, sums.low, wa, wb, lane);
    if constexpr (!BF16) {
      if (st + 1 == stages && !sums.finish()) *redo = 1;
    }
    __syncthreads();
  }
  if (stages == 0) __syncthreads();  // row_out
  if constexpr (!BF16) {
    if (stages > 0 && __builtin_amdgcn_readfirstlane(*redo)) {  // (uniform, rare) the tile once more in fp32, its weights from the caller's
      const int nt3[3] = {g0.nt, g1.nt, g2.nt}, tf3[3] = {g0.tf, g1.tf, g2.tf}, ts3[3] = {g0.ts, g1.ts, g2.ts};
      sums.zero();
#pragma unroll 1
      for (int st = 0; st < stages; ++st) {
        load_stage(st, false);
        write_octets(std::true_type{});
#pragma unroll 1
        for (int piece = tid; piece < KS * 32 * NT; piece += 256) {  // [octet][column]
          const int col = piece % (32 * NT), oct = piece / (32 * NT);
          float wv[8];
          any_weight_octet<BF16, FLAT>(a, nt3, tf3, ts3, st * KS + oct, ntile * 32 * NT + col, wv);
          put_octet<BF16, true>(lb + oct * b_pitch(NT, BF16) + col * 16, 32 * NT * 16, wv);
          if constexpr (MODE == 1) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (not_finite(wv[e])) redo[1] = 1;
          }
        }
        __syncthreads();
        multiply_stage_halves<ROWS, NT>(sums.acc, wa, wb, lane);
        __syncthreads();
      }
    }
  }

  auto store = [&](int row, int ch, float bias, float s) {
    const uint32_t ro = row_out[row];
    const uint32_t off = ch < a.nc ? ro + (uint32_t)ch * ES : kOob;
    if constexpr (BF16) __builtin_amdgcn_raw_buffer_store_b16((uint16_t)pack_bf16(s + bias, 0.f), rout, off, 0, 0);
    else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(s + bias), rout, off, 0, 0);
  };
  bool terms = false;  // the tile has weights that are not finite
  if constexpr (!BF16 && MODE == 1) terms = __builtin_amdgcn_readfirstlane(redo[1]) != 0;
  auto again = [&](int row, int ch) {
    int n, q0, q1, q2;
    if (ch < a.nc && position(row, n, q0, q1, q2))
      ((float*)out_bufs[worker])[row_out[row] / 4 + ch] = corr_direct(a, g0, g1, g2, (const float*)in_bufs[worker], q0, q1, q2, n, ch);
  };
  auto bias_of = [&](int ch) { return a.bias && ch < a.nc ? ld((const typename Elem<BF16>::T*)a.bias, ch) : 0.f; };
  const int ch0 = ntile * 32 * NT;
  // register e of lane (h, ml) of MFMA tile (i, j): row 32 i + 8 (e / 4) + 4 h + e % 4, column 32 j + ml
  if constexpr (ROWS == 256) {
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const float bias = bias_of(ch0 + 32 * j + ml);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          store(wave * 64 + 32 * i + 8 * (e / 4) + 4 * h + (e % 4), ch0 + 32 * j + ml, bias, sums.acc[i][j][e]);
    }
    if constexpr (!BF16 && MODE == 1) {
      if (terms) {
        uint64_t which = 0;
#pragma unroll
        for (int t = 0; t < 32 * NT; ++t) which |= (uint64_t)not_finite(sums.acc[t & 1][t >> 5][(t >> 1) & 15]) << t;
        for (; which; which &= which - 1) {
          const int t = __ffsll((unsigned long long)which) - 1, e = (t >> 1) & 15;
          again(wave * 64 + 32 * (t & 1) + 8 * (e >> 2) + 4 * h + (e & 3), ch0 + 32 * (t >> 5) + ml);
        }
      }
    }
  } else {
    float* const red = (float*)smem;  // [wave][row][column]; the last barrier above came after the last read of a stage
    constexpr int NB = 32 * NT;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          red[(wave * 64 + 32 * i + 8 * (e / 4) + 4 * h + (e % 4)) * NB + 32 * j + ml] = sums.acc[i][j][e];
    __syncthreads();
    const int col = tid % NB;
    const float bias = bias_of(ch0 + col);
#pragma unroll
    for (int t = 0; t < 64 * NB / 256; ++t) {
      const int row = tid / NB + t * (256 / NB);
      const float* p = red + row * NB + col;
      const float s = ((p[0] + p[64 * NB]) + p[2 * 64 * NB]) + p[3 * 64 * NB];
      store(row, ch0 + col, bias, s);
      if constexpr (!BF16 && MODE == 1) {
        if (terms && not_finite(s)) again(row, ch0 + col);
      }
    }
  }
}

// grid: (row tiles * column tiles, chunks, workers)
template <int ROWS, int NT, bool BF16>
__global__ __launch_bounds__(256, 2) void wgrad_any_kernel(const WorkerDev* __restrict__ workers, void* const* x_bufs,
                                                           void* const* dy_bufs, float* __restrict__ partial, WgradAnyArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr uint32_t ES = BF16 ? 2 : 4;
  constexpr int KS = octets_of(ROWS), POS = 8 * KS;  // octets of positions, positions of a stage
  const int mt = (int)blockIdx.x % a.ntm, ntile = (int)blockIdx.x / a.ntm, chunk = (int)blockIdx.y, worker = (int)blockIdx.z;
  const WorkerDev wd = workers[worker];
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, ml = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t sx1 = (uint32_t)wd.buf[2] * a.ci, sx0 = (uint32_t)wd.buf[1] * sx1, sxn = (uint32_t)wd.buf[0] * sx0;
  const int npos = a.n_b * wd.out[0] * wd.out[1] * wd.out[2];
  const int all = (npos + POS - 1) / POS;  // stages of the worker, dealt to the chunks
  const int s_begin = (int)((int64_t)all * chunk / a.nchunks), s_end = (int)((int64_t)all * (chunk + 1) / a.nchunks);
  const __amdgpu_buffer_rsrc_t rx = rsrc_of(x_bufs[worker], (uint32_t)a.n_b * sxn * ES);
  const __amdgpu_buffer_rsrc_t ry = rsrc_of(dy_bufs[worker], (uint32_t)npos * a.co * ES);

  // this thread's row: tap and input channel
  uint32_t base = kOob;
  {
    const int k = mt * ROWS + tid % ROWS;
    if (k < a.rows) {
      const int tap = k / a.ci, c = k - tap * a.ci;
      const int t2 = tap % a.k[2], t01 = tap / a.k[2], t1 = t01 % a.k[1], t0 = t01 / a.k[1];
      base = ((uint32_t)(wd.origin[0] + t0 * a.dil[0]) * sx0 + (uint32_t)(wd.origin[1] + t1 * a.dil[1]) * sx1 +
              (uint32_t)(wd.origin[2] + t2 * a.dil[2]) * a.ci + c) * ES;
    }
  }
  // and its column of dy, an octet of positions
  constexpr int NB = 32 * NT, YO = (KS * NB + 255) / 256;  // octets of dy per thread
  char* const la = smem;
  char* const lb = smem + KS * a_pitch(ROWS, BF16);
  float v[4][8], y[YO][8];
  uint32_t yoff[YO];
#pragma unroll
  for (int i = 0; i < YO; ++i) {
    const int u = tid + i * 256, col = u % NB, o = u / NB, ch = ntile * NB + col;
    yoff[i] = o < KS && ch < a.co ? ((uint32_t)(o * 8) * a.co + ch) * ES : kOob;
  }
  auto load_stage = [&](int st) {
    // lane l works out where position l % 8 of this wave's octet l / 8 lies
    uint32_t t = (uint32_t)(st * POS + ((ROWS == 256 ? 0 : wave) + (256 / ROWS) * ((lane & 31) >> 3)) * 8 + (lane & 7));
    uint32_t po = kOob;
    if ((int)t < npos) {
      const uint32_t o2 = t % (uint32_t)wd.out[2]; t /= (uint32_t)wd.out[2];
      const uint32_t o1 = t % (uint32_t)wd.out[1]; t /= (uint32_t)wd.out[1];
      const uint32_t o0 = t % (uint32_t)wd.out[0], n = t / (uint32_t)wd.out[0];
      po = (n * sxn + o0 * a.s[0] * sx0 + o1 * a.s[1] * sx1 + o2 * a.s[2] * (uint32_t)a.ci) * ES;
    }
#pragma unroll
    for (int o = 0; o < 4; ++o)
#pragma unroll
      for (int e = 0; e < 8; ++e) v[o][e] = load1<BF16>(rx, base, __builtin_amdgcn_readlane(po, 8 * o + e));
    // positions beyond the last lie beyond the resource and read as zero
#pragma unroll
    for (int i = 0; i < YO; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) y[i][e] = load1<BF16>(ry, yoff[i], (uint32_t)(st * POS + e) * a.co * ES);
  };
  const bool bias_wg = mt == 0;  // these workgroups see every dy element of their columns and chunk once
  float bsum[YO];
#pragma unroll
  for (int i = 0; i < YO; ++i) bsum[i] = 0.f;
  auto write_stage = [&](auto raw) {
    constexpr bool RAW = decltype(raw)::value;
#pragma unroll
    for (int o = 0; o < 4; ++o)
      put_octet<BF16, RAW>(la + (tid / ROWS + (256 / ROWS) * o) * a_pitch(ROWS, BF16) + tid % ROWS * 16, ROWS * 16, v[o]);
#pragma unroll
    for (int i = 0; i < YO; ++i) {
      const int u = tid + i * 256;
      if (u < KS * NB) put_octet<BF16, RAW>(lb + (u / NB) * b_pitch(NT, BF16) + u % NB * 16, NB * 16, y[i]);
      if (bias_wg && !RAW)
        bsum[i] += ((y[i][0] + y[i][1]) + (y[i][2] + y[i][3])) + ((y[i][4] + y[i][5]) + (y[i][6] + y[i][7]));
    }
  };
  Sums<NT, BF16> sums;
  const char* const wa = la + (ROWS == 256 ? wave * 64 * 16 : wave * 4 * a_pitch(ROWS, BF16));
  const char* const wb = lb + (ROWS == 256 ? 0 : wave * 4 * b_pitch(NT, BF16));
  int* const redo = (int*)(smem + any_lds(ROWS, NT, BF16) - 16);  // set if a sum of the tile is not finite
  if (!BF16 && tid == 0) *redo = 0;
  sums.zero();
  if (s_begin < s_end) load_stage(s_begin);
  for (int st = s_begin; st < s_end; ++st) {
    write_stage(std::false_type{});
    __syncthreads();
    if (st + 1 < s_end) load_stage(st + 1);
    multiply_stage<ROWS, NT, BF16>(sums.acc, sums.low, wa, wb, lane);
    if constexpr (!BF16) {
      if (st + 1 == s_end && !sums.finish()) *redo = 1;
    }
    __syncthreads();
  }
  if constexpr (!BF16) {
    if (s_begin < s_end && __builtin_amdgcn_readfirstlane(*redo)) {  // (uniform, rare) the tile once more in fp32
      sums.zero();
#pragma unroll 1
      for (int st = s_begin; st < s_end; ++st) {
        load_stage(st);
        write_stage(std::true_type{});
        __syncthreads();
        multiply_stage_halves<ROWS, NT>(sums.acc, wa, wb, lane);
        __syncthreads();
      }
    }
  }
  float* const slot = partial + ((size_t)worker * a.nchunks + chunk) * a.slot;
  if constexpr (ROWS == 64) {
    float* const red = (float*)smem;  // [wave][row][column]; the last barrier above came after the last read of a stage
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          red[(wave * 64 + 32 * i + 8 * (e / 4) + 4 * h + (e % 4)) * NB + 32 * j + ml] = sums.acc[i][j][e];
    __syncthreads();
    const int col = tid % NB, ch = ntile * NB + col;
#pragma unroll
    for (int t = 0; t < 64 * NB / 256; ++t) {
      const int row = tid / NB + t * (256 / NB), k = mt * ROWS + row;
      const float* p = red + row * NB + col;
      if (k < a.rows && ch < a.co) slot[(size_t)k * a.co + ch] = ((p[0] + p[64 * NB]) + p[2 * 64 * NB]) + p[3 * 64 * NB];
    }
  } else
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int ch = ntile * NB + 32 * j + ml;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int k = mt * ROWS + wave * 64 + 32 * i + 8 * (e / 4) + 4 * h + (e % 4);
        if (k < a.rows && ch < a.co) slot[(size_t)k * a.co + ch] = sums.acc[i][j][e];
      }
  }
  if (bias_wg) {  // the octets of a column, in order
    float* const red = (float*)smem;  // (the last barrier above came after the last read of the stage)
    __syncthreads();
#pragma unroll
    for (int i = 0; i < YO; ++i)
      if (tid + i * 256 < KS * NB) red[tid + i * 256] = bsum[i];
    __syncthreads();
    if (tid < NB && ntile * NB + tid < a.co) {
      float sum = red[tid];
#pragma unroll
      for (int o = 1; o < KS; ++o) sum += red[o * NB + tid];
      slot[(size_t)a.rows * a.co + ntile * NB + tid] = sum;
    }
  }
}

// ---- host side ------------------------------------------------------------------

int nt_of(int64_t channels) { return channels > 32 ? 2 : 1; }

AnyArgs any_args(const distdl_plan* p, int mode, int NT) {
  AnyArgs a{};
  a.mode = mode;
  a.n_b = (int32_t)p->n_b;
  a.ci = (int32_t)p->n_ci;
  a.co = (int32_t)p->n_co;
  a.kc = mode == 0 ? a.ci : a.co;
  a.nc = mode == 0 ? a.co : a.ci;
  a.taps = 1;
  a.ncls = 1;
  for (int d = 0; d < 3; ++d) {
    a.k[d] = p->ksize[d];
    a.s[d] = p->stride[d];
    a.dil[d] = p->dilation[d];
    a.taps *= a.k[d];
    if (mode == 1) a.ncls *= a.s[d];
  }
  a.run = 1;
  a.n_workers = p->n_workers;
  a.ntn = (a.nc + 32 * NT - 1) / (32 * NT);
  return a;
}


// octets of weights of every class; returns their sum
int64_t class_octets(const AnyArgs& a, bool flat, int32_t* first, int& most, int* k_most = nullptr) {
  int64_t sum = 0;
  most = 0;
  if (k_most) *k_most = 0;
  for (int cls = 0; cls < a.ncls; ++cls) {
    int ntaps = 1;
    const int par[3] = {cls / (a.s[1] * a.s[2]), cls / a.s[2] % a.s[1], cls % a.s[2]};
    for (int d = 0; d < 3; ++d) {
      int nt = a.k[d], tf, ts;
      if (a.mode == 1) class_taps(a.k[d], a.s[d], a.dil[d], par[d], nt, tf, ts);
      ntaps *= nt;
    }
    const int K = flat ? ntaps * a.kc : ntaps / a.run * ((a.run * a.kc + 7) / 8) * 8;
    const int octs = (K + 8 * kOctPad - 1) / (8 * kOctPad) * kOctPad;
    if (first) first[cls] = (int32_t)sum;
    sum += octs;
    most = std::max(most, octs);
    if (k_most) *k_most = std::max(*k_most, K);
  }
  return sum;
}

int64_t positions_max(const distdl_plan* p, const AnyArgs& a) {
  int64_t mx = 0;
  for (const WorkerDev& wd : p->workers) {
    int64_t v = p->n_b;
    for (int d = 0; d < 3; ++d) v *= a.mode == 0 ? wd.out[d] : (wd.buf[d] + a.s[d] - 1) / a.s[d];
    mx = std::max(mx, v);
  }
  return mx;
}

size_t weight_floats(const distdl_plan* p, int mode) {
  AnyArgs a = any_args(p, mode, 2);
  int most;
  int64_t octs = class_octets(a, true, nullptr, most);
  for (const int run : {1, mode == 0 ? a.k[2] : 1}) a.run = run, octs = std::max(octs, class_octets(a, false, nullptr, most));
  return (size_t)octs * a.ntn * planes_of(p->dtype == DISTDL_BF16) * 32 * 2 * 4;
}

template <int ROWS, int NT, bool BF16, int MODE, int BY>
int launch_corr_any(distdl_plan* p, const AnyArgs& a, void** in_tab, void** out_tab, const char* name, hipStream_t st) {
  constexpr int lds = any_lds(ROWS, NT, BF16);
  const int64_t blocks = ((int64_t)a.tiles_max * p->n_workers + 7) / 8 * 8;
  if (lds > 64 * 1024)
    if (int rc = allow_large_lds<corr_any_kernel<ROWS, NT, BF16, MODE, BY>>()) return rc;
  ProfScope prof(name, st);
  hipLaunchKernelGGL((corr_any_kernel<ROWS, NT, BF16, MODE, BY>), dim3((unsigned)blocks, (unsigned)a.ncls), dim3(256), lds,
                     st, p->d_workers, in_tab, out_tab, a);
  return DISTDL_OK;
}

template <int ROWS, int NT, bool BF16>
int pick_corr_any(distdl_plan* p, const AnyArgs& a, int by, void** in_tab, void** out_tab, const char* name, hipStream_t st) {
#define DISTDL_BY(MODE_, BY_) launch_corr_any<ROWS, NT, BF16, MODE_, BY_>(p, a, in_tab, out_tab, name, st)
  if (by == kByQuad) return a.mode == 0 ? DISTDL_BY(0, kByQuad) : DISTDL_BY(1, kByQuad);
  if (by == kByRun) return a.mode == 0 ? DISTDL_BY(0, kByRun) : DISTDL_BY(1, kByRun);
  return a.mode == 0 ? DISTDL_BY(0, kByOne) : DISTDL_BY(1, kByOne);
#undef DISTDL_BY
}

// The launch of a direction: its arguments, rows of a tile, columns / 32; of its largest class: octets of weights, k
struct AnyLaunch {
  AnyArgs a;
  bool few;
  int by, NT, most, k;
};
AnyLaunch any_launch(const distdl_plan* p, int mode, bool aligned) {
  AnyLaunch l;
  l.NT = nt_of(mode == 0 ? p->n_co : p->n_ci);
  l.a = any_args(p, mode, l.NT);
  AnyArgs& a = l.a;
  const bool quads = aligned && a.kc % 4 == 0, bf16 = p->dtype == DISTDL_BF16;
  l.by = quads ? kByQuad : kByOne;
  if (!quads || bf16) {
    const int run = mode == 0 && a.dil[2] == 1 ? a.k[2] : 1, k = a.taps * a.kc;
    const int64_t runs = (int64_t)a.taps / run * ((run * a.kc + 7) / 8), stages = (runs + 3) / 4;
    if (run * a.kc >= (quads ? 16 : 8) && k >= (mode == 0 && !quads ? 16 : 33 * a.ncls) &&
        (mode == 1 || stages <= (quads ? 1.1 : 1.3) * ((k + 31) / 32)))
      l.by = kByRun, a.run = run;
  }
  class_octets(a, flat_k(mode, l.by), a.woff, l.most, &l.k);
  // (the estimates are of quads: octets in their place take no longer, whatever the ends of the runs add)
  if (int most; quads) class_octets(a, true, nullptr, most, &l.k);
  // 64 rows where 256 would leave compute units idle and there is enough k for four waves (32 columns: with 64 their
  // accumulators and the larger stages of weights do not fit the registers)
  const int64_t pos = positions_max(p, a);
  l.few = (pos + 255) / 256 * a.ntn * p->n_workers * a.ncls < 384 && l.most > kOctPad;
  const int rows = l.few ? 64 : 256;
  if (l.few) l.NT = 1, a.ntn = (a.nc + 31) / 32;
  a.tiles_max = (int32_t)((pos + rows - 1) / rows * a.ntn);
  return l;
}

int run_corr_any(distdl_plan* p, int mode, const void* w, const void* bias, bool aligned, void** in_tab, void** out_tab,
                 const char* name, hipStream_t st) {
  AnyLaunch l = any_launch(p, mode, aligned);
  AnyArgs& a = l.a;
  const bool few = l.few, bf16 = p->dtype == DISTDL_BF16;
  const int NT = l.NT;
  a.w = w;
  a.bias = bias;
  a.wt = (const u32x4*)p->d_wt;
#define DISTDL_ANY(ROWS_, NT_)                                                               \
  (bf16 ? pick_corr_any<ROWS_, NT_, true>(p, a, l.by, in_tab, out_tab, name, st)       \
        : pick_corr_any<ROWS_, NT_, false>(p, a, l.by, in_tab, out_tab, name, st))
  return few ? DISTDL_ANY(64, 1) : NT == 1 ? DISTDL_ANY(256, 1) : DISTDL_ANY(256, 2);
#undef DISTDL_ANY
}

}  // namespace

// 31-bit byte offsets into one worker's tensors, all classes in one launch
bool conv_any_supported(const distdl_plan* p) {
  if (p->explicit_halo) return false;
  if ((double)p->n_b * p->max_buf_cells * std::max(p->n_ci, p->n_co) * 4.0 >= 2147480000.0) return false;
  if ((double)p->n_b * p->max_out_cells * std::max(p->n_ci, p->n_co) * 4.0 >= 2147480000.0) return false;
  int64_t cls = 1, taps = 1;
  for (int d = 0; d < 3; ++d) {
    cls *= p->stride[d];
    taps *= p->ksize[d];
    if (p->stride[d] > 64) return false;
  }
  // (k is divided through a float reciprocal: fewer than 2^22)
  if (cls > kMaxCls || taps * (std::max(p->n_ci, p->n_co) + 8) >= (int64_t(1) << 22)) return false;
  if (taps * (p->n_ci + 64) * (p->n_co + 64) >= (int64_t(1) << 28)) return false;
  for (int mode = 0; mode < 2; ++mode) {  // a launch has fewer than 2^32 threads (64-row tiles: only small layers)
    const AnyArgs a = any_args(p, mode, nt_of(mode == 0 ? p->n_co : p->n_ci));
    if ((double)(positions_max(p, a) / 256 + 1) * a.ntn * p->n_workers + 8 >= kMaxBlocks256) return false;
  }
  return p->n_workers <= 65535;
}

// Estimated time of a launch: rounds of 512 workgroups, each a number of stages (32 k, or with 64 rows 128 k, which are shorter
// while a workgroup is alone on its compute unit) and an epilogue.  Fitted to 186 directions of 93 layers, 1 to 64 channels,
// 100 to 4 M positions, and 222 of 111 bf16 layers; nine tenths of them are within a quarter of it.  (Runs take what quads take:
// of 69 layers half are within 12 %.)
double corr_any_us(const distdl_plan* p, bool backward, bool aligned) {
  const AnyLaunch l = any_launch(p, backward ? 1 : 0, aligned);
  const double tiles = (double)l.a.tiles_max * p->n_workers * l.a.ncls, stages = std::max(1, (l.k + (l.few ? 127 : 31)) / (l.few ? 128 : 32));
  const double alone = tiles <= 256 ? 0.57 : 1.0, rounds = std::max(1.0, tiles / 512);
  if (p->dtype == DISTDL_BF16) {
    const double short_ = tiles <= 256 ? 0.5 : 1.0;
    if (l.few) return l.by != kByOne ? 4.5 + rounds * (stages * 1.43 * (tiles <= 256 ? 0.8 : 1.0) + 0.9) : 3.2 + rounds * stages * 2.1;
    if (l.by == kByOne) return 4.0 + rounds * (stages * 1.95 * short_ + 2.2) * (l.NT == 1 ? 1.0 : 1.3);
    return l.NT == 1 ? 4.7 + rounds * (stages * short_ + 2.7) : 4.5 + rounds * (stages * 1.28 * short_ + 4.8);
  }
  if (l.few) return l.by != kByOne ? 1.4 + rounds * (stages * 3.1 * alone + 5.6) : 4.9 + rounds * stages * 3.7 * alone;
  if (l.by == kByOne) return 3.4 + rounds * (stages * 4.6 * alone + 2.2) * l.NT;
  return l.NT == 1 ? 2.6 + rounds * (stages * 2.3 * alone + 5.2) : 1.0 + rounds * (stages * 3.4 * alone + 7.5);
}

int any_weight_job(distdl_plan* p, bool backward, const void* w, bool aligned, hipStream_t st, WeightJob& job) {
  if (int rc = ensure_wscratch(p, std::max(weight_floats(p, 0), weight_floats(p, 1)), st)) return rc;
  const AnyLaunch l = any_launch(p, backward ? 1 : 0, aligned);
  job.any = l.a;
  job.any.w = w;
  job.bf16 = p->dtype == DISTDL_BF16;
  job.flat = flat_k(l.a.mode, l.by);
  job.cols = 32 * l.NT;
  job.dst = (u32x4*)p->d_wt;
  job.per_class = (int32_t)(((int64_t)l.a.ntn * l.most * job.cols + 255) / 256);
  job.blocks = job.per_class * l.a.ncls;
  job.kind = job.blocks > 0 ? 2 : 0;
  return DISTDL_OK;
}

int conv_fwd_any(distdl_plan* p, const void* w, const void* bias, bool aligned, hipStream_t st) {
  return run_corr_any(p, 0, w, bias, aligned, p->tab_x.dev, p->tab_y.dev, "conv_fwd_any", st);
}

int conv_bwd_data_any(distdl_plan* p, const void* w, bool aligned, hipStream_t st) {
  return run_corr_any(p, 1, w, nullptr, aligned, p->tab_dy.dev, p->tab_dx.dev, "conv_bwd_data_any", st);
}

namespace {
// The tiles of a worker's weight gradient: rows, columns / 32; chunks of positions, about two workgroups per compute unit;
// the stages of a compute unit, one after the other; estimated time of the launch and of what its partials add to R.
struct WgradTiles {
  int rows, NT, chunks;
  bool alone;  // no second workgroup on a compute unit
  int64_t serial;
  double us;
};
// Rounds of 512 workgroups, the stages of one (shorter while it is alone on its compute unit), the tensors, the partials.  Fitted to
// 680 fp32 and 130 bf16 layers with tiles of either kind (1 to 64 channels, 100 to 20 M positions): four fifths are within 15 %
// (fp32) and 20 % of it.
WgradTiles tiles_of(const distdl_plan* p, int rows) {
  const int64_t k = (int64_t)p->ksize[0] * p->ksize[1] * p->ksize[2] * p->n_ci, pos = p->n_b * p->max_out_cells;
  WgradTiles t;
  t.rows = rows;
  t.NT = rows == 64 ? 1 : nt_of(p->n_co);
  const int per = 8 * octets_of(rows);
  const int64_t tiles = (k + rows - 1) / rows * ((p->n_co + 32 * t.NT - 1) / (32 * t.NT)) * p->n_workers, stages = (pos + per - 1) / per;
  // (a stage of a workgroup takes about 2 us, adding one more partial almost nothing: small layers one stage each)
  const int64_t most = std::max<int64_t>(std::min<int64_t>(stages, 64), stages / 4);
  t.chunks = (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>((512 + tiles - 1) / tiles, most), 512));
  const bool bf16 = p->dtype == DISTDL_BF16, alone = t.alone = tiles * t.chunks <= 256;
  const bool spread = p->n_ci == 1 && k > 32;  // a tap to every row: cells loaded one by one, from as many places as rows
  const double stage = rows == 64 ? (spread ? 1.7 : 1.0) * (bf16 ? (alone ? 0.96 : 1.2) : (alone ? 1.8 : 2.4))
                       : t.NT == 1 ? (bf16 ? (alone ? 0.61 : 1.06) : (alone ? 1.66 : 2.05)) : (bf16 ? 1.1 : (alone ? 2.85 : 2.57));
  const double elements = (double)p->n_workers * p->n_b * ((double)p->max_buf_cells * p->n_ci + (double)p->max_out_cells * p->n_co);
  t.serial = (tiles * t.chunks + 511) / 512 * ((stages + t.chunks - 1) / t.chunks);
  t.us = (bf16 ? 6.2 : 5.3) + t.serial * stage + (rows == 64 ? 0.21e-6 : 0.33e-6) * elements + 0.045e-3 * k * p->n_co;
  return t;
}
// 64 rows where they are estimated to take no more time, 0.95 of it from the third tile on, and a worker has more than one stage of
// positions (us, 64 and 256 rows: 49 rows 8 and 19, 120 rows 14 and 21, 147 rows, three tiles, 33 and 24; 125 rows and 37 columns,
// which are two tiles of 32 or one of 64, 1 -> 37 channels, 5^3, stride 2, 12 x 73 x 92 x 57, 213 and 120; bf16 layers of several kernel
// planes 0.9: 52 -> 3, 3^3, stride 2, 8 x 77 x 50 x 22, estimates 82 and 87, 93 and 73)
bool few_rows(const distdl_plan* p) { return (int64_t)p->ksize[0] * p->ksize[1] * p->ksize[2] * p->n_ci <= 128; }
WgradTiles wgrad_tiles(const distdl_plan* p) {
  const WgradTiles few = tiles_of(p, 64), many = tiles_of(p, 256);
  const bool planes = p->dtype == DISTDL_BF16 && p->ksize[0] > 1;
  return p->n_b * p->max_out_cells > 32 && few.us < (few_rows(p) ? 1.05 : planes ? 0.9 : 0.95) * many.us ? few : many;
}
}  // namespace

int wgrad_any_chunks(const distdl_plan* p) { return wgrad_tiles(p).chunks; }

int wgrad_any_rows(const distdl_plan* p) { return wgrad_tiles(p).rows; }
bool wgrad_any_unsure(const distdl_plan* p) { return wgrad_tiles(p).rows == 64 && (p->dtype != DISTDL_BF16 || few_rows(p)); }

// Against the other kernels.  256 rows by their stages alone, at the price that the factors of the others' estimates were found with:
// with the estimate above the choice is no better (1.025 of the fastest for 1.026 over the fp32 layers), and layers whose split
// estimate is high for its time (44 -> 48, 5 x 5) would change kernels.
// bf16 layers of more than 128 rows are weighed against the planes of conv_mfma.hip in the same way whichever tiles they get, in one
// and two dimensions also by the estimate of 64 rows: the planes' estimate is below their time there and above it with several kernel
// planes (us, planes / gather, kernel and reduction: 32 -> 32, 3 x 3, 2 x 60 x 64, 20 / 13; 24 -> 48, 5 x 5, 7 x 16 x 31, 19 / 12; 48 ->
// 8, 3^3, 3 x 55 x 30 x 33, 104 / 138).
double wgrad_any_us(const distdl_plan* p) {
  const WgradTiles t = wgrad_tiles(p), many = tiles_of(p, 256);
  const bool bf16 = p->dtype == DISTDL_BF16;
  const double stages = 4.5 + (double)many.serial * (many.alone ? 1.6 : 2.4) * many.NT * (bf16 ? 0.56 : 1.0);
  if (t.rows == 256) return stages;
  return bf16 && !few_rows(p) ? (p->ksize[0] > 1 ? stages : std::min(stages, t.us)) : t.us;
}

int conv_wgrad_any(distdl_plan* p, float* partial, hipStream_t st) {
  WgradAnyArgs a{};
  a.n_b = (int32_t)p->n_b;
  a.ci = (int32_t)p->n_ci;
  a.co = (int32_t)p->n_co;
  a.rows = a.ci;
  for (int d = 0; d < 3; ++d) {
    a.k[d] = p->ksize[d];
    a.s[d] = p->stride[d];
    a.dil[d] = p->dilation[d];
    a.rows *= a.k[d];
  }
  const WgradTiles t = wgrad_tiles(p);
  a.nchunks = t.chunks;
  const int NT = t.NT;
  a.ntm = (a.rows + t.rows - 1) / t.rows;
  a.ntn = (a.co + 32 * NT - 1) / (32 * NT);
  a.slot = (int64_t)a.rows * a.co + a.co;
  const dim3 grid((unsigned)(a.ntm * a.ntn), (unsigned)a.nchunks, (unsigned)p->n_workers);
  ProfScope prof("conv_bwd_weight_any", st);
#define DISTDL_WANY(ROWS_, NT_, BF_)                                                                                          \
  do {                                                                                                                 \
    constexpr int lds = any_lds(ROWS_, NT_, BF_);                                                                          \
    if (lds > 64 * 1024)                                                                                               \
      if (int rc_ = allow_large_lds<wgrad_any_kernel<ROWS_, NT_, BF_>>()) return rc_;                                         \
    hipLaunchKernelGGL((wgrad_any_kernel<ROWS_, NT_, BF_>), grid, dim3(256), lds, st, p->d_workers, p->tab_x.dev,             \
                       p->tab_dy.dev, partial, a);                                                                     \
  } while (0)
  if (p->dtype == DISTDL_BF16) {
    if (t.rows == 64) DISTDL_WANY(64, 1, true);
    else if (NT == 1) DISTDL_WANY(256, 1, true);
    else DISTDL_WANY(256, 2, true);
  } else {
    if (t.rows == 64) DISTDL_WANY(64, 1, false);
    else if (NT == 1) DISTDL_WANY(256, 1, false);
    else DISTDL_WANY(256, 2, false);
  }
#undef DISTDL_WANY
  return DISTDL_OK;
}

}  // namespace distdl
