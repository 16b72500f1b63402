// Small affine layers (Sec. 4 "Dense layers"): the forward pass in one launch, dx, dW and db of the adjoint in another.
//
// A layer of a few hundred features takes the tiled kernels 8 to 20 us a launch, and a second launch of 4 us wherever their K is
// split over workgroups, while its weights can be read in 2.  What they wait for is the chain of a staged tile (load, split,
// LDS, barrier, for every 64 k) and how few tiles there are.  Here no wave waits for another: each makes MT x NT tiles of 16 x 16
// from what its own lanes bring in, 32 k ahead, and where K is long the eight waves of a workgroup share a tile's K and add their
// parts up through LDS.
//   operand contiguous along k (x and W forward, dy in dx): eight rows of 32 k in a load, turned in LDS of the wave's own.  Loads
//     by sixteen rows of 4 k, as the matrix instructions take them, bring 15 bytes a clock to a compute unit: every row is a tag
//   operand that lies in memory as k lines (W in dx, both of dW): a lane reads NT (MT) neighbouring rows of one line
// fp32 tensors are multiplied and summed in fp64 (their sums are rounded once: 2.5e-8 against fp64 in the 2-norm, the tiled kernels
// 9e-8 and more), bf16 ones are widened and multiplied in fp32.  256 x 400 -> 120 on 2 x 2, forward and back: 11.9 -> 7.8 and
// 11.6 -> 9.4 us a call, of which a launch from the host is 6 to 7.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "affine_small.h"
#include "buffer.h"
#include "common.h"
#include "gemm_mfma.h"
#include "profile.h"

namespace distdl {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(4))) GemmBlock* BlockPtr;  // (scalar loads: nothing writes the descriptors while a kernel runs)

constexpr int kWaves = 8;

// N neighbouring elements at byte offset `off`.  V4: bf16 elements in pairs of 4 bytes (fp32 buffer loads ask for no more alignment).
template <bool BF16, bool V4, int N>
__device__ __forceinline__ void load_n(float (&v)[N], __amdgpu_buffer_rsrc_t rs, uint32_t off) {
  if constexpr (BF16) {
    if constexpr (V4 && N % 2 == 0) {
      uint32_t w[N / 2];
      if constexpr (N == 4) {
        const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
        w[0] = t[0], w[1] = t[1];
      } else {
        w[0] = __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < N; ++e) v[e] = __uint_as_float(e & 1 ? w[e / 2] & 0xffff0000u : w[e / 2] << 16);
    } else {
#pragma unroll
      for (int e = 0; e < N; ++e) v[e] = __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rs, off + 2 * e, 0, 0) << 16);
    }
  } else if constexpr (N == 4) {
    const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(t[e]);
  } else if constexpr (N == 2) {
    const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
    v[0] = __uint_as_float(t[0]), v[1] = __uint_as_float(t[1]);
  } else {
    v[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
  }
}

constexpr int kChunk = 32;           // k that a wave fetches at a time
constexpr int kPitch = kChunk + 4;   // floats from row to row in LDS: 9 units of 16 bytes, so that 16 rows' pieces fall into different banks

// T tiles of 16 rows of an operand that is contiguous along k.  Fetched as eight rows of 32 k an instruction (with a row to each of 16
// lanes, as the matrix instructions take them, a load's 64 lanes touch 64 pieces of lines, and a compute unit loads 15 bytes a clock:
// 37 x 2000 -> 1001 forward 13 us), and brought into order by way of LDS, in a part of it that is the wave's own.
template <bool BF16, bool V4, int T>
struct RowTiles {
  static constexpr uint32_t ES = BF16 ? 2 : 4;
  float v[T][2][4];
  int left;  // of k, from this lane's first
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, int ld, int rows, int K, int first, int lane, int k0) {
    const int k = k0 + 4 * (lane & 7);
    left = K - k;
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int row = first + 16 * t + 8 * r + (lane >> 3);
        load_n<BF16, V4, 4>(v[t][r], rs, row < rows && left > 0 ? ((uint32_t)row * ld + k) * ES : kOob);
      }
  }
  __device__ __forceinline__ void stage(float* lds, int lane) const {
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = e < left ? v[t][r][e] : 0.f;  // (what lies beyond K is the next row's)
        *(f32x4*)(lds + (16 * t + 8 * r + (lane >> 3)) * kPitch + 4 * (lane & 7)) = x;
      }
  }
  // what the lane of row `row` and quarter kq gives to the four products of step s
  static __device__ __forceinline__ f32x4 get(const float* lds, int t, int row, int kq, int s) {
    return *(const f32x4*)(lds + (16 * t + row) * kPitch + 16 * s + 4 * kq);
  }
};
// T tiles of an operand that lies in memory as k lines, over a chunk: val[s][j][t] is what the lane gives to product j of step s of
// tile t, row first + T * row + t of line 4 kq + j, or of line 4 j + kq (BOTH operands are lines: products beyond K can be left out)
template <bool BF16, bool V4, bool BOTH, int T>
struct LineTiles {
  static constexpr uint32_t ES = BF16 ? 2 : 4;
  float val[kChunk / 16][4][T];
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, int ld, int rows, int K, int first, int lane, int k0) {
    const int r = first + T * (lane & 15), kq = lane >> 4;
#pragma unroll
    for (int s = 0; s < kChunk / 16; ++s)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = k0 + 16 * s + (BOTH ? 4 * j + kq : 4 * kq + j);
        load_n<BF16, V4, T>(val[s][j], rs, k < K && r < rows ? ((uint32_t)k * ld + r) * ES : kOob);
      }
  }
};

template <bool BF16>
using SumOf = std::conditional_t<BF16, f32x4, f64x4>;
template <bool BF16>
using OneOf = std::conditional_t<BF16, float, double>;
template <bool BF16>
__device__ __forceinline__ SumOf<BF16> mma(float a, float b, SumOf<BF16> c) {
  if constexpr (BF16) return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  else return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// The tiles of a wave at (m0, n0), C[m][n] = sum_k A[m][k] B[n][k] over all segments.  B's rows are the instructions' rows, so that
// the four sums of a lane are of neighbouring n (see n_of).  SPLIT: the workgroup's waves take every eighth chunk.
template <bool A_KC, bool B_KC, int MT, int NT>
constexpr int stage_floats() {  // of a wave
  return ((A_KC ? MT : 0) + (B_KC ? NT : 0)) * 16 * kPitch;
}
template <bool BF16, bool V4, bool A_KC, bool B_KC, int MT, int NT, bool SPLIT>
__device__ __forceinline__ void small_tiles(BlockPtr gb, int m0, int n0, SumOf<BF16> (&acc)[MT][NT], char* smem) {
  constexpr bool BOTH = !A_KC && !B_KC;
  constexpr uint32_t ES = BF16 ? 2 : 4;
  const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int brow = B_KC && !BF16 ? 4 * (i & 3) + (i >> 2) : i;
  float* const la = (float*)smem + wave * stage_floats<A_KC, B_KC, MT, NT>();
  float* const lb = la + (A_KC ? MT : 0) * 16 * kPitch;
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[m][n] = SumOf<BF16>{0, 0, 0, 0};
  typedef std::conditional_t<A_KC, RowTiles<BF16, V4, MT>, LineTiles<BF16, V4, BOTH, MT>> TA;
  typedef std::conditional_t<B_KC, RowTiles<BF16, V4, NT>, LineTiles<BF16, V4, BOTH, NT>> TB;
  const int M = gb->M, N = gb->N;
  constexpr int STRIDE = SPLIT ? kWaves : 1;
  // The chunks of all segments are one sequence, so that loads run ahead from one into the next: `seg` holds chunks from ... to - 1.
  int total = 0;
  for (int s = 0; s < gb->nseg; ++s) total += (gb->seg[s].K + kChunk - 1) / kChunk;
  int seg = -1, from = 0, to = 0, K = 0, lda = 0, ldb = 0;
  __amdgpu_buffer_rsrc_t ra, rb;
  struct Set {
    TA a;
    TB b;
    int left;  // k of the chunk and after it, in its segment
  };
  auto fetch = [&](Set& x, int c) {
    if (c >= total) return;  // (uniform)
    while (c >= to) {
      ++seg;
      K = gb->seg[seg].K, lda = gb->seg[seg].lda, ldb = gb->seg[seg].ldb;
      from = to, to += (K + kChunk - 1) / kChunk;
      ra = rsrc_of(gb->seg[seg].a, (uint32_t)(A_KC ? M : K) * (uint32_t)lda * ES);
      rb = rsrc_of(gb->seg[seg].b, (uint32_t)(B_KC ? N : K) * (uint32_t)ldb * ES);
    }
    const int k0 = (c - from) * kChunk;
    x.left = K - k0;
    x.a.load(ra, lda, M, K, m0, lane, k0);
    x.b.load(rb, ldb, N, K, n0, lane, k0);
  };
  auto multiply = [&](const Set& x) {
#pragma unroll
    for (int s = 0; s < kChunk / 16; ++s) {
      if (16 * s >= x.left) break;  // (uniform)
      f32x4 va[MT], vb[NT];
      if constexpr (A_KC) {
#pragma unroll
        for (int m = 0; m < MT; ++m) va[m] = TA::get(la, m, i, kq, s);
      }
      if constexpr (B_KC) {
#pragma unroll
        for (int n = 0; n < NT; ++n) vb[n] = TB::get(lb, n, brow, kq, s);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (BOTH && 16 * s + 4 * j >= x.left) break;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int n = 0; n < NT; ++n) {
            float a, b;
            if constexpr (A_KC) a = va[m][j];
            else a = x.a.val[s][j][m];
            if constexpr (B_KC) b = vb[n][j];
            else b = x.b.val[s][j][n];
            acc[m][n] = mma<BF16>(b, a, acc[m][n]);
          }
      }
    }
  };
  // Two sets of registers in turn; rows are free for the next but one chunk once they are in LDS, lines once they are multiplied.
  Set set[2];
  int c = SPLIT ? wave : 0;
  fetch(set[0], c);
  fetch(set[1], c + STRIDE);
  while (c < total) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      if (c >= total) break;
      if constexpr (A_KC || B_KC) {
        // (the wave's lanes read what others of them wrote: its LDS instructions are carried out in order, and so they have to be compiled)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if constexpr (A_KC) set[d].a.stage(la, lane);
        if constexpr (B_KC) set[d].b.stage(lb, lane);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
      if constexpr (A_KC && B_KC) {
        Set at;
        at.left = set[d].left;
        fetch(set[d], c + 2 * STRIDE);
        multiply(at);
      } else {
        multiply(set[d]);
        fetch(set[d], c + 2 * STRIDE);
      }
      c += STRIDE;
    }
  }
}

// n of register e of tile t for the lanes of quarter kq, from the tiles' first; m of lane i
template <bool BF16, bool B_KC, int NT>
__device__ __forceinline__ int n_of(int t, int kq, int e) {
  return B_KC ? 16 * t + 4 * kq + e : NT * (BF16 ? 4 * kq + e : kq + 4 * e) + t;
}
template <bool A_KC, int MT>
__device__ __forceinline__ int m_of(int t, int i) {
  return A_KC ? 16 * t + i : MT * i + t;
}

template <bool BF16>
__device__ __forceinline__ float bias_of(BlockPtr gb, int n) {
  return gb->bias && n < gb->N ? ld((const std::conditional_t<BF16, uint16_t, float>*)gb->bias, n) : 0.f;
}

// Tiles whose K the eight waves have shared: added in wave order, one sum a thread at a time.
template <bool BF16, bool A_KC, bool B_KC, int MT, int NT>
__device__ __forceinline__ void reduce_and_store(BlockPtr gb, int m0, int n0, const SumOf<BF16> (&acc)[MT][NT], char* smem) {
  typedef OneOf<BF16> One;
  typedef std::conditional_t<BF16, uint16_t, float> T;
  SumOf<BF16>* const red = (SumOf<BF16>*)smem;  // [wave][tile][lane]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __syncthreads();  // (what the waves staged lies there)
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n) red[(wave * MT * NT + m * NT + n) * 64 + lane] = acc[m][n];
  __syncthreads();
  constexpr int ALL = MT * NT * 256;
#pragma unroll
  for (int r = 0; r < (ALL + 511) / 512; ++r) {
    const int v = tid + 512 * r;
    if (ALL % 512 && v >= ALL) break;
    const int tile = v >> 8, l = (v >> 2) & 63, e = v & 3;
    const int m = m0 + m_of<A_KC, MT>(tile / NT, l & 15), n = n0 + n_of<BF16, B_KC, NT>(tile % NT, l >> 4, e);
    const One* const p = (const One*)red + v;
    One s = p[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) s += p[w * ALL];
    s += bias_of<BF16>(gb, n);
    if (m < gb->M && n < gb->N) st((T*)gb->c, (size_t)m * gb->ldc + n, (float)s);
  }
}
// Tiles of one wave's own: 16 bytes at a time where a lane holds four neighbouring n (a store asks for 4-byte alignment)
template <bool BF16, bool A_KC, bool B_KC, int MT, int NT>
__device__ __forceinline__ void store_own(BlockPtr gb, int m0, int n0, const SumOf<BF16> (&acc)[MT][NT]) {
  typedef std::conditional_t<BF16, uint16_t, float> T;
  typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));
  const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  auto quad = [&](int m, int n, const float (&v)[4]) {
    if (m >= gb->M) return;
    const size_t at = (size_t)m * gb->ldc + n;
    if (!BF16 && n + 4 <= gb->N) {
      const u32x4_any t = {__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
      *(u32x4_any*)((float*)gb->c + at) = t;  // (64 bytes of a row: written past the L2 they would leave as parts of lines)
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < gb->N) st((T*)gb->c, at + e, v[e]);
    }
  };
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int row = m0 + m_of<A_KC, MT>(m, i);
    if constexpr (B_KC) {
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        const int col = n0 + n_of<BF16, true, NT>(n, kq, 0);
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (float)(acc[m][n][e] + bias_of<BF16>(gb, col + e));
        quad(row, col, v);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int col = n0 + n_of<BF16, false, NT>(0, kq, e);
        if constexpr (NT == 4) {
          const float v[4] = {(float)acc[m][0][e], (float)acc[m][1][e], (float)acc[m][2][e], (float)acc[m][3][e]};
          quad(row, col, v);
        } else {
#pragma unroll
          for (int n = 0; n < NT; ++n)
            if (row < gb->M && col + n < gb->N) st((T*)gb->c, (size_t)row * gb->ldc + col + n, (float)acc[m][n][e]);
        }
      }
    }
  }
}

// One product of a launch: its tiles of (16 MT) x (16 NT), SPLIT one a workgroup, else one a wave.
struct SmallGrid {
  const GemmBlock* blocks;
  int32_t tiles_m, tiles_n, wgs;  // of the largest block; workgroups a block
};
template <bool BF16, bool V4, bool A_KC, bool B_KC, int MT, int NT, bool SPLIT>
__device__ __forceinline__ void small_product(const SmallGrid& g, int wg, char* smem) {
  const int block = wg / g.wgs, rest = wg - block * g.wgs;
  const int tile = SPLIT ? rest : rest * kWaves + (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (tile >= g.tiles_m * g.tiles_n) return;
  const int m0 = tile % g.tiles_m * 16 * MT, n0 = tile / g.tiles_m * 16 * NT;  // (neighbouring tiles share B, the larger operand)
  const BlockPtr gb = (BlockPtr)(uintptr_t)(g.blocks + block);
  if (m0 >= gb->M || n0 >= gb->N) return;
  SumOf<BF16> acc[MT][NT];
  small_tiles<BF16, V4, A_KC, B_KC, MT, NT, SPLIT>(gb, m0, n0, acc, smem);
  if constexpr (SPLIT) reduce_and_store<BF16, A_KC, B_KC, MT, NT>(gb, m0, n0, acc, smem);
  else store_own<BF16, A_KC, B_KC, MT, NT>(gb, m0, n0, acc);
}

// db: 16 features a workgroup, 32 slices of the batch each, added in order
template <bool BF16>
__device__ __forceinline__ void small_colsum(const ColsumBlock& cb, int f0, char* smem) {
  typedef std::conditional_t<BF16, uint16_t, float> T;
  typedef OneOf<BF16> One;
  One* const red = (One*)smem;
  const int fl = threadIdx.x & 15, sl = threadIdx.x >> 4, f = f0 + fl;
  const bool live = cb.out && f < cb.n_f;
  One s = 0;
  if (live) {
    int n = sl;
    for (; n + 96 < cb.n_b; n += 128) {
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = ld((const T*)cb.in, (size_t)(n + 32 * u) * cb.n_f + f);
#pragma unroll
      for (int u = 0; u < 4; ++u) s += v[u];
    }
    for (; n < cb.n_b; n += 32) s += ld((const T*)cb.in, (size_t)n * cb.n_f + f);
  }
  red[sl * 16 + fl] = s;
  __syncthreads();
  if (sl != 0 || !live) return;
#pragma unroll
  for (int g = 1; g < 32; ++g) s += red[g * 16 + fl];
  st((T*)cb.out, f, (float)s);
}

template <bool BF16, bool V4, int MT, int NT, bool SPLIT>
__global__ __launch_bounds__(512, 2) void affine_small_fwd_kernel(SmallGrid g) {
  extern __shared__ __attribute__((aligned(32))) char smem[];
  small_product<BF16, V4, true, true, MT, NT, SPLIT>(g, (int)blockIdx.x, smem);
}

// workgroups: nx make dx, nw dW, the rest db
template <bool BF16, bool V4, int MTX, bool SPLITX, bool SPLITW>
__global__ __launch_bounds__(512, 2) void affine_small_bwd_kernel(SmallGrid gx, SmallGrid gw, const ColsumBlock* cs, int nx, int nw, int cs_chunks) {
  extern __shared__ __attribute__((aligned(32))) char smem[];
  const int b = (int)blockIdx.x;
  if (b < nx) small_product<BF16, V4, true, false, MTX, 2, SPLITX>(gx, b, smem);
  else if (b < nx + nw) small_product<BF16, V4, false, false, 2, SPLITW ? 2 : 4, SPLITW>(gw, b - nx, smem);
  else small_colsum<BF16>(cs[(b - nx - nw) / cs_chunks], (b - nx - nw) % cs_chunks * 16, smem);
}

}  // namespace

// ---- host side ------------------------------------------------------------------

bool affine_small_words(const std::vector<GemmBlock>& blocks) {
  for (const GemmBlock& b : blocks)
    for (int s = 0; s < b.nseg; ++s) {
      const GemmSeg& g = b.seg[s];
      if (g.lda % 2 || g.ldb % 2 || (uintptr_t)g.a % 4 || (uintptr_t)g.b % 4) return false;
    }
  return true;
}

struct SmallShape {
  SmallGrid g;
  int wgs, steps, chunks;  // in all; of 16 and of 32 k of a block's K
  int mt, nt;
  bool split;
};
static SmallShape shape_of(const GemmBlock* d_blocks, const std::vector<GemmBlock>& blocks, int mt, int nt, bool split) {
  int M = 0, N = 0, steps = 0, chunks = 0;
  for (const GemmBlock& b : blocks) {
    M = std::max(M, b.M), N = std::max(N, b.N);
    int st = 0, ch = 0;
    for (int s = 0; s < b.nseg; ++s) st += (b.seg[s].K + 15) / 16, ch += (b.seg[s].K + kChunk - 1) / kChunk;
    steps = std::max(steps, st), chunks = std::max(chunks, ch);
  }
  SmallShape s;
  s.g.blocks = d_blocks;
  s.g.tiles_m = (M + 16 * mt - 1) / (16 * mt), s.g.tiles_n = (N + 16 * nt - 1) / (16 * nt);
  const int64_t tiles = (int64_t)s.g.tiles_m * s.g.tiles_n;
  s.g.wgs = (int32_t)std::min<int64_t>(split ? tiles : (tiles + kWaves - 1) / kWaves, INT32_MAX / 64);
  s.wgs = (int)std::min<int64_t>((int64_t)s.g.wgs * blocks.size(), INT32_MAX);
  s.steps = steps, s.chunks = split ? (chunks + kWaves - 1) / kWaves : chunks;
  s.mt = mt, s.nt = nt, s.split = split;
  return s;
}
// What the shape of a product is chosen by: rounds of two workgroups a compute unit, matrix instructions and loads of a wave's steps
static double shape_us(const SmallShape& s, bool bf16) {
  const double per = std::ceil(s.steps / (s.split ? 8.0 : 1.0));
  const double step = s.mt * s.nt * (bf16 ? 0.06 : 0.115) + 0.05;  // us, two waves on a SIMD
  return std::max(1.0, s.wgs / 512.0) * (per * step * (s.wgs > 256 ? 2.0 : 1.0) + 1.5) + 0.25 * std::min(per, 8.0);
}
static SmallShape best_fwd(const GemmBlock* d, const std::vector<GemmBlock>& b, bool bf16) {
  SmallShape best{};
  double us = 1e30;
  auto consider = [&](int mt, int nt, bool split) {
    const SmallShape s = shape_of(d, b, mt, nt, split);
    if (const double t = shape_us(s, bf16); t < us) us = t, best = s;
  };
  for (int mt = 1; mt <= 4; ++mt) consider(mt, 1, true);
  consider(2, 2, false);
  return best;
}
static SmallShape best_dx(const GemmBlock* d, const std::vector<GemmBlock>& b, bool bf16) {
  SmallShape best{};
  double us = 1e30;
  for (int mt = 1; mt <= 2; ++mt)
    for (int split = 0; split < 2; ++split) {
      const SmallShape s = shape_of(d, b, mt, 2, split != 0);
      if (const double t = shape_us(s, bf16); t < us) us = t, best = s;
    }
  return best;
}
static SmallShape best_dw(const GemmBlock* d, const std::vector<GemmBlock>& b, bool bf16) {
  const SmallShape own = shape_of(d, b, 2, 4, false), shared = shape_of(d, b, 2, 2, true);
  return shape_us(shared, bf16) < shape_us(own, bf16) ? shared : own;
}

// Estimated times of the calls, fitted to 3000 layers of 1 to 1024 rows and 10 to 8192 features; four fifths are within 10 % (bf16
// 13 %).  A product: a start, and a wave's chunks with their loads and matrix instructions, which take longer with two workgroups on
// a compute unit; what is written, value by value in bf16.  With it, by a fourth power: what the host takes.  Forward a second
// workgroup on a compute unit is all but a second round (0.75, bf16 0.83; of four M-tiles, whose operands take 92 KB, it is one).
static double shared_cu(const SmallShape& s, double more) { return 1 + more * std::min(s.wgs / 256.0, 2.0); }
static double written(const std::vector<GemmBlock>& blocks) {  // 10^6 elements
  double n = 0;
  for (const GemmBlock& b : blocks) n += 1e-6 * b.M * b.N;
  return n;
}
double affine_small_fwd_us(const std::vector<GemmBlock>& blocks, bool bf16, double arrays) {
  const SmallShape s = best_fwd(nullptr, blocks, bf16);
  const double rounds = std::ceil(s.wgs / 256.0), chunks = s.chunks * (1 + (s.mt == 4 ? 1.0 : bf16 ? 0.83 : 0.75) * (rounds - 1));
  const double us = bf16 ? 0.25 * rounds + chunks * (0.24 + 0.46 * s.mt * s.nt) + 0.22 * written(blocks)
                         : 0.7 * rounds + chunks * (0.21 + 0.7 * s.mt * s.nt) + 0.7 * written(blocks);
  return joined(5.7 + arrays, us * (bf16 && !affine_small_words(blocks) ? 1.75 : 1.0));  // (rows of odd bf16 come value by value)
}
double affine_small_bwd_us(const std::vector<GemmBlock>& bx, const std::vector<GemmBlock>& bw, bool bf16, double arrays) {
  const SmallShape x = best_dx(nullptr, bx, bf16), w = best_dw(nullptr, bw, bf16);
  auto both = [&](double tx, double tw, double least) {
    const double longest = std::max(tx, tw), all = tx * x.wgs / 512.0 + tw * w.wgs / 512.0;
    return std::max(longest, all) + least * std::min(longest, all);
  };
  if (!bf16) {
    const double us = both(2.7 + 0.64 * x.chunks * x.mt * x.nt * shared_cu(x, 0.5), 0.66 * w.chunks * (1 + w.mt * w.nt) * shared_cu(w, 0.5), 0.32);
    return joined(6.5 + arrays, us + 1.2 * (std::ceil(std::max(x.wgs + w.wgs, 1) / 512.0) - 1));
  }
  const double odd = affine_small_words(bx) && affine_small_words(bw) ? 1.0 : 1.4, dw = written(bw);
  const double store = 1.7 * (written(bx) + dw) + 0.36 * dw / std::min(1.0, std::max(0.05, w.wgs / 256.0));
  return joined(7.7 + arrays, both(odd * (1.0 + x.chunks * (0.46 + 0.22 * x.mt * x.nt) * shared_cu(x, 0.48)), odd * (0.5 + w.chunks * (0.1 + 0.4 * w.mt * w.nt)), 0.64) + store);
}

template <bool BF16, bool A_KC, bool B_KC, int MT, int NT, bool SPLIT>
constexpr int lds_of() {
  return std::max(kWaves * stage_floats<A_KC, B_KC, MT, NT>() * 4, SPLIT ? kWaves * MT * NT * 64 * 4 * (BF16 ? 4 : 8) : 0);
}

template <bool BF16, bool V4, int MT, int NT, bool SPLIT>
static int fwd_variant(const SmallShape& s, hipStream_t st) {
  constexpr int lds = lds_of<BF16, true, true, MT, NT, SPLIT>();
  if (lds > 64 * 1024)
    if (int rc = allow_large_lds<affine_small_fwd_kernel<BF16, V4, MT, NT, SPLIT>>()) return rc;
  hipLaunchKernelGGL((affine_small_fwd_kernel<BF16, V4, MT, NT, SPLIT>), dim3((unsigned)s.wgs), dim3(512), lds, st, s.g);
  return DISTDL_OK;
}
template <bool BF16, bool V4>
static int fwd_pick(const SmallShape& s, hipStream_t st) {
  if (!s.split) return fwd_variant<BF16, V4, 2, 2, false>(s, st);
  return s.mt == 1 ? fwd_variant<BF16, V4, 1, 1, true>(s, st) : s.mt == 2 ? fwd_variant<BF16, V4, 2, 1, true>(s, st)
       : s.mt == 3 ? fwd_variant<BF16, V4, 3, 1, true>(s, st) : fwd_variant<BF16, V4, 4, 1, true>(s, st);
}
int launch_affine_small_fwd(const GemmBlock* d_blocks, const std::vector<GemmBlock>& blocks, bool bf16, hipStream_t st) {
  ProfScope prof("affine_fwd_small", st);
  const SmallShape s = best_fwd(d_blocks, blocks, bf16);
  if (!bf16) return fwd_pick<false, true>(s, st);
  return affine_small_words(blocks) ? fwd_pick<true, true>(s, st) : fwd_pick<true, false>(s, st);
}

template <bool BF16, bool V4, int MTX, bool SPLITX, bool SPLITW>
static int bwd_variant(const SmallShape& x, const SmallShape& w, const ColsumBlock* cs, int n_cs, int chunks, hipStream_t st) {
  constexpr int lds = std::max({lds_of<BF16, true, false, MTX, 2, SPLITX>(), lds_of<BF16, false, false, 2, SPLITW ? 2 : 4, SPLITW>(), 512 * (BF16 ? 4 : 8)});
  if (lds > 64 * 1024)
    if (int rc = allow_large_lds<affine_small_bwd_kernel<BF16, V4, MTX, SPLITX, SPLITW>>()) return rc;
  hipLaunchKernelGGL((affine_small_bwd_kernel<BF16, V4, MTX, SPLITX, SPLITW>), dim3((unsigned)(x.wgs + w.wgs + n_cs * chunks)), dim3(512), lds, st, x.g,
                     w.g, cs, x.wgs, w.wgs, std::max(chunks, 1));
  return DISTDL_OK;
}
template <bool BF16, bool V4>
static int bwd_pick(const SmallShape& x, const SmallShape& w, const ColsumBlock* cs, int n_cs, int chunks, hipStream_t st) {
#define DISTDL_SMALL(MT_, X_, W_) bwd_variant<BF16, V4, MT_, X_, W_>(x, w, cs, n_cs, chunks, st)
  if (w.split)
    return x.mt == 1 ? (x.split ? DISTDL_SMALL(1, true, true) : DISTDL_SMALL(1, false, true)) : (x.split ? DISTDL_SMALL(2, true, true) : DISTDL_SMALL(2, false, true));
  return x.mt == 1 ? (x.split ? DISTDL_SMALL(1, true, false) : DISTDL_SMALL(1, false, false)) : (x.split ? DISTDL_SMALL(2, true, false) : DISTDL_SMALL(2, false, false));
#undef DISTDL_SMALL
}
int launch_affine_small_bwd(const GemmBlock* d_bx, const std::vector<GemmBlock>& bx, const GemmBlock* d_bw, const std::vector<GemmBlock>& bw,
                            const ColsumBlock* d_cs, int n_cs, int max_f, bool bf16, hipStream_t st) {
  ProfScope prof("affine_bwd_small", st);
  const SmallShape x = best_dx(d_bx, bx, bf16), w = best_dw(d_bw, bw, bf16);
  const int chunks = d_cs ? (max_f + 15) / 16 : 0;
  if (!d_cs) n_cs = 0;
  if (!bf16) return bwd_pick<false, true>(x, w, d_cs, n_cs, chunks, st);
  return affine_small_words(bx) && affine_small_words(bw) ? bwd_pick<true, true>(x, w, d_cs, n_cs, chunks, st) : bwd_pick<true, false>(x, w, d_cs, n_cs, chunks, st);
}

}  // namespace distdl
