// GEMM of the partitioned affine layer (Sec. 4 "Dense layers") for fp32 operands of any shape and alignment, on the
// bf16 matrix cores (split_bf16.h), and for bf16 operands whose rows are not whole 16-byte pieces.
//
// A workgroup of four waves makes a tile of 64 T x 64 T outputs.  Per stage it takes 64 / T values of k from 64 T rows
// of each operand: global -> registers (the stage after is in flight while one is multiplied), split into three bf16
// planes once, written to LDS as MFMA operand pieces (8 consecutive k of one row).
//   T = 2: wave (wy, wx) multiplies the 64 x 64 quarter (wy, wx) of the tile (2 x 2 MFMA tiles), both 16-k slices of the
//     stage; every operand piece is read by two waves: 96 KB read and 48 KB written per 192 MFMAs, 3/4 of what LDS can
//     do in the time of the MFMAs.
//   T = 1 (tiles that 128 would mostly waste, and launches too small to fill the chip): every wave multiplies the whole
//     tile for one of the stage's four 16-k slices, and the four partial tiles are summed through LDS, in wave order.
// Piece (kp, p, r), octet of k kp, plane p, row r, lies at kp * pitch + (p * rows + r) * 16: a fragment read is 512
// contiguous bytes per half-wave, and pitch is a little more than three planes, so that the
// pieces that eight neighbouring lanes write fall into different banks.
// An operand whose rows are contiguous in memory instead of its k (W in dx, both operands of dW) is loaded two rows
// wide for eight k lines by each thread: the transpose happens in registers and costs nothing.
// fp32 operands of any alignment are loaded 8 or 16 bytes at a time (buffer loads and global stores of that width ask
// for 4-byte alignment): an issue of a load is what a small product spends most of its stages on, and eight per octet
// instead of two made a pass of 37 x 2000 -> 1001 on 2 x 3 workers, whose rows are no multiples of four wide, 34.8 us instead of 29.6.
#include <algorithm>
#include <type_traits>

#include "buffer.h"
#include "common.h"
#include "gemm_mfma.h"
#include "profile.h"
#include "split_bf16.h"

namespace distdl {

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));


union Frag {
  u32x4 u;
  bf16x8 v;
};

template <bool BF16>
__device__ inline float load_one(const void* p, size_t i) {
  if constexpr (BF16) return __uint_as_float((uint32_t)((const uint16_t*)p)[i] << 16);
  else return ((const float*)p)[i];
}

constexpr int planes_of(bool bf16) { return bf16 ? 1 : 3; }
constexpr int kStageKp(int T) { return 8 / T; }  // octets of k per stage
constexpr int operand_bytes(int T, bool bf16) { return kStageKp(T) * (planes_of(bf16) * 64 * T * 16) + 128; }
constexpr int split_lds(int T, bool bf16) {
  return (T == 1 ? std::max(2 * operand_bytes(T, bf16), 4 * 64 * 64 * 4) : 2 * operand_bytes(T, bf16)) + 16;  // (T = 1: four partial tiles at the end)
}

// The NP x 8 values a thread takes per operand and stage.  K-contiguous operand: NP pieces of 8 k; otherwise NP rows of
// eight k lines.  The per-lane offsets are fixed for a segment; the stage's k goes into the scalar offset.
template <bool BF16, bool KC, int T, bool VEC>
struct Operand {
  static constexpr int R = 64 * T, KP = kStageKp(T), NP = R * KP / 256;
  static constexpr uint32_t ES = BF16 ? 2 : 4;
  __amdgpu_buffer_rsrc_t rs;
  uint32_t off[NP];  // KC: of the pieces; else of the rows on line kp * 8
  uint32_t line;     // bytes from one row (KC) or k line to the next
  int K;
  bool lone;         // k lines, two rows: the second is beyond the last

  // rows r0 ... of an operand with `rows` rows; the resource ends with the operand, so that k lines beyond K read as zero.
  // (Lines of a GiB: 64 of them are more than 32 bits; octets of k beyond a K shorter than a stage are left out here, single
  // lines in load(), and an operand of K >= 64 that is below 2 GiB has lines of at most 32 MiB.)
  __device__ inline void enter(const void* base, int ld, int rows, int K_, int r0, int tid) {
    rs = rsrc_of(base, (uint32_t)(KC ? rows : K_) * (uint32_t)ld * ES);
    line = (uint32_t)ld * ES;
    K = K_;
    lone = false;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      if constexpr (KC) {
        const int idx = tid + i * 256, kp = idx % KP, r = r0 + idx / KP;
        off[i] = r < rows ? (uint32_t)r * line + kp * 8 * ES : kOob;
      } else {
        const int r = r0 + (tid % (R / NP)) * NP + i, kp = tid / (R / NP);
        off[i] = r < rows && kp * 8 < K_ ? (uint32_t)(kp * 8) * line + r * ES : kOob;
        if (!VEC && i == 1) lone = off[0] != kOob && off[1] == kOob;
      }
    }
  }
};
template <bool BF16, bool KC, int T, bool VEC>
struct Stager {
  typedef Operand<BF16, KC, T, VEC> Op;
  static constexpr int R = Op::R, KP = Op::KP, NP = Op::NP, PLANES = planes_of(BF16);
  static constexpr uint32_t ES = Op::ES;
  static constexpr uint32_t kPitch = PLANES * R * 16 + 128 / KP;
  float v[NP][8];

  template <bool TAIL>
  __device__ inline void octets(const Op& op, uint32_t so, int left, int tid) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int k = (tid + i * 256) % KP * 8;
      if constexpr (VEC) {  // K is a multiple of 4
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const uint32_t off = TAIL && k + 4 * j >= left ? kOob : op.off[i] + 16u * j;
          const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(op.rs, off, so, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[i][4 * j + e] = __uint_as_float(t[e]);
        }
      } else if constexpr (!TAIL && !BF16) {  // (buffer loads ask for 4-byte alignment only)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(op.rs, op.off[i] + 16u * j, so, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[i][4 * j + e] = __uint_as_float(t[e]);
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[i][j] = one(op.rs, TAIL && k + j >= left ? kOob : op.off[i] + ES * j, so);
      }
    }
  }
  // the values at k0 ... of the operand's segment
  __device__ __forceinline__ void load(const Op& op, int k0, int tid) {
    if constexpr (KC) {
      const uint32_t so = (uint32_t)k0 * ES;
      const int left = op.K - k0;  // pieces beyond K read as zero
      if (left >= KP * 8) octets<false>(op, so, left, tid);  // uniform: a whole stage
      else octets<true>(op, so, left, tid);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t so = k0 + j < op.K ? (uint32_t)(k0 + j) * op.line : kOob;  // (uniform)
        if constexpr (!BF16 && NP == 2) {  // two rows: where the second is not there (`lone`), the first in a load of its own
          const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(op.rs, VEC || !op.lone ? op.off[0] : kOob, so, 0);
          v[0][j] = __uint_as_float(t[0]);
          v[1][j] = __uint_as_float(t[1]);
        } else {
#pragma unroll
          for (int i = 0; i < NP; ++i) v[i][j] = one(op.rs, op.off[i], so);
        }
      }
      if constexpr (!VEC && !BF16 && NP == 2) {
        if (__builtin_amdgcn_ballot_w64(op.lone)) {  // (a wave at the operand's last row)
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const float x = one(op.rs, op.lone ? op.off[0] : kOob, k0 + j < op.K ? (uint32_t)(k0 + j) * op.line : kOob);
            v[0][j] = op.lone ? x : v[0][j];
          }
        }
      }
    }
  }
  static __device__ inline float one(__amdgpu_buffer_rsrc_t rs, uint32_t off, uint32_t so) {
    if constexpr (BF16) return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rs, off, so, 0) << 16);
    else return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off, so, 0));
  }
  template <bool RAW>
  __device__ inline void write(char* lds, int tid) const {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      int kp, r;
      if constexpr (KC) kp = (tid + i * 256) % KP, r = (tid + i * 256) / KP;
      else kp = tid / (R / NP), r = (tid % (R / NP)) * NP + i;
      char* const at = lds + kp * kPitch + r * 16;
      if constexpr (BF16) {
        u32x4 h;
#pragma unroll
        for (int j = 0; j < 4; ++j) h[j] = pack_bf16(v[i][2 * j], v[i][2 * j + 1]);  // exact
        *(u32x4*)at = h;
      } else if constexpr (RAW) {
        u32x4 u, w;
        halve_eight(v[i], u, w);
        *(u32x4*)at = u;
        *(u32x4*)(at + R * 16) = w;
      } else {
        u32x4 h, m, l;
        split_eight(v[i], kSplitScale, h, m, l);
        *(u32x4*)at = h;
        *(u32x4*)(at + R * 16) = m;
        *(u32x4*)(at + 2 * R * 16) = l;
      }
    }
  }
};

// Workgroup `wg` of one launch over `blocks`: wg = (block, split, tile), tile fastest.
struct SplitGrid {
  const GemmBlock* blocks;
  float* partial;          // nsplit > 1: fp32 partial tiles [block][split][M][N]
  int64_t partial_stride;  // floats between two splits
  int32_t tiles, nsplit, nblocks;
};

template <bool BF16, bool A_KC, bool B_KC, int T, bool VEC>
__device__ inline void gemm_split_tile(const SplitGrid& sg_, int wg, char* smem) {
  typedef Stager<BF16, A_KC, T, VEC> SA;
  typedef Stager<BF16, B_KC, T, VEC> SB;
  constexpr int PLANES = planes_of(BF16), SK = 8 * kStageKp(T), R = 64 * T;
  constexpr uint32_t kPitch = SA::kPitch;
  int tile = wg % sg_.tiles;
  const int rest = wg / sg_.tiles, split = rest % sg_.nsplit, block = rest / sg_.nsplit;
  // (nothing writes the descriptors while the kernel runs: read through the constant address space they are scalar loads
  // wherever they stand)
  const auto& gb = *(const __attribute__((address_space(4))) GemmBlock*)(uintptr_t)(sg_.blocks + block);
  const int tiles_m = (gb.M + R - 1) / R, tiles_n = (gb.N + R - 1) / R;
  if (tile >= tiles_m * tiles_n) return;
  const int m0 = (tile % tiles_m) * R, n0 = (tile / tiles_m) * R;
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, ml = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wy = T == 2 ? wave >> 1 : 0, wx = T == 2 ? wave & 1 : 0;
  char* const la = smem;
  char* const lb = smem + operand_bytes(T, BF16);

  int total = 0;
  for (int s = 0; s < gb.nseg; ++s) total += (gb.seg[s].K + SK - 1) / SK;
  const int s_begin = (int)((int64_t)total * split / sg_.nsplit), s_end = (int)((int64_t)total * (split + 1) / sg_.nsplit);

  // acc: the hi * hi products, one rounding of the running sum per 16 k; low: the other five, whose running sum is 2^-8
  // of it, so that its roundings do not count.  With all six in one accumulator the sums of a 2048^3 product were
  // 7.0e-7 off, with two 2.6e-7 (fp32 MFMAs, K split in two: 5.7e-7).
  floatx16 acc[2][2], low[2][2];
  auto zero = [&]() {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        for (int v = 0; v < 16; ++v) acc[i][j][v] = low[i][j][v] = 0.f;
  };

  // cursor of the next stage to load: its segment, its stage there, stages left there
  int seg, kin, left;
  SA sa;
  SB sb;
  typename SA::Op oa;
  typename SB::Op ob;
  auto load_stage = [&]() {
    while (left <= 0) {  // uniform: the segment that holds stage kin (stages of earlier segments taken off)
      if (seg >= 0) kin = -left;
      ++seg;
      left = (gb.seg[seg].K + SK - 1) / SK - kin;
      if (left > 0) {
        const auto& g = gb.seg[seg];
        oa.enter(g.a, g.lda, gb.M, g.K, m0, tid);
        ob.enter(g.b, g.ldb, gb.N, g.K, n0, tid);
      }
    }
    sa.load(oa, kin * SK, tid);
    sb.load(ob, kin * SK, tid);
    ++kin;
    --left;
  };
  const uint32_t fra = (T == 2 ? h : 2 * wave + h) * kPitch + (64 * wy + ml) * 16;
  const uint32_t frb = (T == 2 ? h : 2 * wave + h) * kPitch + (64 * wx + ml) * 16;
  Frag fa[PLANES][2], fb[PLANES][2];
  auto read = [&](const char* a, const char* b) {
#pragma unroll
    for (int p = PLANES - 1; p >= 0; --p)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        fa[p][t].u = *(const u32x4*)(a + fra + (p * R + 32 * t) * 16);
        fb[p][t].u = *(const u32x4*)(b + frb + (p * R + 32 * t) * 16);
      }
  };
  auto multiply = [&]() {
    auto mm = [&](floatx16 (&c)[2][2], int pa, int pb) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          c[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[pb][j].v, fa[pa][i].v, c[i][j], 0, 0, 0);
    };
    if constexpr (!BF16) {
      mm(low, 2, 0);
      mm(low, 0, 2);
      mm(low, 1, 1);
      mm(low, 1, 0);
      mm(low, 0, 1);
    }
    mm(acc, 0, 0);
  };
  auto multiply_halves = [&](const char* a, const char* b) {
    Eight xa[2], xb[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const char *const pa = a + fra + 32 * t * 16, *const pb = b + frb + 32 * t * 16;
      xa[t] = join_halves(*(const u32x4*)pa, *(const u32x4*)(pa + R * 16));
      xb[t] = join_halves(*(const u32x4*)pb, *(const u32x4*)(pb + R * 16));
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = multiply_fp32(xb[j], xa[i], acc[i][j]);
  };
  int* const redo = (int*)(smem + split_lds(T, BF16) - 16);  // set if a sum of the tile is not finite
  // The whole sum, from operands that are split, or (RAW) multiplied as they are.
  auto pass = [&](auto raw) __attribute__((always_inline)) {
    constexpr bool RAW = decltype(raw)::value;
    seg = -1, kin = s_begin, left = 0;
    zero();
    if (s_begin < s_end) load_stage();
    for (int s = s_begin; s < s_end; ++s) {
      sa.template write<RAW>(la, tid);
      sb.template write<RAW>(lb, tid);
      __syncthreads();
      if (s + 1 < s_end) load_stage();  // in flight while this stage multiplies
#pragma unroll
      for (int sl = 0; sl < (T == 2 ? 2 : 1); ++sl) {
        if constexpr (RAW) {
          multiply_halves(la + sl * 2 * kPitch, lb + sl * 2 * kPitch);
        } else {
          read(la + sl * 2 * kPitch, lb + sl * 2 * kPitch);
          multiply();
        }
      }
      if constexpr (!BF16 && !RAW) {
        if (s + 1 == s_end) {
          float seen = 0.f;
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              acc[i][j] += low[i][j];
#pragma unroll
              for (int v = 0; v < 16; ++v) seen = note_not_finite(acc[i][j][v] *= kUnsplit, seen);
            }
          if (any_not_finite(seen)) *redo = 1;
        }
      }
      __syncthreads();
    }
  };
  if (!BF16 && tid == 0) *redo = 0;
  pass(std::false_type{});
  if constexpr (!BF16) {
    if (s_begin < s_end && __builtin_amdgcn_readfirstlane(*redo)) pass(std::true_type{});  // (uniform)
  }

  // The products were accumulated transposed: register v of lane (h, ml) of MFMA tile (i, j) is
  // C[32 i + ml][32 j + 8 (v / 4) + 4 h + v % 4], so that a register quad is four consecutive columns.  The tile goes
  // through LDS (the last barrier above came after the last read of the stage) and leaves in whole lines: 16 bytes per
  // lane, 256 contiguous bytes per row.  Stored straight from the registers, one float per lane and the bias fetched
  // for each, the 268 MB of dW of a 16 x 8192 x 8192 layer took 260 us longer.
  typedef std::conditional_t<BF16, uint16_t, float> Out;
  float* const pc = sg_.nsplit > 1 ? sg_.partial + ((int64_t)block * sg_.nsplit + split) * sg_.partial_stride : nullptr;
  float* const red = (float*)smem;
  const int ldc = pc ? gb.N : gb.ldc;
  const void* const bias = pc ? nullptr : gb.bias;
  auto put = [&](int row, int col, float v) {
    if (pc) pc[(size_t)row * ldc + col] = v;
    else st((Out*)gb.c, (size_t)row * ldc + col, v);
  };
  // four columns from `col` of a row, in one store whatever its alignment (a store asks for 4 bytes)
  typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));
  auto quad = [&](int row, int col, const float (&b)[4], float4 s) {
    const float o[4] = {s.x + b[0], s.y + b[1], s.z + b[2], s.w + b[3]};
    if (row >= gb.M) return;
    if (!BF16 && col + 4 <= gb.N) {
      const u32x4_any t = {__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]), __float_as_uint(o[3])};
      if (pc) *(u32x4_any*)(pc + (size_t)row * ldc + col) = t;  // read again by the reduction
      else __builtin_nontemporal_store(t, (u32x4_any*)((float*)gb.c + (size_t)row * ldc + col));
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (col + e < gb.N) put(row, col + e, o[e]);
    }
  };
  auto bias_of = [&](int col, float (&b)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) b[e] = bias && col + e < gb.N ? load_one<BF16>(bias, col + e) : 0.f;
  };
  if constexpr (T == 2) {
    // each wave 32 rows of its quarter at a time, in 8 KB of its own; row r keeps its quad c at c ^ (r & 15)
    float4* const mine = (float4*)(smem + wave * 8192);
    const int col = n0 + 64 * wx + 4 * (lane & 15);
    float b[4];
    bias_of(col, b);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          mine[ml * 16 + ((8 * j + 2 * q + h) ^ (ml & 15))] =
              float4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
#pragma unroll
      for (int r8 = 0; r8 < 8; ++r8) {
        const int r = 4 * r8 + (lane >> 4);
        quad(m0 + 64 * wy + 32 * i + r, col, b, mine[r * 16 + ((lane & 15) ^ (r & 15))]);
      }
    }
  } else {
    // the four waves' partial tiles, [wave][64 rows][16 quads], added in wave order
    const int col = n0 + 4 * (tid & 15);
    float b[4];
    bias_of(col, b);  // (in flight while the tiles are written)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          ((float4*)red)[wave * 1024 + (32 * i + ml) * 16 + ((8 * j + 2 * q + h) ^ (ml & 15))] =
              float4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = (tid >> 4) + 16 * q;
      const float4* p = (const float4*)red + r * 16 + ((tid & 15) ^ (r & 15));
      float4 s = p[0];
#pragma unroll
      for (int w = 1; w < 4; ++w) {
        const float4 u = p[w * 1024];
        s.x += u.x, s.y += u.y, s.z += u.z, s.w += u.w;
      }
      quad(m0 + r, col, b, s);
    }
  }
}

// db_i[f] = sum over the batch of dy_i[n][f], 16 features per workgroup, 16 slices of the batch each, added in order
template <bool BF16>
__device__ inline void colsum_16(const ColsumBlock& cb, int f0, float* red) {
  const int fl = threadIdx.x & 15, sl = threadIdx.x >> 4, f = f0 + fl;
  const bool live = cb.out && f < cb.n_f;
  float part[4] = {0.f, 0.f, 0.f, 0.f};
  if (live) {
    int n = sl;
    for (; n + 48 < cb.n_b; n += 64)
#pragma unroll
      for (int u = 0; u < 4; ++u) part[u] += load_one<BF16>(cb.in, (size_t)(n + 16 * u) * cb.n_f + f);
    for (; n < cb.n_b; n += 16) part[0] += load_one<BF16>(cb.in, (size_t)n * cb.n_f + f);
  }
  red[sl * 16 + fl] = (part[0] + part[1]) + (part[2] + part[3]);
  __syncthreads();
  if (sl != 0 || !live) return;
  float s = red[fl];
#pragma unroll
  for (int g = 1; g < 16; ++g) s += red[g * 16 + fl];
  st((std::conditional_t<BF16, uint16_t, float>*)cb.out, f, s);
}

// A launch of n workgroups: rows of kGridX of them (along one dimension a launch holds fewer than 2^32 threads); the last row
// may have too many.
constexpr int kGridX = 1 << 22;
__device__ inline int workgroup() { return (int)(blockIdx.y * gridDim.x + blockIdx.x); }
inline dim3 grid_of_workgroups(int64_t n) { return dim3((unsigned)std::min<int64_t>(n, kGridX), (unsigned)((n + kGridX - 1) / kGridX)); }

// consecutive tiles share rows of an operand: each eighth of a launch's workgroups goes to one XCD (one L2)
__device__ inline int xcd_order(int wg, int n) {
  return n % 8 == 0 ? (wg & 7) * (n >> 3) + (wg >> 3) : wg;
}

template <bool BF16, int T, bool VEC>
__global__ __launch_bounds__(256, 2) void gemm_split_fwd_kernel(SplitGrid g) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int b = workgroup(), n = g.tiles * g.nsplit * g.nblocks;
  if (b < n) gemm_split_tile<BF16, true, true, T, VEC>(g, xcd_order(b, n), smem);
}

// The adjoint in one launch: the first nx workgroups make dx, the next nw dW, the rest db.  They are independent, and
// at the sizes that are short of workgroups each is too small to fill the chip alone.
template <bool BF16, int TX, int TW, bool VEC>
__global__ __launch_bounds__(256, 2) void gemm_split_bwd_kernel(SplitGrid gx, SplitGrid gw, const ColsumBlock* cs, int nx,
                                                                int nw, int n, int cs_chunks) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int b = workgroup();
  if (b >= n) return;
  if (b < nx) gemm_split_tile<BF16, true, false, TX, VEC>(gx, xcd_order(b, nx), smem);
  else if (b < nx + nw) gemm_split_tile<BF16, false, false, TW, VEC>(gw, xcd_order(b - nx, nw), smem);
  else colsum_16<BF16>(cs[(b - nx - nw) / cs_chunks], (b - nx - nw) % cs_chunks * 16, (float*)smem);
}

// C = sum over the splits, in order, of the partial tiles + bias; both contractions of an adjoint that are split are one
// launch (`second`: no splits, if there is one).  Bound by latency: a thread makes one element, or where rows, bias and
// arrays allow one quad, and has eight splits' loads in flight; with one load at a time and four elements a thread the
// two launches of a 37 x 2000 x 1001 layer (16 splits) took 17.2 and 10.1 us, and its whole pass 57.2 us; now 35.0.
template <bool BF16, bool QUADS>
__global__ __launch_bounds__(256) void gemm_split_reduce_kernel(SplitGrid first, SplitGrid second) {
  const bool in_first = (int)blockIdx.y < first.nblocks;
  const SplitGrid& g = in_first ? first : second;
  const int block = in_first ? (int)blockIdx.y : (int)blockIdx.y - first.nblocks;
  const GemmBlock& gb = g.blocks[block];
  const float* const pp = g.partial + (int64_t)block * g.nsplit * g.partial_stride;
  constexpr int V = QUADS ? 4 : 1;
  typedef float Vec __attribute__((ext_vector_type(V)));
  const int64_t e = ((int64_t)blockIdx.x * 256 + threadIdx.x) * V;
  if (e >= (int64_t)gb.M * gb.N) return;
  Vec s;
  for (int t0 = 0; t0 < g.nsplit; t0 += 8) {
    Vec u[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) u[t] = *(const Vec*)(pp + min(t0 + t, g.nsplit - 1) * g.partial_stride + e);
#pragma unroll
    for (int t = 0; t < 8; ++t)
      if (t0 + t < g.nsplit) s = t0 + t == 0 ? u[0] : s + u[t];
  }
  const int col = (int)(e % gb.N);  // (QUADS: N is a multiple of 4)
#pragma unroll
  for (int i = 0; i < V; ++i) {
    if (gb.bias) s[i] += load_one<BF16>(gb.bias, col + i);
  }
  if constexpr (QUADS) *(Vec*)((float*)gb.c + e) = s;  // (ldc = N)
  else st((std::conditional_t<BF16, uint16_t, float>*)gb.c, (size_t)(e / gb.N) * gb.ldc + col, s[0]);
}

}  // namespace

// ---- host side ------------------------------------------------------------------

bool gemm_split_usable(const std::vector<GemmBlock>& blocks, bool bf16, bool a_kc, bool b_kc) {
  const size_t es = bf16 ? 2 : 4;
  for (const GemmBlock& b : blocks) {
    if (b.nseg < 1 || b.nseg > kGemmMaxSeg) return false;
    for (int s = 0; s < b.nseg; ++s) {
      const GemmSeg& g = b.seg[s];
      const double a_bytes = (double)(a_kc ? b.M : g.K) * g.lda * es, b_bytes = (double)(b_kc ? b.N : g.K) * g.ldb * es;
      if (a_bytes >= 2147480000.0 || b_bytes >= 2147480000.0) return false;  // 31-bit byte offsets
    }
  }
  return true;
}

// 16-byte pieces of K-contiguous operands, 8-byte pairs of k lines (fp32)
static bool all_vec(const std::vector<GemmBlock>& blocks, bool a_kc, bool b_kc) {
  for (const GemmBlock& b : blocks)
    for (int s = 0; s < b.nseg; ++s) {
      const GemmSeg& g = b.seg[s];
      if ((uintptr_t)g.a % 16 || (uintptr_t)g.b % 16 || g.lda % 4 || g.ldb % 4) return false;
      if ((a_kc || b_kc) && g.K % 4) return false;
      if (!a_kc && b.M % 4) return false;
      if (!b_kc && b.N % 4) return false;
    }
  return true;
}

bool gemm_split_vec(const std::vector<GemmBlock>& blocks, bool bf16, bool a_kc, bool b_kc) {
  return !bf16 && all_vec(blocks, a_kc, b_kc);
}

GemmSplitPlan gemm_split_plan(const std::vector<GemmBlock>& blocks, bool vec) {
  GemmSplitPlan p;
  p.vec = vec;
  auto count = [&](int t, int& most, int64_t& all) {
    most = 0, all = 0;
    for (const GemmBlock& b : blocks) {
      const int n = ((b.M + t - 1) / t) * ((b.N + t - 1) / t);
      most = std::max(most, n);
      all += n;
    }
  };
  int64_t macs = 0, macs128 = 0, all = 0;
  int stages = INT32_MAX;  // of 32 k, least over the blocks
  for (const GemmBlock& b : blocks) {
    int st = 0;
    for (int s = 0; s < b.nseg; ++s) {
      st += (b.seg[s].K + 31) / 32;
      macs += (int64_t)b.M * b.N * b.seg[s].K;
      macs128 += (int64_t)((b.M + 127) / 128 * 128) * ((b.N + 127) / 128 * 128) * b.seg[s].K;
    }
    stages = std::min(stages, st);
    p.max_mn = std::max<int64_t>(p.max_mn, (int64_t)b.M * b.N);
  }
  p.max_mn = (p.max_mn + 3) / 4 * 4;
  // 128-tiles where they waste little and, with K split, make enough workgroups of enough stages
  count(128, p.tiles, all);
  p.T = p.vec && macs128 <= macs + macs / 4 && all * std::max(1, stages / 8) >= 256 ? 2 : 1;
  if (p.T == 1) {
    count(64, p.tiles, all);
    stages = (stages + 1) / 2;
  }
  // K split over workgroups, by an estimate of the launch's time in us: stages of 1.4 with one workgroup on a compute
  // unit, 2.2 with two, and for the split 5 for the second launch and its partial tiles written and read at 5 TB/s.
  // Measured forward launches, 256 x 4096 x 4096: 4 / 6 / 8 / 12 splits 74 / 66 / 62 / 63 us; 1000 x 1024 x 1024,
  // whole layer: 4 / 6 / 8 splits 80 / 80 / 88 us.
  double best = 1e30;
  for (int ns = 1; ns <= 16 && ns <= std::max(1, stages / 2); ++ns) {
    const double res = (double)all * ns / 256, tau = res <= 1 ? 1.4 : 1.4 + 0.8 * (std::min(res, 2.0) - 1);
    const double work = (stages + ns - 1) / ns * tau * std::max(1.0, res / 2), split = ns > 1 ? 5 + ns * (double)p.max_mn * blocks.size() * 8 / 5e6 : 0;
    if (work + split < best * 0.98) best = work + split, p.stages_us = work, p.split_us = split, p.nsplit = ns;
  }
  p.wgs = p.tiles * p.nsplit * (int)blocks.size();
  p.partial_floats = p.nsplit > 1 ? (size_t)p.max_mn * p.nsplit * blocks.size() : 0;
  return p;
}

static SplitGrid grid_of(const GemmBlock* d_blocks, size_t n, const GemmSplitPlan& p, float* partial) {
  return SplitGrid{d_blocks, partial, p.max_mn, p.tiles, p.nsplit, (int32_t)n};
}

// rows that are whole quads, in 16-byte aligned arrays
static bool quad_rows(const std::vector<GemmBlock>& blocks) {
  for (const GemmBlock& b : blocks)
    if (b.N % 4 || b.ldc != b.N || (uintptr_t)b.c % 16) return false;
  return true;
}

// (a launch that is not split: no blocks)
static void launch_reduce(SplitGrid a, SplitGrid b, bool quads, bool bf16, hipStream_t st) {
  if (a.nsplit <= 1) a.nblocks = 0;
  if (b.nsplit <= 1) b.nblocks = 0;
  if (a.nblocks + b.nblocks == 0) return;
  const int64_t most = std::max(a.nblocks ? a.partial_stride : 0, b.nblocks ? b.partial_stride : 0), per = quads ? 1024 : 256;
  const dim3 grid((unsigned)((most + per - 1) / per), (unsigned)(a.nblocks + b.nblocks));
  if (bf16) hipLaunchKernelGGL((gemm_split_reduce_kernel<true, false>), grid, dim3(256), 0, st, a, b);
  else if (quads) hipLaunchKernelGGL((gemm_split_reduce_kernel<false, true>), grid, dim3(256), 0, st, a, b);
  else hipLaunchKernelGGL((gemm_split_reduce_kernel<false, false>), grid, dim3(256), 0, st, a, b);
}

template <bool BF16, int T, bool VEC>
static int fwd_variant(const SplitGrid& g, int wgs, hipStream_t st) {
  constexpr int lds = split_lds(T, BF16);
  if (lds > 64 * 1024)
    if (int rc = allow_large_lds<gemm_split_fwd_kernel<BF16, T, VEC>>()) return rc;
  hipLaunchKernelGGL((gemm_split_fwd_kernel<BF16, T, VEC>), grid_of_workgroups(wgs), dim3(256), lds, st, g);
  return DISTDL_OK;
}

int launch_gemm_split_fwd(const GemmBlock* d_blocks, const std::vector<GemmBlock>& blocks, bool bf16,
                          const GemmSplitPlan& p, float* partial, hipStream_t st) {
  ProfScope prof("affine_fwd_split", st);
  const SplitGrid g = grid_of(d_blocks, blocks.size(), p, partial);
  int rc = bf16 ? fwd_variant<true, 1, false>(g, p.wgs, st)
                : p.T == 2 ? fwd_variant<false, 2, true>(g, p.wgs, st)
                           : p.vec ? fwd_variant<false, 1, true>(g, p.wgs, st) : fwd_variant<false, 1, false>(g, p.wgs, st);
  if (!rc) launch_reduce(g, SplitGrid{}, !bf16 && quad_rows(blocks), bf16, st);
  return rc;
}

template <bool BF16, int TX, int TW, bool VEC>
static int bwd_variant(const SplitGrid& gx, const SplitGrid& gw, const ColsumBlock* cs, int nx, int nw, int n_cs,
                       int cs_chunks, hipStream_t st) {
  constexpr int lds = std::max(split_lds(TX, BF16), split_lds(TW, BF16));
  if (lds > 64 * 1024)
    if (int rc = allow_large_lds<gemm_split_bwd_kernel<BF16, TX, TW, VEC>>()) return rc;
  const int n = nx + nw + n_cs * cs_chunks;
  hipLaunchKernelGGL((gemm_split_bwd_kernel<BF16, TX, TW, VEC>), grid_of_workgroups(n), dim3(256), lds, st, gx, gw, cs, nx, nw, n,
                     std::max(cs_chunks, 1));
  return DISTDL_OK;
}

int launch_gemm_split_bwd(const GemmBlock* d_bx, const std::vector<GemmBlock>& bx, const GemmSplitPlan& px,
                          const GemmBlock* d_bw, const std::vector<GemmBlock>& bw, const GemmSplitPlan& pw,
                          const ColsumBlock* d_cs, int n_cs, int max_f, bool bf16, float* partial, hipStream_t st) {
  ProfScope prof("affine_bwd_split", st);
  const SplitGrid gx = grid_of(d_bx, bx.size(), px, partial);
  const SplitGrid gw = grid_of(d_bw, bw.size(), pw, partial + px.partial_floats);
  const int chunks = d_cs ? (max_f + 15) / 16 : 0;
  if (!d_cs) n_cs = 0;
  int rc;
#define DISTDL_BWD(BF_, TX_, TW_, V_) rc = bwd_variant<BF_, TX_, TW_, V_>(gx, gw, d_cs, px.wgs, pw.wgs, n_cs, chunks, st)
  const bool vec = px.vec && pw.vec;
  if (bf16) DISTDL_BWD(true, 1, 1, false);
  else if (!vec) DISTDL_BWD(false, 1, 1, false);
  else if (px.T == 2 && pw.T == 2) DISTDL_BWD(false, 2, 2, true);
  else if (px.T == 2) DISTDL_BWD(false, 2, 1, true);
  else if (pw.T == 2) DISTDL_BWD(false, 1, 2, true);
  else DISTDL_BWD(false, 1, 1, true);
#undef DISTDL_BWD
  if (rc) return rc;
  launch_reduce(gx, gw, !bf16 && (px.nsplit <= 1 || quad_rows(bx)) && (pw.nsplit <= 1 || quad_rows(bw)), bf16, st);
  return DISTDL_OK;
}

}  // namespace distdl
