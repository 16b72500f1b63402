// The weights of a convolution launch, laid out in the order its kernel stages them: work of its own that is small and reads
// nothing but the caller's weights, so it rides as extra workgroups in a launch that runs before the convolution anyway: the
// halo exchange of the forward pass, the reduction of the partial weight gradients of the adjoint.  (A launch of its own takes
// 3 to 5 us, and a pass has two.  Eight launches, now six: 12 -> 55 channels, 7 taps, stride 2, 15 x 952 cells 51.0 and 46.3 us;
// 20 -> 4, 3^3, 9 x 4^3 59.6 and 55.1; 32 <- 3, 7 x 7, stride 2, 8 x 224 x 224 101 and 94.)
#pragma once
#include "common.h"
#include "conv_mfma.h"
#include "split_bf16.h"

#include <type_traits>

namespace distdl {

// ---- conv_split.hip -------------------------------------------------------------

constexpr int kMaxGroups = 32, kMaxTaps = 64, kMaxOff2 = 40;

struct SplitArgs {
  CorrArgs c;
  int32_t ci, co, taps, k1, k2;
  int64_t woff;                             // first weight piece
  int32_t ngroups;
  int32_t gbegin[kMaxGroups + 1];           // taps of group i: gbegin[i] ... gbegin[i + 1]
  int32_t gbase[kMaxGroups][2];             // input offset of the group's first patch row / cell (of position 0)
  int32_t tapcell[kMaxTaps];                // patch cell of a tap for position 0
  uint8_t tap12[kMaxTaps][2];               // its indices along dimensions 1 and 2
  int32_t fold, nch;                        // cells along dimension 2 that are one position's columns; channels of a cell
  FastDiv div_nch;
  int32_t dil2;
  int32_t off2[kMaxOff2];                   // input offset of tap i along dimension 2
  int32_t nfull, npairs;                    // chunks of 16 channels; MFMAs of a last chunk of at most 8 (0: there is none)
  int32_t hbegin[kMaxGroups + 1];           // of these those of group i
};

// The arguments of a launch of several classes lie in a table of the plan's; read through the constant address space its
// entries are scalar loads.
typedef const __attribute__((address_space(4))) SplitArgs* TablePtr;
__device__ inline TablePtr args_at(const SplitArgs* tab, int i) { return (TablePtr)(uintptr_t)(tab + i); }
// The layer's tap along dimension 2 that joins tap `i2` of a launch with cell j of a position's; negative: none.
template <class ArgsPtr>
__device__ inline int tap2_of(ArgsPtr a, int i2, int j) {
  const auto& c = a->c;
  if (a->fold == 1) return c.tapid[2][i2];
  const int at = c.mode == 0 ? a->off2[i2] - j * c.s[2] : j - a->off2[i2] * c.s[2];
  return at < 0 || at % a->dil2 != 0 || at / a->dil2 >= a->k2 ? -1 : at / a->dil2;
}

// eight channels of a weight piece: k0 ... of column col, tap `tap` (in group order) of kernel plane t0
template <class ArgsPtr>
__device__ inline void split_weight_octet(ArgsPtr a, const float* __restrict__ w, int t0, int k0, int tap, int col, float (&v)[8]) {
  const auto& c = a->c;
  const FastDiv div_nch{a->div_nch.mul, a->div_nch.sh1, a->div_nch.sh2, a->div_nch.d};
  const int j = a->fold > 1 ? (int)fd_div((uint32_t)col, div_nch) : 0, ch = col - j * a->nch, t2 = tap2_of(a, a->tap12[tap][1], j);
  const int ft = (c.tapid[0][t0] * a->k1 + c.tapid[1][a->tap12[tap][0]]) * a->k2 + t2;
  const int left = col < c.nc && t2 >= 0 ? c.kc - k0 : 0;
  const size_t per_k = c.mode == 0 ? (size_t)a->taps : (size_t)a->ci * a->taps;
  const float* const at = w + (left <= 0 ? (size_t)0 : c.mode == 0 ? ((size_t)ch * a->ci + k0) * a->taps + ft : ((size_t)k0 * a->ci + ch) * a->taps + ft);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = at[e < left ? e * per_k : (size_t)0];
  // (loaded in any case and all at once: left alone the compiler makes a branch, and a wait, of each)
#pragma unroll
  for (int e = 0; e < 8; ++e) asm volatile("" : "+v"(v[e]));
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = e < left ? v[e] : 0.f;
}

// Weights in the order the kernel stages them: pieces [ntile][t0][chunk][tap in group order][plane][h][nn], 8 channels
// k = 16 chunk + 8 h ... each of column ntile * 32 + nn; a last chunk of at most 8 channels instead [pair of taps][plane][h]
// [nn], those of the pair's tap h; zero beyond the channel counts and taps.  One thread per piece of all three planes.
__device__ inline void split_weights(TablePtr a, const float* __restrict__ w, split_u32x4* __restrict__ dst, int idx) {
  const auto& c = a->c;
  const int ntaps = a->gbegin[a->ngroups], whole = a->nfull * ntaps, per_t0 = whole + a->npairs;
  if (idx >= c.ntn * c.nt[0] * per_t0 * 64) return;
  const int nn = idx & 31, h = (idx >> 5) & 1;
  int r = idx >> 6;
  const int at_t0 = r % per_t0; r /= per_t0;
  const int t0 = r % c.nt[0], ntile = r / c.nt[0];
  int cc = at_t0 / ntaps, k0 = cc * 16 + h * 8, tap = at_t0 - cc * ntaps;
  bool there = true;
  if (at_t0 >= whole) {
    const int pair = at_t0 - whole;
    int gr = 0;
    while (a->hbegin[gr + 1] <= pair) ++gr;
    tap = a->gbegin[gr] + 2 * (pair - a->hbegin[gr]) + h;
    there = tap < a->gbegin[gr + 1];
    if (!there) tap = 0;
    k0 = a->nfull * 16;
  }
  float v[8];
  split_weight_octet(a, w, t0, k0, tap, there ? ntile * 32 + nn : c.nc, v);
  split_u32x4 hi, mid, lo;
  split_eight(v, kSplitScale, hi, mid, lo);
  split_u32x4* const at = dst + a->woff + (size_t)(idx >> 6) * 192 + (idx & 63);
  at[0] = hi;
  at[64] = mid;
  at[128] = lo;
}

// ---- conv_any.hip -----------------------------------------------------------------

constexpr int kMaxCls = 64;

struct AnyArgs {
  int32_t mode;          // 0: forward, 1: data gradient
  int32_t n_b, kc, nc;   // batch, contraction channels, output channels
  int32_t k[3], s[3], dil[3];
  int32_t n_workers, ntn, ncls, tiles_max;
  int32_t ci, co, taps;
  int32_t run;             // taps along dimension 2 whose channels are one run of k (octets of runs; 1: of taps)
  const split_u32x4* wt;         // weights as operand pieces
  const void* w;           // the caller's weights
  const void* bias;        // may be null
  int32_t woff[kMaxCls];   // first octet of a class's weights
};

template <bool BF16>
struct Elem {
  typedef float T;
};
template <>
struct Elem<true> {
  typedef uint16_t T;
};

__host__ __device__ inline int gcd_of(int a, int b) {
  while (b) {
    const int t = a % b;
    a = b, b = t;
  }
  return a;
}
// taps along one dimension of parity class `par`: t * dil == par modulo s
__host__ __device__ inline void class_taps(int k, int s, int dil, int par, int& nt, int& tf, int& ts) {
  ts = s / gcd_of(dil, s);
  tf = 0;
  while (tf < ts && (tf * dil) % s != par) ++tf;
  nt = tf < ts && tf < k ? (k - 1 - tf) / ts + 1 : 0;
}
constexpr int planes_of(bool bf16) { return bf16 ? 1 : 3; }
constexpr int kOctPad = 16;  // a class's weights are padded to whole stages of either kind

// eight values -> the operand pieces of one (octet, row); RAW: as they are, for fp32 MFMAs
template <bool BF16, bool RAW = false>
__device__ inline void put_octet(char* at, uint32_t plane, const float (&v)[8]) {
  if constexpr (BF16) {
    split_u32x4 h;
#pragma unroll
    for (int j = 0; j < 4; ++j) h[j] = pack_bf16(v[2 * j], v[2 * j + 1]);  // exact
    *(split_u32x4*)at = h;
  } else if constexpr (RAW) {
    split_u32x4 u, w;
    halve_eight(v, u, w);
    *(split_u32x4*)at = u;
    *(split_u32x4*)(at + plane) = w;
  } else {
    split_u32x4 h, m, l;
    split_eight(v, kSplitScale, h, m, l);
    *(split_u32x4*)at = h;
    *(split_u32x4*)(at + plane) = m;
    *(split_u32x4*)(at + 2 * plane) = l;
  }
}

// octet `oct` of output channel ch of a class: the weights, or zero beyond the channels, runs and taps
template <bool BF16, bool FLAT>
__device__ inline void any_weight_octet(const AnyArgs& a, const int (&nt)[3], const int (&tf)[3], const int (&ts)[3], int oct, int ch,
                                    float (&v)[8]) {
  const int n2 = FLAT ? nt[2] : nt[2] / a.run, ntaps = nt[0] * nt[1] * n2, len = FLAT ? a.kc : a.run * a.kc, noct = (len + 7) / 8;
  bool ok[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    int tap, c;
    if (FLAT) {
      const int k = oct * 8 + e;
      tap = k / a.kc, c = k - tap * a.kc;
    } else {
      tap = oct / noct, c = (oct - tap * noct) * 8 + e;
    }
    ok[e] = tap < ntaps && c < len && ch < a.nc;
    int i2 = tap % n2;
    const int i01 = tap / n2, i1 = i01 % nt[1], i0 = i01 / nt[1];
    if (!FLAT && a.run > 1) i2 = c / a.kc, c -= i2 * a.kc;
    const int t = ((tf[0] + i0 * ts[0]) * a.k[1] + tf[1] + i1 * ts[1]) * a.k[2] + tf[2] + i2 * ts[2];
    const int oc = a.mode == 0 ? ch : c, ic = a.mode == 0 ? c : ch;
    v[e] = ld((const typename Elem<BF16>::T*)a.w, ok[e] ? ((size_t)oc * a.ci + ic) * a.taps + t : (size_t)0);
  }
  // (loaded in any case and all at once: left alone the compiler makes a branch, and a wait, of each)
#pragma unroll
  for (int e = 0; e < 8; ++e) asm volatile("" : "+v"(v[e]));
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = ok[e] ? v[e] : 0.f;
}

// Weights as the correlation stages them: pieces [class][column tile][octet][plane][column], 8 k each; zero beyond the
// channels and taps.  One thread per (column tile, octet, column), all planes.
template <bool BF16, bool FLAT>
__device__ inline void any_weights(const AnyArgs& a, split_u32x4* __restrict__ dst, int cols, int cls, int idx) {
  constexpr int PL = planes_of(BF16);
  const int par[3] = {cls / (a.s[1] * a.s[2]), cls / a.s[2] % a.s[1], cls % a.s[2]};
  int nt[3], tf[3], ts[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    if (a.mode == 0) nt[d] = a.k[d], tf[d] = 0, ts[d] = 1;
    else class_taps(a.k[d], a.s[d], a.dil[d], par[d], nt[d], tf[d], ts[d]);
  }
  const int ntaps = nt[0] * nt[1] * nt[2];
  const int K = FLAT ? ntaps * a.kc : ntaps / a.run * ((a.run * a.kc + 7) / 8) * 8, octs = (K + 8 * kOctPad - 1) / (8 * kOctPad) * kOctPad;
  if (idx >= a.ntn * octs * cols) return;
  const int col = idx % (cols), r = idx / (cols), oct = r % octs, ntile = r / octs;
  float v[8];
  any_weight_octet<BF16, FLAT>(a, nt, tf, ts, oct, ntile * cols + col, v);
  split_u32x4* const at = dst + ((size_t)a.woff[cls] * a.ntn + (size_t)ntile * octs + oct) * (PL * cols) + col;
  put_octet<BF16>((char*)at, cols * 16, v);
}

// ---- the job ------------------------------------------------------------------------

struct WeightJob {
  int32_t kind = 0;               // 0: nothing to do, 1: of conv_split, 2: of conv_any
  int32_t per_class = 0;          // blocks of a class
  int32_t blocks = 0;             // in all
  int32_t at = 0;                 // the first of them in the launch
  const SplitArgs* tab = nullptr; // kind 1: classes tab[first] ...
  int32_t first = 0;
  int32_t cols = 0;               // kind 2
  int32_t bf16 = 0, flat = 0;
  const void* w = nullptr;
  split_u32x4* dst = nullptr;
  AnyArgs any = {};
};

// (blocks of 256 threads)
__device__ inline void run_weight_job(const WeightJob& j, int block) {
  const int cls = block / j.per_class, idx = (block - cls * j.per_class) * 256 + (int)threadIdx.x;
  if (j.kind == 1) split_weights(args_at(j.tab, j.first + cls), (const float*)j.w, j.dst, idx);
  else if (j.bf16 && j.flat) any_weights<true, true>(j.any, j.dst, j.cols, cls, idx);
  else if (j.bf16) any_weights<true, false>(j.any, j.dst, j.cols, cls, idx);
  else if (j.flat) any_weights<false, true>(j.any, j.dst, j.cols, cls, idx);
  else any_weights<false, false>(j.any, j.dst, j.cols, cls, idx);
}

// What a launch that may carry a job takes as its argument.
struct NoJob {};
template <bool JOB>
using JobArg = std::conditional_t<JOB, WeightJob, NoJob>;

int launch_weight_job(const WeightJob& job, hipStream_t st);  // on its own
// x <- H x; a job that the launch carried has kind 0 afterwards
int run_halo_with(distdl_plan* p, bool adjoint, PtrTable& tab, void* const* bufs_host, WeightJob* job, hipStream_t st);

}  // namespace distdl
