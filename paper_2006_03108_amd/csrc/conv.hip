// Partitioned convolution (Sec. 4, Forward / Adjoint Convolution Algorithms
// with P_co = P_ci = 1): x <- H x, the local cross-correlation on every
// worker's padded buffer, and in the adjoint the local [dConv]*, the
// sum-reduce of dw / db over workers and H* on dx.
//
// Layout: channels-last.  x^ is [n_b][B0][B1][B2][Ci], y is [n_b][O0][O1][O2][Co],
// weights arrive as [Co][Ci][T] (T = taps, last fastest) and are re-laid out
// once per call: by each family of kernels in its own order, by the direct
// kernels here into wt[T][Ci][Co], so that the output-channel axis is the
// contiguous one.
//
// This file: the calls, the choice of kernels, the reduction of dw / db, and
// the direct kernels, which take what no other does (tensors of 2 GiB and
// more, over 64 stride classes).
#include <algorithm>
#include <cmath>

#include "common.h"
#include "conv_any.h"
#include "conv_core.h"
#include "conv_fused.h"
#include "conv_mfma.h"
#include "conv_split.h"
#include "conv_wsplit.h"
#include "profile.h"
#include "ranges.h"
#include "weight_job.h"

namespace distdl {

int plan_prepare_device(distdl_plan* p);
int run_halo(distdl_plan* p, bool adjoint, PtrTable& tab, void* const* bufs_host, hipStream_t st);

struct ConvDev {
  int32_t n_b, ci, co;
  int32_t k[3], s[3], dil[3];
  int32_t taps;
};

static ConvDev conv_params(const distdl_plan* p) {
  ConvDev c;
  c.n_b = (int32_t)p->n_b;
  c.ci = (int32_t)p->n_ci;
  c.co = (int32_t)p->n_co;
  c.taps = 1;
  for (int d = 0; d < 3; ++d) {
    c.k[d] = p->ksize[d];
    c.s[d] = p->stride[d];
    c.dil[d] = p->dilation[d];
    c.taps *= p->ksize[d];
  }
  return c;
}

// wt[(t*Ci + ci)*Co + co] = w[(co*Ci + ci)*T + t]
template <class T>
__global__ void relayout_w_kernel(const T* __restrict__ w, float* __restrict__ wt, int co_n, int ci_n, int taps) {
  int idx = blockIdx.x * blockDim.x + threadIdx.x;
  int total = co_n * ci_n * taps;
  if (idx >= total) return;
  int co = idx % co_n;
  int r = idx / co_n;
  int ci = r % ci_n;
  int t = r / ci_n;
  wt[idx] = ld(w, ((size_t)co * ci_n + ci) * taps + t);
}

// ---- reference-shaped kernels: any D, stride, dilation, channel count -------

template <class T>
__global__ __launch_bounds__(256) void conv_fwd_direct_kernel(const WorkerDev* __restrict__ workers,
                                                              void* const* x_bufs, const float* __restrict__ wt,
                                                              const T* __restrict__ bias, void* const* y_bufs,
                                                              ConvDev c) {
  const WorkerDev wd = workers[blockIdx.y];
  const int64_t total = (int64_t)c.n_b * wd.out[0] * wd.out[1] * wd.out[2] * c.co;
  int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const T* __restrict__ x = (const T*)x_bufs[blockIdx.y];
  T* __restrict__ y = (T*)y_bufs[blockIdx.y];
  int co = (int)(idx % c.co);
  int64_t r = idx / c.co;
  int o2 = (int)(r % wd.out[2]); r /= wd.out[2];
  int o1 = (int)(r % wd.out[1]); r /= wd.out[1];
  int o0 = (int)(r % wd.out[0]);
  int n = (int)(r / wd.out[0]);
  float acc = bias ? ld(bias, co) : 0.f;
  const int64_t s2 = c.ci, s1 = (int64_t)wd.buf[2] * s2, s0 = (int64_t)wd.buf[1] * s1, sn = (int64_t)wd.buf[0] * s0;
  const T* xn = x + n * sn;
  int t = 0;
  for (int t0 = 0; t0 < c.k[0]; ++t0)
    for (int t1 = 0; t1 < c.k[1]; ++t1)
      for (int t2 = 0; t2 < c.k[2]; ++t2, ++t) {
        const T* xc = xn + (wd.origin[0] + o0 * c.s[0] + t0 * c.dil[0]) * s0 +
                          (wd.origin[1] + o1 * c.s[1] + t1 * c.dil[1]) * s1 +
                          (wd.origin[2] + o2 * c.s[2] + t2 * c.dil[2]) * s2;
        const float* wp = wt + (size_t)t * c.ci * c.co + co;
        for (int ci = 0; ci < c.ci; ++ci) acc = fmaf(wp[(size_t)ci * c.co], ld(xc, ci), acc);
      }
  st(y, idx, acc);
}

// dx^[n][cell][ci] over the whole padded buffer (cells no output reads get 0).
template <class T>
__global__ __launch_bounds__(256) void conv_bwd_data_direct_kernel(const WorkerDev* __restrict__ workers,
                                                                   void* const* dy_bufs, const float* __restrict__ wt,
                                                                   void* const* dx_bufs, ConvDev c) {
  const WorkerDev wd = workers[blockIdx.y];
  const int64_t total = (int64_t)c.n_b * wd.buf[0] * wd.buf[1] * wd.buf[2] * c.ci;
  int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const T* __restrict__ dy = (const T*)dy_bufs[blockIdx.y];
  T* __restrict__ dx = (T*)dx_bufs[blockIdx.y];
  int ci = (int)(idx % c.ci);
  int64_t r = idx / c.ci;
  int c2 = (int)(r % wd.buf[2]); r /= wd.buf[2];
  int c1 = (int)(r % wd.buf[1]); r /= wd.buf[1];
  int c0 = (int)(r % wd.buf[0]);
  int n = (int)(r / wd.buf[0]);
  const int64_t so2 = c.co, so1 = (int64_t)wd.out[2] * so2, so0 = (int64_t)wd.out[1] * so1,
                son = (int64_t)wd.out[0] * so0;
  float acc = 0.f;
  int t = 0;
  for (int t0 = 0; t0 < c.k[0]; ++t0) {
    int q0 = c0 - wd.origin[0] - t0 * c.dil[0];
    bool ok0 = q0 >= 0 && q0 % c.s[0] == 0 && q0 / c.s[0] < wd.out[0];
    for (int t1 = 0; t1 < c.k[1]; ++t1) {
      int q1 = c1 - wd.origin[1] - t1 * c.dil[1];
      bool ok1 = q1 >= 0 && q1 % c.s[1] == 0 && q1 / c.s[1] < wd.out[1];
      for (int t2 = 0; t2 < c.k[2]; ++t2, ++t) {
        int q2 = c2 - wd.origin[2] - t2 * c.dil[2];
        bool ok2 = q2 >= 0 && q2 % c.s[2] == 0 && q2 / c.s[2] < wd.out[2];
        if (!(ok0 && ok1 && ok2)) continue;
        const T* dyc = dy + n * son + (q0 / c.s[0]) * so0 + (q1 / c.s[1]) * so1 + (q2 / c.s[2]) * so2;
        const float* wp = wt + ((size_t)t * c.ci + ci) * c.co;
        for (int co = 0; co < c.co; ++co) acc = fmaf(wp[co], ld(dyc, co), acc);
      }
    }
  }
  st(dx, idx, acc);
}

// Partial dw^ / db^ of one worker over one chunk of its (n, o) positions, in
// the wt layout followed by Co bias slots.
template <class T>
__global__ __launch_bounds__(256) void conv_bwd_weight_direct_kernel(const WorkerDev* __restrict__ workers,
                                                                     void* const* x_bufs, void* const* dy_bufs,
                                                                     float* __restrict__ partial, ConvDev c,
                                                                     int nchunks) {
  const int worker = blockIdx.z, chunk = blockIdx.y;
  const WorkerDev wd = workers[worker];
  const int nw = c.taps * c.ci * c.co;
  int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= nw + c.co) return;
  const T* __restrict__ x = (const T*)x_bufs[worker];
  const T* __restrict__ dy = (const T*)dy_bufs[worker];
  const int64_t npos = (int64_t)c.n_b * wd.out[0] * wd.out[1] * wd.out[2];
  const int64_t per = (npos + nchunks - 1) / nchunks;
  const int64_t p0 = chunk * per, p1 = std::min<int64_t>(npos, p0 + per);
  float acc = 0.f;
  if (idx >= nw) {  // bias gradient slot
    int co = idx - nw;
    for (int64_t p = p0; p < p1; ++p) acc += ld(dy, p * c.co + co);
  } else {
    int co = idx % c.co;
    int r = idx / c.co;
    int ci = r % c.ci;
    int t = r / c.ci;
    int t2 = t % c.k[2];
    int t1 = (t / c.k[2]) % c.k[1];
    int t0 = t / (c.k[2] * c.k[1]);
    const int64_t s2 = c.ci, s1 = (int64_t)wd.buf[2] * s2, s0 = (int64_t)wd.buf[1] * s1,
                  sn = (int64_t)wd.buf[0] * s0;
    for (int64_t p = p0; p < p1; ++p) {
      int64_t rr = p;
      int o2 = (int)(rr % wd.out[2]); rr /= wd.out[2];
      int o1 = (int)(rr % wd.out[1]); rr /= wd.out[1];
      int o0 = (int)(rr % wd.out[0]);
      int n = (int)(rr / wd.out[0]);
      const float xv = ld(x, n * sn + (wd.origin[0] + o0 * c.s[0] + t0 * c.dil[0]) * s0 +
                                (wd.origin[1] + o1 * c.s[1] + t1 * c.dil[1]) * s1 +
                                (wd.origin[2] + o2 * c.s[2] + t2 * c.dil[2]) * s2 + ci);
      acc = fmaf(ld(dy, p * c.co + co), xv, acc);
    }
  }
  partial[((size_t)worker * nchunks + chunk) * (nw + c.co) + idx] = acc;
}

// R dw^, R db^ (Sec. 4, adjoint algorithm): sum the partials in worker order
// and write dw in the caller's [Co][Ci][T] shape.
template <int E, class T, bool JOB>
__global__ __launch_bounds__(256) void conv_reduce_dw_kernel(const float* __restrict__ partial, int nparts,
                                                             T* __restrict__ dw, T* __restrict__ db, ConvDev c, JobArg<JOB> job) {
  if constexpr (JOB) {  // (the data gradient's weights)
    if ((int)blockIdx.x >= job.at) return run_weight_job(job, (int)blockIdx.x - job.at);
  }
  // E elements per block, L = 256 / E lanes of partials each (few elements: more lanes, so that the launch still
  // has enough blocks); every lane adds its partials in ascending order (four independent chains for latency),
  // the lanes are then combined in ascending order
  constexpr int L = 256 / E;
  const int nw = c.taps * c.ci * c.co;
  const int e = threadIdx.x % E, lanep = threadIdx.x / E;
  const int idx = blockIdx.x * E + e;
  const size_t slot = (size_t)nw + c.co;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  if (idx < nw + c.co) {
    int p = lanep;
    for (; p + 3 * L < nparts; p += 4 * L)
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] += partial[(size_t)(p + L * u) * slot + idx];
    for (; p < nparts; p += L) acc[0] += partial[(size_t)p * slot + idx];
  }
  __shared__ float red[L][E];
  red[lanep][e] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  __syncthreads();
  if (lanep != 0 || idx >= nw + c.co) return;
  float sum = red[0][e];
#pragma unroll
  for (int l = 1; l < L; ++l) sum += red[l][e];
  if (idx >= nw) {
    if (db) st(db, idx - nw, sum);
  } else {
    int co = idx % c.co;
    int r = idx / c.co;
    int ci = r % c.ci;
    int t = r / c.ci;
    st(dw, ((size_t)co * c.ci + ci) * c.taps + t, sum);
  }
}

static int direct_chunks(const distdl_plan* p) {
  ConvDev c = conv_params(p);
  int64_t nw = (int64_t)c.taps * c.ci * c.co + c.co;
  int64_t blocks = (nw + 255) / 256 * p->n_workers;
  int64_t want = (2048 + blocks - 1) / blocks;
  int64_t npos = p->n_b * p->max_out_cells;
  return (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(want, 64), npos));
}

static int check_conv_plan(const distdl_plan* p) {
  if (p->explicit_halo) return set_error(DISTDL_ERR_UNSUPPORTED, "conv: plan has no kernel (explicit halo plan)");
  return DISTDL_OK;
}

// The kernel of the forward pass and of the data gradient, by shape and alignment of the arrays (16 bytes).  The split kernels
// take any weights' alignment, the tiled ones do not.
enum class Corr { kDirect, kMfma, k16, kSplit, kAny };

//
// Among the three that make fp32 products of small layers, the one whose estimated time is the lowest, with an allowance for
// what the estimates do not know (each is off by up to a quarter): the 16 x 16 kernel stays unless another one and its weights,
// which make the launch before them 1 us longer (H) or 2 (the reduction of dw), take less than 0.85 of its time (all of it where
// its classes write every second cell of the last dimension: 8 -> 16 channels, 7 taps, stride 2, 9 x 33496, 70 us with an adjoint on
// it and 61 with the split kernel's), the split one
// (where it takes the layer) unless the gather kernel takes less than two thirds, or half if the split kernel's windows are full;
// the data gradient of few cells in two classes of a stride or more does not start from the 16 x 16 kernel, which has a launch for
// each (5 -> 10 channels, 5 x 5, stride 2, 15 x 84 x 79: 52 us, gather 27; 8 -> 9, 7 x 7, stride 1 x 2, 2 x 22 x 134: 34 and 17; of 70
// layers of two classes the choice is within 3 % of the fastest in the mean, 17 % when they start from it), but takes it only for
// less than three quarters of the time.  What decides: the split kernel's windows
// lie in one plane of one sample, so planes of a few cells leave them empty, where the gather kernel counts all positions
// through; the gather kernel fetches a cell for each tap; the 16 x 16 kernel has a launch for each class of a stride.  us,
// 16 x 16 / split / gather: forward 36 -> 24, 3^3, 6 x 13 x 13 x 11: - / 41 / 21; 8 -> 4, 7^3, stride 2, 13 x 11 x 16 x 15: 214 / 302 /
// 53; 16 -> 4, 3 x 3, 2 x 808 x 1000: 91 / 67 / 181; data gradient 12 -> 1, 3 x 3, stride 2, 15 x 727 x 494: 148 / 77 / -.
// Over 737 directions of 370 layers (1 to 64 channels, one to three dimensions, 100 to 20 M positions, every kernel and form
// measured) the choice takes 0.89 times what it starts from takes, in the mean, nine directions more than 1.03 times; and 1.10
// times the fastest.
static Corr choose_small(const distdl_plan* p, bool backward, bool aligned, bool k16, bool split) {
  const bool any = conv_any_supported(p);
  const int64_t classes = (int64_t)p->stride[0] * p->stride[1] * p->stride[2];
  const bool together = backward && classes >= 2 && p->n_workers * p->n_b * p->max_buf_cells <= (classes << 16) && (split || any);
  const bool apart = backward && p->stride[2] > 1;  // each class writes every stride[2]th cell, of at most 64 bytes
  const double ride = backward ? 2.0 : 1.0;
  Corr best = k16 && !together ? Corr::k16 : split ? Corr::kSplit : Corr::kAny;
  double us = best == Corr::k16 ? corr16_us(p, backward) * (apart ? 1.0 : 0.85) - ride : best == Corr::kSplit ? corr_split_us(p, backward) : corr_any_us(p, backward, aligned);
  if (k16 && together)
    if (const double t = corr16_us(p, backward) - ride; t < us * 0.75) us = t, best = Corr::k16;
  if (best == Corr::k16 && split)
    if (const double t = corr_split_us(p, backward); t < us) us = t, best = Corr::kSplit;
  if (any && corr_any_us(p, backward, aligned) < us * (best != Corr::kSplit ? 1.0 : corr_split_used(p, backward) < 0.5 ? 0.66 : 0.5))
    best = Corr::kAny;
  return best;
}

static bool wgrad_on_tiles(const distdl_plan* p);
static Corr choose_corr(const distdl_plan* p, bool backward, bool aligned, bool w_aligned) {
  int8_t& known = p->corr_kernel[backward][aligned][w_aligned];
  if (known >= 0) return (Corr)known;
  const bool k16 = backward ? corr16_bwd_supported(p, aligned) : corr16_fwd_supported(p, aligned);
  const bool split = aligned && corr_split_supported(p, backward);
  Corr c = conv_any_supported(p) ? Corr::kAny : Corr::kDirect;
  if (k16 || split) c = choose_small(p, backward, aligned, k16, split);
  else if (aligned && w_aligned && corr_mfma_supported(p)) {
    // bf16: 32-wide tiles or the gather kernel, by estimated time.  The tiles stage a cell once for all taps; they have a launch,
    // and another for the weights, for each class, windows in one plane of one sample, and channel counts that are no multiples
    // of 8 on fp32 MFMAs.  us, tiles (with their weights' launches) / gather: forward 32 -> 16, 3^3, stride 2, 2 x 101 x 95 x 100:
    // 66 / 79, data gradient 156 / 94; forward 44 -> 36, 3^3, 9 x 4 x 4 x 4: 179 / 17; data gradient 56 -> 8, 5 x 5, stride 2, 10 x 44 x 75:
    // 51 / 13; forward 12 -> 44, 3 x 3, 6 x 602 x 675: 430 / 163.  (Without estimates, tiles wherever they fit, a direction took 2.1
    // times the faster of the two in the mean of 166, with them 1.1.)
    // Layers whose weight gradient is on the tiles keep all three directions there: nearly all of them are large and faster that way
    // (32 -> 32, 5^3, stride 2, 256^3: forward 691 / 3900, data gradient 1090 / 2440; 24 -> 8, 3^3, 3 x 42 x 36 x 38: forward 23 / 42); the
    // data gradient of the few that are small and strided would not be.
    const bool gather = p->dtype == DISTDL_BF16 && conv_any_supported(p) && !wgrad_on_tiles(p) &&
                        corr_any_us(p, backward, aligned) < 0.8 * corr_mfma_us(p, backward);
    c = gather ? Corr::kAny : Corr::kMfma;
  }
  known = (int8_t)c;
  return c;
}
static Corr choose_fwd(const distdl_plan* p, bool xy_aligned, bool w_aligned) { return choose_corr(p, false, xy_aligned, w_aligned); }
static Corr choose_data(const distdl_plan* p, bool aligned) { return choose_corr(p, true, aligned, true); }

// The kernel of the weight gradient: of those that take the layer, the one whose estimated time (us) is the lowest:
//   16 x 16 tiles: a set-up that grows with the taps of a plane, then 7 ps per tap and position (12 with several planes);
//   gather: rounds of stages of 128 positions by 64 rows or 32 by 256, the tensors, the partials (tiles_of in conv_any.hip);
//   bf16 planes: 1.2 us a step of 32 positions or its matrix instructions;
//   split planes: its own estimate counts matrix instructions; 1.6 times that was taken.
// Tiles of 64 rows (bf16: of layers of at most 128) have to be estimated at less than 0.9 of another kernel (0.8 of the 16 x 16
// tiles, whose estimate is the surer): where the two are that close, either may be the faster, and their rounds and tensors vary more from layer to layer.
// A layer of at most 64 rows, one tile that reads x once, leaves the split kernel up to 1.1 of its estimate: most such layers
// have one tap, and the split kernel's estimate leaves out the tensors (us, split / gather: 56 -> 4, one tap, 8 x 884 x 841: 451 / 280,
// 12 -> 36, 7 x 449 x 365: 124 / 109; a forward pass and an adjoint of 56 -> 36, 7 x 66 x 57 x 74: 818 / 762).
// Over 680 fp32 layers of 1 to 64 channels, one to three dimensions, 10^2 to 2 x 10^7 positions, every kernel that takes each: the choice
// is within 3 % of the fastest in the mean.  us, 16 x 16 / gather / split: 16 -> 16 channels, 3 x 3, 8 x 256 x 256:
// 38.7 / 83 / 47; 4 -> 4, 5 x 5, 8 x 660 x 860: - / 318 / 222; 64 -> 64, 3^3, 2 x 40 x 44 x 48: - / 384 / 240; 16 -> 4, one
// dimension, 2 x 4000: - / 17 / 111; 32 -> 32, 5^3, stride 2, 256^3: - / 5030 / 3110.
enum class Wgrad { k16, kSplit, kAny, kMfma, kDirect };

static double wgrad_us(const distdl_plan* p, Wgrad w);
static Wgrad choose_wgrad(const distdl_plan* p, bool vec16) {
  if (p->wgrad_kernel[vec16] >= 0) return (Wgrad)p->wgrad_kernel[vec16];
  const bool bf16 = p->dtype == DISTDL_BF16;
  const double T = (double)p->ksize[1] * p->ksize[2];
  Wgrad best = Wgrad::kDirect;
  double least = 1e300;
  auto consider = [&](Wgrad w, double us) {
    if (us < least) least = us, best = w;
  };
  if (wgrad16_supported(p, vec16)) consider(Wgrad::k16, wgrad_us(p, Wgrad::k16));
  if (vec16 && wgrad_split_supported(p)) consider(Wgrad::kSplit, wgrad_us(p, Wgrad::kSplit));
  const bool fits = wgrad_mfma_supported(p) && p->n_workers * wgrad_chunks(p) <= 65535;
  if (fits && bf16 && vec16) consider(Wgrad::kMfma, wgrad_taps_us(p));
  if (conv_any_supported(p)) {
    const bool one_tile = p->ksize[0] * T * (double)p->n_ci <= 64;
    const double room = best == Wgrad::kDirect || !wgrad_any_unsure(p) ? 1.0 : best == Wgrad::k16 ? 0.8 : best == Wgrad::kSplit && one_tile ? 1.1 : 0.9;
    consider(Wgrad::kAny, wgrad_any_us(p) / room);
  }
  if (best == Wgrad::kDirect && fits && (!bf16 || vec16)) best = Wgrad::kMfma;
  p->wgrad_kernel[vec16] = (int)best;
  return best;
}

// estimated time of a kernel; 0: unknown
static double wgrad_us(const distdl_plan* p, Wgrad w) {
  const double T = (double)p->ksize[1] * p->ksize[2], pos = (double)p->n_workers * p->n_b * p->max_out_cells;
  switch (w) {
    case Wgrad::k16: return 6.0 + 0.8 * T + pos * p->ksize[0] * T * (p->ksize[0] > 1 ? 12e-6 : 7e-6);
    case Wgrad::kSplit: return 1.6 * wgrad_split_us(p);
    case Wgrad::kAny: return wgrad_any_us(p);
    case Wgrad::kMfma: return p->dtype == DISTDL_BF16 ? wgrad_taps_us(p) : 0;
    default: return 0;
  }
}

static bool wgrad_on_tiles(const distdl_plan* p) { return choose_wgrad(p, true) == Wgrad::kMfma; }

static int wgrad_partials(const distdl_plan* p, Wgrad w, bool vec16) {  // per worker
  switch (w) {
    case Wgrad::k16: return wgrad16_chunks(p, vec16);
    case Wgrad::kSplit: return wgrad_split_chunks(p);
    case Wgrad::kAny: return wgrad_any_chunks(p);
    case Wgrad::kMfma: return wgrad_chunks(p);
    default: return direct_chunks(p);
  }
}

// Small layers: everything of a direction in one launch (conv_fused.hip) where that is estimated at less than 0.8 (0.75 from 20 us; back
// 0.95) of the launches it replaces; theirs are H and its kernel, or both contractions, the reduction and H*, each estimated as above,
// and what the host takes for them; its time for the workers' arrays is on neither side.  Without a halo exchange there is one launch
// less to save; the forward pass then goes that way only where it would take little more than a launch.  us, launches apart /
// together, forward and back: 1 -> 1, 3 taps, 64 on four workers 11.7 / 6.8 and 18.0 / 8.6; 20 -> 4, 3^3, 4 x 13 x 12 x 17 on
// 3 x 2 x 2 26.8 / 14.1 and 38.5 / 22.4; but 5 -> 32, 5^3, stride 2, bf16, 13 x 14 x 11 x 15 22 / 45 and 58 / 400.  Up to 100 us
// forward and 40 us back, where the fp64 matrix instructions and the second reading of x weigh more than the launches (27 -> 11,
// 3 x 3, 10 x 244 x 329 258 / 283; 24 -> 4, 3^3, bf16, 11 x 62 x 54 x 61 1026 / 2498).
// Estimates are off by an eighth either way.  Of 4200 directions forward 2482 go together, 1.60 times as fast in the mean, 12 of them
// more than 0.15 slower than apart; at 0.9 and 0.85 45, for 1.325 instead of 1.318 over all.  Back 2401 of 3900, 1.68 times, 9 more
// than 0.15 slower; at 0.85 and 0.8 3, but 1.365 instead of 1.378 over all, and a hundred left apart that take a fifth longer so (5 -> 1,
// 3^3, dilated, 13 x 7 x 9 x 6 on 1 x 3 x 2 30.8 / 17.1).
static double arrays_us(const distdl_plan* p, bool backward) { return (backward ? 0.25 : 0.2) * p->n_workers; }  // the host's time for them, either way
static bool has_boxes(const distdl_plan* p) { return !p->fwd1.blocks.empty() || !p->fwd16.blocks.empty(); }
static double launches_us(const distdl_plan* p, bool backward) {  // and for the launches apart
  return (!backward ? 9.5 : has_boxes(p) ? 12.0 : 9.0) + arrays_us(p, backward);
}
static bool choose_fused(const distdl_plan* p, bool backward, bool vec, bool aligned, bool w_aligned) {
  int8_t& known = p->fused_kernel[backward][vec][aligned][w_aligned];
  if (known >= 0) return known != 0;
  const double us = conv_fused_us(p, backward, vec);
  const bool boxes = has_boxes(p);
  double apart = launches_us(p, backward);
  const double room = backward ? 0.95 : us < 20 ? 0.8 : 0.75, arrays = arrays_us(p, backward);
  if (us - arrays >= room * (apart - arrays) && std::isfinite(us) && (backward || boxes)) {
    const Corr k = choose_corr(p, backward, aligned, w_aligned);
    double corr = 0, wgrad = 0;
    if (k == Corr::k16) corr = corr16_us(p, backward);
    else if (k == Corr::kSplit) corr = corr_split_us(p, backward);
    else if (k == Corr::kAny) corr = corr_any_us(p, backward, aligned);
    else if (k == Corr::kMfma && p->dtype == DISTDL_BF16) corr = corr_mfma_us(p, backward);
    // (a weight gradient on the split kernel or the bf16 planes is one of a layer that fills the chip)
    const Wgrad wk = backward ? choose_wgrad(p, vec) : Wgrad::kAny;
    if (backward && (wk == Wgrad::kAny || wk == Wgrad::k16)) wgrad = wgrad_us(p, wk);
    const double device = backward ? (boxes ? 6.1 : 3.0) + 1.1 * corr + wgrad : 2.2 + 1.2 * corr;
    apart = corr <= 0 || (backward && wgrad <= 0) ? 0.0 : joined(apart, device);
  }
  known = us - arrays < room * (apart - arrays) && us < (backward ? 40 : 100);
  return known != 0;
}

// Where the reduction of dw lays out the weights of the data gradient, that comes last, and the launch after it waits for the write-back
// of dx; the weight gradient, which would hide that where it is long for the tensors it reads (the gather kernel with several taps),
// comes before.  For a large dx, far larger than dy, that costs more than the launch for the weights, 5 us.  us of a forward and
// backward pass with the data gradient last / first: 5 x 610884, 44 -> 12, 3 taps, 1052 / 1023 (5 x 305442 547 / 518, 5 x 200000 366 /
// 359, 5 x 100000 196 / 200; the forward pass of 60 -> 20, 5 taps, stride 2, 8 x 81385, after an adjoint of the one order 84 and of the
// other 74); 60 -> 4, 5 x 400000, 732 / 700; but one tap, whose weight gradient reads what the forward pass left in
// the caches, 722 / 750; 32 -> 16, 5 x 610884, 626 / 628; 12 -> 44 847 / 881; weight gradients of the split kernel 44 -> 12, 2^3,
// 3 x 100 x 101 x 102, 1585 / 1607; 24 -> 20, 3 x 3, 8 x 512^2, 638 / 643; 32 -> 32, 5^3, stride 2, 256^3, 10250 / 10280.
static bool write_back_hides(const distdl_plan* p, Corr kernel, Wgrad wgrad) {
  if (kernel != Corr::kSplit || wgrad != Wgrad::kAny) return false;
  const double x = 4.0 * p->n_workers * p->n_b * p->max_buf_cells * p->n_ci, dy = 4.0 * p->n_workers * p->n_b * p->max_out_cells * p->n_co;
  return x > 130e6 && x >= 2.5 * dy && wgrad_any_us(p) > 1.5 * (x + dy) / 4.6e6;
}

// The weights of a launch of `kernel` that a launch before it can lay out.
static int weight_job(distdl_plan* p, Corr kernel, bool backward, const void* w, bool aligned, hipStream_t st, WeightJob& job) {
  if (kernel == Corr::kSplit) return split_weight_job(p, backward, (const float*)w, st, job);
  return kernel == Corr::kAny ? any_weight_job(p, backward, w, aligned, st, job) : DISTDL_OK;
}

// The tables that go to the device with those of a plan whose first call is a fused forward pass: its own, and the adjoint's where they
// are few and it is likely to want them.  (A copy of their own takes 15 to 20 us of the first adjoint; 64 records take 3 us of a
// forward pass that may be all that the plan ever makes.)
static void fused_first_tables(const distdl_plan* p, bool vec) {
  conv_fused_make_tables(p, false);
  if (conv_fused_records(p, true) <= 64 && conv_fused_us(p, true, vec) < 1.25 * launches_us(p, true)) conv_fused_make_tables(p, true);
}

// Whether an output of a call lies on one of its inputs, or on another output: the fused kernels write y, and dx, dw and db, while
// the inputs are still being read.
static size_t x_bytes(const distdl_plan* p, int w) {
  const WorkerDev& wd = p->workers[w];
  return (size_t)p->n_b * wd.buf[0] * wd.buf[1] * wd.buf[2] * p->n_ci * dtype_size(p->dtype);
}
static size_t y_bytes(const distdl_plan* p, int w) {
  const WorkerDev& wd = p->workers[w];
  return (size_t)p->n_b * wd.out[0] * wd.out[1] * wd.out[2] * p->n_co * dtype_size(p->dtype);
}
static size_t w_bytes(const distdl_plan* p) { return (size_t)p->ksize[0] * p->ksize[1] * p->ksize[2] * p->n_ci * p->n_co * dtype_size(p->dtype); }
static bool fwd_overlaps(const distdl_plan* p, const void* const x[], const void* w, const void* bias, void* const y[]) {
  Ranges r((size_t)2 * p->n_workers + 2);
  r.one(w, w_bytes(p), false);
  r.one(bias, p->n_co * dtype_size(p->dtype), false);
  r.begin(false);
  for (int i = 0; i < p->n_workers; ++i) r.add(x[i], x_bytes(p, i));
  r.begin(true);
  for (int i = 0; i < p->n_workers; ++i) r.add(y[i], y_bytes(p, i));
  return r.clash();
}
static bool bwd_overlaps(const distdl_plan* p, const void* const x[], const void* w, const void* const dy[], void* const dx[], const void* dw,
                         const void* db, const void* ws, size_t ws_bytes) {
  Ranges r((size_t)3 * p->n_workers + 4);
  r.one(w, w_bytes(p), false);
  r.one(ws, ws_bytes, true);
  r.one(dw, w_bytes(p), true);
  r.one(db, p->n_co * dtype_size(p->dtype), true);
  r.begin(false);
  for (int i = 0; i < p->n_workers; ++i) r.add(x[i], x_bytes(p, i));
  r.begin(false);
  for (int i = 0; i < p->n_workers; ++i) r.add(dy[i], y_bytes(p, i));
  r.begin(true);
  for (int i = 0; i < p->n_workers; ++i) r.add(dx[i], x_bytes(p, i));
  return r.clash();
}

static int prepare_weights(distdl_plan* p, const void* w, hipStream_t st) {
  ConvDev c = conv_params(p);
  size_t n = (size_t)c.taps * c.ci * c.co;
  if (int rc = ensure_wscratch(p, n, st)) return rc;
  ProfScope prof("conv_relayout_w", st);
  if (p->dtype == DISTDL_BF16)
    hipLaunchKernelGGL(relayout_w_kernel<uint16_t>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                       (const uint16_t*)w, p->d_wt, c.co, c.ci, c.taps);
  else
    hipLaunchKernelGGL(relayout_w_kernel<float>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const float*)w,
                       p->d_wt, c.co, c.ci, c.taps);
  return DISTDL_OK;
}

}  // namespace distdl

using namespace distdl;

extern "C" {

size_t distdl_conv_bwd_workspace(const distdl_plan* plan) {
  if (!plan || plan->explicit_halo) return 0;
  ConvDev c = conv_params(plan);
  size_t nw = (size_t)c.taps * c.ci * c.co + c.co;
  const bool vec = plan->n_ci % 4 == 0 && plan->n_co % 4 == 0;  // (as for aligned and for any other tensors)
  const int chunks = std::max(wgrad_partials(plan, choose_wgrad(plan, vec), vec), wgrad_partials(plan, choose_wgrad(plan, false), false));
  return nw * sizeof(float) * plan->n_workers * chunks;
}

int distdl_conv_fwd(distdl_plan* plan, void* const x_bufs_dev[], const void* w_dev, const void* bias_dev,
                    void* const y_dev[], void* stream) {
  return distdl::conv_fwd_core(plan, x_bufs_dev, w_dev, bias_dev, y_dev, (hipStream_t)stream, true);
}

int distdl_conv_bwd(distdl_plan* plan, const void* const x_bufs_dev[], const void* w_dev, const void* const dy_dev[],
                    void* const dx_bufs_dev[], void* dw_dev, void* dbias_dev, void* workspace_dev,
                    size_t workspace_bytes, void* stream) {
  return distdl::conv_bwd_core(plan, x_bufs_dev, w_dev, dy_dev, dx_bufs_dev, dw_dev, dbias_dev, workspace_dev,
                               workspace_bytes, (hipStream_t)stream, true);
}

int distdl_debug_conv_path(const distdl_plan* plan, int32_t out[3]) {
  if (!plan || !out) return set_error(DISTDL_ERR_NULL, "conv_path: null argument");
  if (plan->explicit_halo) return set_error(DISTDL_ERR_UNSUPPORTED, "conv_path: plan has no kernel");
  // by shape and 16-byte aligned arrays; distdl_debug_conv_kernels says which kernels run
  const bool vec = plan->n_ci % 4 == 0 && plan->n_co % 4 == 0;
  const bool mfma = corr_mfma_supported(plan);
  out[0] = corr16_fwd_supported(plan, true) ? 2 : mfma ? 1 : 0;
  out[1] = corr16_bwd_supported(plan, true) ? 2 : mfma ? 1 : 0;
  out[2] = wgrad16_supported(plan, vec) ? 2 : (wgrad_mfma_supported(plan) && (plan->dtype != DISTDL_BF16 || vec)) ? 1 : 0;
  return DISTDL_OK;
}

int distdl_debug_conv_kernels(const distdl_plan* plan, int aligned, int32_t out[3]) {
  if (!plan || !out) return set_error(DISTDL_ERR_NULL, "conv_kernels: null argument");
  if (plan->explicit_halo) return set_error(DISTDL_ERR_UNSUPPORTED, "conv_kernels: plan has no kernel");
  auto code = [](Corr c) { return c == Corr::kMfma ? 1 : c == Corr::k16 ? 2 : c == Corr::kSplit ? 3 : c == Corr::kAny ? 4 : 0; };
  out[0] = code(choose_fwd(plan, aligned != 0, aligned != 0));
  out[1] = code(choose_data(plan, aligned != 0));
  const Wgrad w = choose_wgrad(plan, aligned && plan->n_ci % 4 == 0 && plan->n_co % 4 == 0);
  out[2] = w == Wgrad::kMfma ? 1 : w == Wgrad::k16 ? 2 : w == Wgrad::kSplit ? 3 : w == Wgrad::kAny ? 4 : 0;
  return DISTDL_OK;
}

int distdl_debug_conv_fused(const distdl_plan* plan, int aligned, int32_t out[2]) {
  if (!plan || !out) return set_error(DISTDL_ERR_NULL, "conv_fused: null argument");
  if (plan->explicit_halo) return set_error(DISTDL_ERR_UNSUPPORTED, "conv_fused: plan has no kernel");
  const bool vec = aligned && plan->n_ci % 4 == 0 && plan->n_co % 4 == 0;
  for (int backward = 0; backward < 2; ++backward) out[backward] = choose_fused(plan, backward != 0, vec, aligned != 0, backward || aligned == 1);
  return DISTDL_OK;
}

int distdl_debug_conv_split(const distdl_plan* plan, int backward, int32_t out[5]) {
  if (!plan || !out) return set_error(DISTDL_ERR_NULL, "conv_split: null argument");
  if (plan->explicit_halo) return set_error(DISTDL_ERR_UNSUPPORTED, "conv_split: plan has no kernel");
  corr_split_shape(plan, backward != 0, out);
  return DISTDL_OK;
}

int distdl_debug_conv_wgrad_rows(const distdl_plan* plan, int32_t* rows) {
  if (!plan || !rows) return set_error(DISTDL_ERR_NULL, "conv_wgrad_rows: null argument");
  if (plan->explicit_halo) return set_error(DISTDL_ERR_UNSUPPORTED, "conv_wgrad_rows: plan has no kernel");
  *rows = !conv_any_supported(plan) ? 0 : wgrad_any_rows(plan);
  return DISTDL_OK;
}

int distdl_conv_local_fwd(distdl_plan* plan, void* const x_bufs_dev[], const void* w_dev, const void* bias_dev,
                          void* const y_dev[], void* stream) {
  return distdl::conv_fwd_core(plan, x_bufs_dev, w_dev, bias_dev, y_dev, (hipStream_t)stream, false);
}

int distdl_conv_local_bwd(distdl_plan* plan, const void* const x_bufs_dev[], const void* w_dev,
                          const void* const dy_dev[], void* const dx_bufs_dev[], void* dw_dev, void* dbias_dev,
                          void* workspace_dev, size_t workspace_bytes, void* stream) {
  return distdl::conv_bwd_core(plan, x_bufs_dev, w_dev, dy_dev, dx_bufs_dev, dw_dev, dbias_dev, workspace_dev,
                               workspace_bytes, (hipStream_t)stream, false);
}

}  // extern "C"

namespace distdl {

// The two layer calls; `halo` = false leaves out H (forward) / H* (backward) for callers that apply them
// themselves (the channel-partitioned layer exchanges halos once per input block, not once per weight block).
int conv_fwd_core(distdl_plan* plan, void* const x_bufs_dev[], const void* w_dev, const void* bias_dev,
                  void* const y_dev[], hipStream_t st, bool halo) {
  if (!plan || !x_bufs_dev || !w_dev || !y_dev) return set_error(DISTDL_ERR_NULL, "conv_fwd: null argument");
  int rc = check_conv_plan(plan);
  if (rc) return rc;
  const bool bf16 = plan->dtype == DISTDL_BF16;
  const uintptr_t esz = bf16 ? 2 : 4;
  for (int w = 0; w < plan->n_workers; ++w)
    if (!y_dev[w] || (uintptr_t)y_dev[w] % esz) return set_error(DISTDL_ERR_NULL, "conv_fwd: y of worker %d null or misaligned", w);
  // 16-byte pieces on both sides: the matrix-core kernels load x in them and store y in them
  bool xvec = true;
  for (int w = 0; w < plan->n_workers; ++w) xvec &= (uintptr_t)x_bufs_dev[w] % 16 == 0 && (uintptr_t)y_dev[w] % 16 == 0;
  const bool vec = xvec && plan->n_ci % 4 == 0 && plan->n_co % 4 == 0;
  const bool w_aligned = (uintptr_t)w_dev % 16 == 0;
  const bool fused = halo && choose_fused(plan, false, vec, xvec, w_aligned) && conv_fused_ready(plan, false, st) &&
                     !fwd_overlaps(plan, x_bufs_dev, w_dev, bias_dev, y_dev);
  if (fused && !plan->d_workers) fused_first_tables(plan, vec);
  const Corr kernel = fused ? Corr::kDirect : choose_fwd(plan, xvec, w_aligned);
  if ((rc = plan_prepare_device(plan))) return rc;
  for (int w = 0; w < plan->n_workers; ++w) {
    if (!x_bufs_dev[w]) return set_error(DISTDL_ERR_NULL, "conv_fwd: x of worker %d is null", w);
    if ((uintptr_t)x_bufs_dev[w] % esz) return set_error(halo ? DISTDL_ERR_INVALID_ARG : DISTDL_ERR_NULL, "conv_fwd: x of worker %d is misaligned", w);
  }
  // The pointer tables first: they refuse a call that has not been made on a stream that is being captured, before anything is
  // enqueued or allocated (which would end the capture).
  if ((rc = plan->tab_x.upload((const void* const*)x_bufs_dev, plan->n_workers, st))) return rc;
  if ((rc = plan->tab_y.upload((const void* const*)y_dev, plan->n_workers, st))) return rc;
  if (fused) {
    bool wide = !plan->fwd16.tasks.empty();
    for (int w = 0; w < plan->n_workers; ++w) wide &= (uintptr_t)x_bufs_dev[w] % 16 == 0;
    if ((rc = conv_fwd_fused(plan, w_dev, bias_dev, vec, wide, st))) return rc;
    DISTDL_HIP_TRY(hipGetLastError());
    return DISTDL_OK;
  }
  WeightJob job;
  if ((rc = weight_job(plan, kernel, false, w_dev, xvec, st, job))) return rc;
  if (halo && (rc = run_halo_with(plan, false, plan->tab_x, x_bufs_dev, &job, st))) return rc;  // x <- H x
  if ((rc = launch_weight_job(job, st))) return rc;  // (where H has no launch)
  if (kernel != Corr::kDirect) {
    switch (kernel) {
      case Corr::k16: rc = conv_fwd16(plan, (const float*)w_dev, (const float*)bias_dev, xvec, st); break;
      case Corr::kSplit: rc = conv_fwd_split(plan, (const float*)w_dev, (const float*)bias_dev, st); break;
      case Corr::kMfma: rc = conv_fwd_mfma(plan, w_dev, bias_dev, st); break;
      default: rc = conv_fwd_any(plan, w_dev, bias_dev, xvec, st);
    }
    if (rc) return rc;
    DISTDL_HIP_TRY(hipGetLastError());
    return DISTDL_OK;
  }
  if ((rc = prepare_weights(plan, w_dev, st))) return rc;
  ConvDev c = conv_params(plan);
  int64_t total = plan->n_b * plan->max_out_cells * c.co;
  dim3 grid((unsigned)((total + 255) / 256), plan->n_workers);
  ProfScope prof("conv_fwd_direct", st);
  if (bf16)
    hipLaunchKernelGGL(conv_fwd_direct_kernel<uint16_t>, grid, dim3(256), 0, st, plan->d_workers, plan->tab_x.dev,
                       plan->d_wt, (const uint16_t*)bias_dev, plan->tab_y.dev, c);
  else
    hipLaunchKernelGGL(conv_fwd_direct_kernel<float>, grid, dim3(256), 0, st, plan->d_workers, plan->tab_x.dev,
                       plan->d_wt, (const float*)bias_dev, plan->tab_y.dev, c);
  DISTDL_HIP_TRY(hipGetLastError());
  return DISTDL_OK;
}

int conv_bwd_core(distdl_plan* plan, const void* const x_bufs_dev[], const void* w_dev, const void* const dy_dev[],
                  void* const dx_bufs_dev[], void* dw_dev, void* dbias_dev, void* workspace_dev, size_t workspace_bytes,
                  hipStream_t st, bool halo) {
  if (!plan || !x_bufs_dev || !w_dev || !dy_dev || !dx_bufs_dev || !dw_dev || !workspace_dev)
    return set_error(DISTDL_ERR_NULL, "conv_bwd: null argument");
  int rc = check_conv_plan(plan);
  if (rc) return rc;
  const bool bf16 = plan->dtype == DISTDL_BF16;
  const uintptr_t esz = bf16 ? 2 : 4;
  if (workspace_bytes < distdl_conv_bwd_workspace(plan) || (uintptr_t)workspace_dev % 16)
    return set_error(DISTDL_ERR_INVALID_ARG, "conv_bwd: workspace too small or misaligned (%zu < %zu)", workspace_bytes,
                     distdl_conv_bwd_workspace(plan));
  for (int w = 0; w < plan->n_workers; ++w) {
    if (!x_bufs_dev[w] || !dy_dev[w] || !dx_bufs_dev[w]) return set_error(DISTDL_ERR_NULL, "conv_bwd: worker %d has a null array", w);
    if ((uintptr_t)x_bufs_dev[w] % esz || (uintptr_t)dy_dev[w] % esz || (uintptr_t)dx_bufs_dev[w] % esz)
      return set_error(DISTDL_ERR_INVALID_ARG, "conv_bwd: misaligned array");
  }
  if ((rc = plan_prepare_device(plan))) return rc;
  if ((rc = plan->tab_x.upload(x_bufs_dev, plan->n_workers, st))) return rc;
  if ((rc = plan->tab_dy.upload(dy_dev, plan->n_workers, st))) return rc;
  if ((rc = plan->tab_dx.upload((const void* const*)dx_bufs_dev, plan->n_workers, st))) return rc;
  ConvDev c = conv_params(plan);
  bool aligned = true;  // dy is loaded, dx^ stored in 16-byte pieces
  for (int w = 0; w < plan->n_workers; ++w) aligned &= (uintptr_t)dy_dev[w] % 16 == 0 && (uintptr_t)dx_bufs_dev[w] % 16 == 0;
  bool vec16 = aligned && plan->n_ci % 4 == 0 && plan->n_co % 4 == 0;
  for (int w = 0; w < plan->n_workers; ++w) vec16 &= (uintptr_t)x_bufs_dev[w] % 16 == 0;
  WeightJob job;
  auto reduce_dw = [&](int nparts) {
    const int nw = c.taps * c.ci * c.co + c.co;
    ProfScope prof("conv_reduce_dw", st);
    auto reduce = [&](auto e, auto elem) {
      typedef decltype(elem) T;
      constexpr int E = decltype(e)::value;
      dim3 grid((unsigned)((nw + E - 1) / E));
      if (job.kind != 0 && (int64_t)grid.x + job.blocks < kMaxBlocks256) {
        job.at = (int32_t)grid.x;
        grid.x += (unsigned)job.blocks;
        hipLaunchKernelGGL((conv_reduce_dw_kernel<E, T, true>), grid, dim3(256), 0, st, (const float*)workspace_dev, nparts,
                           (T*)dw_dev, (T*)dbias_dev, c, job);
        job.kind = 0;
      } else {
        hipLaunchKernelGGL((conv_reduce_dw_kernel<E, T, false>), grid, dim3(256), 0, st, (const float*)workspace_dev, nparts,
                           (T*)dw_dev, (T*)dbias_dev, c, NoJob{});
      }
    };
    auto by_type = [&](auto e) { bf16 ? reduce(e, uint16_t{}) : reduce(e, float{}); };
    nw <= 8192 ? by_type(std::integral_constant<int, 16>{}) : by_type(std::integral_constant<int, 64>{});
  };
  if (halo && choose_fused(plan, true, vec16, aligned, true) && conv_fused_ready(plan, true, st) &&
      !bwd_overlaps(plan, x_bufs_dev, w_dev, dy_dev, dx_bufs_dev, dw_dev, dbias_dev, workspace_dev, workspace_bytes)) {
    int partials = 0;
    if ((rc = conv_bwd_fused(plan, w_dev, dw_dev, dbias_dev, (float*)workspace_dev, vec16, st, &partials))) return rc;
    if (partials > 0) reduce_dw(partials);
    DISTDL_HIP_TRY(hipGetLastError());
    return DISTDL_OK;
  }
  const Wgrad wgrad = choose_wgrad(plan, vec16);
  int64_t total = plan->n_b * plan->max_buf_cells * c.ci;
  const Corr kernel = choose_data(plan, aligned);
  if ((rc = weight_job(plan, kernel, true, w_dev, aligned, st, job))) return rc;
  // [dConv]* with respect to x, into the whole padded buffers
  auto data_gradient = [&]() -> int {
    int rc = DISTDL_OK;
    if (kernel == Corr::k16) {
      if ((rc = conv_bwd_data16(plan, (const float*)w_dev, aligned, st))) return rc;
    } else if (kernel == Corr::kSplit) {
      if ((rc = conv_bwd_data_split(plan, (const float*)w_dev, st))) return rc;
    } else if (kernel == Corr::kMfma) {
      if ((rc = conv_bwd_data_mfma(plan, w_dev, st))) return rc;
    } else if (kernel == Corr::kAny) {
      if ((rc = conv_bwd_data_any(plan, w_dev, aligned, st))) return rc;
    } else {
      if ((rc = prepare_weights(plan, w_dev, st))) return rc;
      ProfScope prof("conv_bwd_data_direct", st);
      const dim3 dgrid((unsigned)((total + 255) / 256), plan->n_workers);
      if (bf16)
        hipLaunchKernelGGL(conv_bwd_data_direct_kernel<uint16_t>, dgrid, dim3(256), 0, st, plan->d_workers,
                           plan->tab_dy.dev, plan->d_wt, plan->tab_dx.dev, c);
      else
        hipLaunchKernelGGL(conv_bwd_data_direct_kernel<float>, dgrid, dim3(256), 0, st, plan->d_workers,
                           plan->tab_dy.dev, plan->d_wt, plan->tab_dx.dev, c);
    }
    return rc;
  };
  // Where R's launch can lay out its weights it comes after that; elsewhere before, so that H* does not follow the kernel that
  // wrote what it reads (32 -> 32 channels, 5^3, stride 2, 256^3, bf16: H* 119 -> 105 us, the pass 0.8 % less).
  // (also where dw or db lies on the weights or on dy, which the data gradient reads, and where the weight gradient is the better one
  // to follow the data gradient)
  auto on = [](const void* a, size_t na, const void* b, size_t nb) {
    return a && (uintptr_t)a < (uintptr_t)b + nb && (uintptr_t)b < (uintptr_t)a + na;
  };
  const size_t wb = w_bytes(plan), bb = (size_t)c.co * esz;
  bool in_place = on(dw_dev, wb, w_dev, wb) || on(dbias_dev, bb, w_dev, wb);
  for (int w = 0; w < plan->n_workers; ++w)
    in_place |= on(dw_dev, wb, dy_dev[w], y_bytes(plan, w)) || on(dbias_dev, bb, dy_dev[w], y_bytes(plan, w));
  const bool data_last = job.kind != 0 && !in_place && !write_back_hides(plan, kernel, wgrad);
  if (!data_last) {
    if ((rc = launch_weight_job(job, st))) return rc;
    job.kind = 0;
    if ((rc = data_gradient())) return rc;
  }
  // [dConv]* with respect to w and b, then R over the workers
  const int nchunks = wgrad_partials(plan, wgrad, vec16);
  int nw = c.taps * c.ci * c.co + c.co;
  if (wgrad == Wgrad::k16) {
    if ((rc = conv_wgrad16(plan, (float*)workspace_dev, vec16, st))) return rc;
  } else if (wgrad == Wgrad::kSplit) {
    if ((rc = conv_wgrad_split(plan, (float*)workspace_dev, st))) return rc;
  } else if (wgrad == Wgrad::kAny) {
    if ((rc = conv_wgrad_any(plan, (float*)workspace_dev, st))) return rc;
  } else if (wgrad == Wgrad::kMfma) {
    if ((rc = conv_wgrad_mfma(plan, (float*)workspace_dev, st))) return rc;
  } else {
    ProfScope prof("conv_bwd_weight_direct", st);
    const dim3 wgrid((unsigned)((nw + 255) / 256), nchunks, plan->n_workers);
    if (bf16)
      hipLaunchKernelGGL(conv_bwd_weight_direct_kernel<uint16_t>, wgrid, dim3(256), 0, st, plan->d_workers,
                         plan->tab_x.dev, plan->tab_dy.dev, (float*)workspace_dev, c, nchunks);
    else
      hipLaunchKernelGGL(conv_bwd_weight_direct_kernel<float>, wgrid, dim3(256), 0, st, plan->d_workers,
                         plan->tab_x.dev, plan->tab_dy.dev, (float*)workspace_dev, c, nchunks);
  }
  reduce_dw(nchunks * plan->n_workers);
  if ((rc = launch_weight_job(job, st))) return rc;
  if (data_last && (rc = data_gradient())) return rc;
  DISTDL_HIP_TRY(hipGetLastError());
  // dx <- H* dx
  return halo ? run_halo(plan, true, plan->tab_dx, dx_bufs_dev, st) : DISTDL_OK;
}

}  // namespace distdl
