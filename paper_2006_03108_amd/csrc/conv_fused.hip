// Small convolution layers (Sec. 4, Forward / Adjoint Convolution Algorithms): the forward pass with its halo exchange in one
// launch, the adjoint with H* in one, or two where dw is summed over many workgroups.
//
// What bounds such a layer is not its arithmetic but its launches: H, Conv, the two contractions of [dConv]*, the reduction of dw
// and H* take 3 to 15 us each, most of that spent starting up and waiting for a chain of loads.  Two facts let them run
// side by side.  H writes halo and padding cells only and reads owned ones, so a convolution that fetches what lies in a
// halo from its owner does not depend on H.  And H* [dConv]* puts into an owned cell the sum over every output, of whichever
// worker, that the cell enters, so one thread block can make that sum from the dy of all of them, and write zeros
// into the halos.  So:
//   fused_fwd_kernel   workgroups that make y, reading neighbours' owned cells in place of halos, beside those that do H's boxes
//   fused_bwd_kernel   workgroups that make dw (all of it, or a chunk of positions' part), beside those that make dx
//
// 16 x 16 tiles, 4 k an instruction: a wave's lane holds one position (one row of x^) and 4 consecutive k, fetched from memory
// straight into registers; there is no staging to wait for but that of the weights, which are taken in the caller's order and
// kept in LDS by output channel.  fp32 tensors are multiplied and summed in fp64: twice the matrix time, which is a small part
// here (a pass takes 4 to 8 % longer than with fp32 matrix instructions in chains of 16 products).  y, dx, and dw and db where one
// workgroup sums over all positions, are rounded once, 2.5e-8, where the split products of the general kernels leave 4e-8 to 1e-7,
// and 16 x 16 tiles of fp32 2e-7; dw and db of chunks are rounded for each chunk, and those parts are added in fp32, as the general
// kernels' are.  A sum goes over taps and channels in their order, whichever worker a cell lies with: the order is fixed, but
// in dx it is not that of the workers.  bf16 tensors are widened and multiplied in fp32.
//
// What bounds it is the number of instructions that one wave issues one after the other, at 4 clocks each: of 8900 clocks of a
// workgroup for 1 -> 1 channels, 3 taps, 64 cells on four workers, the loads take a third.  So geometry and taps come from tables
// that the host makes once per plan, the cell that a position's tap meets is worked out once for all its channels, and indexes
// are divided by one multiplication (with geometry and divisions in the kernel that workgroup took 13200 clocks, in the adjoint
// 18100).  us, launches of a forward pass and an adjoint apart / together: this layer 11.7 / 6.8 and 18.0 / 8.6; 8 -> 52 channels,
// 2^3, 4 x 12 x 13 x 13 on 3 x 2 x 2 workers 24 / 12 and 41 / 23; 56 -> 8, 3 x 3, 3 x 58 x 67 on 1 x 2 29 / 15 and 34 / 25.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

#include "buffer.h"
#include "common.h"
#include "conv_fused.h"
#include "halo_box.h"
#include "profile.h"
#include "weight_job.h"

namespace distdl {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));


// Tables of a plan and direction, made once on the host and copied to the device with its first pass.
// A correlation over one worker and class of a stride: dimension by dimension
struct FusedDim {
  int32_t in0, step;               // input coordinate that the first tap meets at position q: in0 + q * step
  int32_t nq, out_ext, out0, ostep;  // positions; extent of the tensor written, where position q is written: out0 + q * ostep
  float rq;                        // 1 / nq
  int32_t lo, hi, vlo, vlen;       // input coordinates that are the worker's own: lo ... hi - 1; that exist: vlo ... vlo + vlen - 1
  int32_t own_lo, own_len;         // written cells that are owned (the others become zero)
};
struct FusedRec {
  FusedDim d[3];
  int32_t ntaps, total;  // taps, positions
  int32_t pad_[3];
};
constexpr int kRecInts = (int)(sizeof(FusedRec) / 4);
// the cells of the worker in direction (a, b, c), by the coordinates of the worker at hand
struct FusedNear {
  int64_t shift;  // elements
  int32_t to, sn, s0, s1;
  int32_t pad_[2];
};
struct Neighbour {
  uint64_t base;
  int32_t sn, s0, s1, pad_;
};

struct FusedArgs {
  int32_t n_b, ci, co, taps, kc, nc;
  int32_t k[3], s[3], dil[3];
  int32_t ncls, ntn, groups, tpw, wk;  // classes, column tiles, workgroups of each, 16-position tiles a wave, waves that share a tile's k
  int32_t cb, nch, pitch;              // channels of a chunk of weights, chunks, floats from one channel's row to the next
  int32_t most_taps;                   // of a class
  int32_t at_red, at_cells, at_taps, at_map, at_nb, at_rec, at_flag;  // LDS
  int32_t blocks;
  const FusedRec* recs;      // [worker][class]
  const FusedNear* nears;    // [worker][27]
  const int4* tap_steps;     // [class][most_taps]: what a tap adds to the input coordinates
  const int32_t* tap_index;  // [class][taps]: a tap's index in the class, or -1
  const void *w, *bias;
  const BlockRef* hblocks;  // forward: H's boxes
  const HaloTaskDev* htasks;
  int32_t wide;
  int32_t dw_mt, dw_nt, dw_chunks, dw_blocks;  // tiles of 64 rows and 16 columns, chunks a worker (0: all workers in one)
  float* partial;
  void *dw, *db;
  int64_t slot;
};

template <class T>
__device__ __forceinline__ T at_address(uint64_t address) {
  return *(const DISTDL_GLOBAL T*)address;
}
template <bool BF16>
__device__ __forceinline__ float load1(uint64_t base, int i) {
  if constexpr (BF16) return __uint_as_float((uint32_t)at_address<uint16_t>(base + (int64_t)i * 2) << 16);
  else return at_address<float>(base + (int64_t)i * 4);
}
template <bool BF16>
__device__ __forceinline__ f32x4 load4(uint64_t base, int i) {
  if constexpr (BF16) {
    const u32x2 t = at_address<u32x2>(base + (int64_t)i * 2);
    return f32x4{__uint_as_float(t[0] << 16), __uint_as_float(t[0] & 0xffff0000u), __uint_as_float(t[1] << 16), __uint_as_float(t[1] & 0xffff0000u)};
  } else {
    return at_address<f32x4>(base + (int64_t)i * 4);
  }
}
// element i of a buffer; zero if !ok
template <bool BF16>
__device__ __forceinline__ float load1(__amdgpu_buffer_rsrc_t rs, int i, bool ok) {
  const uint32_t off = ok ? (uint32_t)i * (BF16 ? 2 : 4) : kOob;
  if constexpr (BF16) return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, 0) << 16);
  else return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
}
template <bool BF16>
__device__ __forceinline__ f32x4 load4(__amdgpu_buffer_rsrc_t rs, int i, bool ok) {
  const uint32_t off = ok ? (uint32_t)i * (BF16 ? 2 : 4) : kOob;
  if constexpr (BF16) {
    const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
    return f32x4{__uint_as_float(t[0] << 16), __uint_as_float(t[0] & 0xffff0000u), __uint_as_float(t[1] << 16), __uint_as_float(t[1] & 0xffff0000u)};
  } else {
    const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
    return f32x4{__uint_as_float(t[0]), __uint_as_float(t[1]), __uint_as_float(t[2]), __uint_as_float(t[3])};
  }
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float rcp(int v) { return __builtin_amdgcn_rcpf((float)v); }
// n / d for n < 2^20 (and no further), through the reciprocal: (n + 1/2) / d is at least 1 / 2d off any integer, and the product is off by less than
// 2^-22 of itself
__device__ __forceinline__ int div_below20(int n, float rcp_d) { return (int)fmaf((float)n, rcp_d, 0.5f * rcp_d); }

// The sums of 16 x 16 products, 4 k at a time.  Register e of lane (kk, i): row kk + 4 e (fp64) or 4 kk + e, column i.
template <bool BF16>
struct Acc {
  typedef std::conditional_t<BF16, f32x4, f64x4> V;
  V v[2];  // (two, so that one does not wait for the other)
  __device__ __forceinline__ void clear() { v[0] = v[1] = V{0, 0, 0, 0}; }
  __device__ __forceinline__ void add(int which, float a, float b) {
    if constexpr (BF16) v[which] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, v[which], 0, 0, 0);
    else v[which] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, v[which], 0, 0, 0);
  }
  __device__ __forceinline__ V sum() const { return v[0] + v[1]; }
  // row of register e, for the lanes of quarter kk
  static __device__ __forceinline__ int row(int kk, int e) { return BF16 ? 4 * kk + e : kk + 4 * e; }
};
// What a tap that meets no cell reads: zeros, as many as a cell has channels.
constexpr int kZeros = 2048;
__device__ __attribute__((aligned(16))) float fused_zeros[kZeros];

template <bool BF16, int MODE, bool VEC, int NT>
__device__ __forceinline__ void fused_corr(void* const* in_bufs, void* const* out_bufs, const FusedArgs& a, int b, char* smem) {
  typedef std::conditional_t<BF16, uint16_t, float> T;
  const int group = b % a.groups;
  int r = b / a.groups;
  const int ntile = r % a.ntn;
  r /= a.ntn;
  const int cls = r % a.ncls, worker = r / a.ncls;
  const int tid = threadIdx.x, lane = tid & 63, i = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int per = 4 / a.wk, kg = wave % a.wk, pg = wave / a.wk;  // tiles of the workgroup at a time; this wave's share of k, its tile
  float* const wl = (float*)smem;
  typedef typename Acc<BF16>::V Sum;
  Sum* const red = (Sum*)(smem + a.at_red);
  uint64_t* const cells = (uint64_t*)(smem + a.at_cells) + (size_t)pg * (a.most_taps + 16) * 16;  // [tap][position]
  int4* const steps_of = (int4*)(smem + a.at_taps);
  int* const map = (int*)(smem + a.at_map);
  Neighbour* const nbs = (Neighbour*)(smem + a.at_nb);
  FusedRec* const rec = (FusedRec*)(smem + a.at_rec);  // (in scalar registers it would not fit them)
  int* const flag = (int*)(smem + a.at_flag);
  const uint64_t nothing = (uint64_t)fused_zeros;
  const bool strided = MODE == 1 && a.ncls > 1;

  // Weights of channels c0 ... + cb: [channel written][tap * cb + channel read], zero up to whole steps (channels beyond the last
  // stay as they are: their sums go nowhere).  Eight of them a thread are on their way at a time, those of the first chunk
  // while the tables are fetched.
  const int ch0 = ntile * 16 * NT, real = min(16 * NT, a.nc - ch0);
  const __amdgpu_buffer_rsrc_t rw = rsrc_of(a.w, (uint32_t)(a.co * a.ci * a.taps) * (uint32_t)sizeof(T));
  const float rt = rcp(a.taps);
  constexpr int WU = 8;
  float wv[WU];
  auto run_of = [&](int cb) { return MODE == 0 ? cb * a.taps : real * a.taps; };
  auto all_of = [&](int cb) { return MODE == 0 ? real * cb * a.taps : cb * real * a.taps; };
  auto stage_one = [&](int c0, int run, float rrun, int all, int idx) {
    const int q = div_below20(idx, rrun), e = idx - q * run;
    const int from = MODE == 0 ? ((ch0 + q) * a.ci + c0) * a.taps + e : ((c0 + q) * a.ci + ch0) * a.taps + e;
    return load1<BF16>(rw, from, idx < all);
  };
  auto stage_load = [&](int c0, int cb) {
    const int run = run_of(cb), all = all_of(cb);
    const float rrun = rcp(run);
#pragma unroll
    for (int u = 0; u < WU; ++u) {
      if (uniform(tid) + 256 * u >= all) break;  // (the first lane's)
      wv[u] = stage_one(c0, run, rrun, all, tid + 256 * u);
    }
  };
  stage_load(0, min(a.cb, a.kc));

  if (tid < 27) {
    const FusedNear near = a.nears[worker * 27 + tid];
    nbs[tid] = Neighbour{(uint64_t)in_bufs[near.to] + near.shift * (int)sizeof(T), near.sn, near.s0, near.s1, 0};
  } else if (tid >= 64 && tid < 64 + kRecInts) {
    ((int*)rec)[tid - 64] = ((const int*)(a.recs + worker * a.ncls + cls))[tid - 64];
  } else if (tid == 255) {
    *flag = 0;
  }
  for (int t = tid; t < a.most_taps; t += 256) steps_of[t] = a.tap_steps[cls * a.most_taps + t];
  if (strided)
    for (int t = tid; t < a.taps; t += 256) map[t] = a.tap_index[cls * a.taps + t];
  __syncthreads();
  const int ntaps = uniform(rec->ntaps), total = uniform(rec->total);
  if (group * a.tpw * per * 16 >= total) return;

  float seen = 0.f;
  auto stage_rest = [&](int c0, int cb) {
    const int run = run_of(cb), all = all_of(cb), K = ntaps * cb;
    const float rrun = rcp(run);
    for (int at = tid; uniform(at) < all; at += 256 * WU) {
#pragma unroll
      for (int u = 0; u < WU; ++u) {
        const int idx = at + 256 * u;
        if (uniform(idx) >= all) break;
        const int q = div_below20(idx, rrun), e = idx - q * run, c = div_below20(e, rt), t = e - c * a.taps;
        const int m = strided ? map[min(t, a.taps - 1)] : t;
        if (idx < all && m >= 0) {
          wl[(MODE == 0 ? q : c) * a.pitch + m * cb + (MODE == 0 ? c : q)] = wv[u];
          if constexpr (MODE == 1) seen = note_not_finite(wv[u], seen);
        }
        if (uniform(idx) + 256 * WU < all) wv[u] = stage_one(c0, run, rrun, all, idx + 256 * WU);
      }
    }
    const int tail = -K & 15;
    if (tail > 0) {
      const float rtail = rcp(tail);
      for (int e = tid; e < real * tail; e += 256) {
        const int row = div_below20(e, rtail);
        wl[row * a.pitch + K + e - row * tail] = 0.f;
      }
    }
    if constexpr (MODE == 1) {
      if (any_not_finite(seen)) *flag = 1;
    }
  };

  for (int it = 0; it < a.tpw; ++it) {
    const int tile = (group * a.tpw + it) * per + pg;
    const int pos = tile * 16 + i;
    const bool live = pos < total;
    bool owned;
    int to;  // the cell written
    {
      const FusedDim g0 = rec->d[0], g1 = rec->d[1], g2 = rec->d[2];
      const int q = min(pos, total - 1);  // (a lane beyond the last does the last's work and keeps it to itself)
      const int q012 = div_below20(q, g2.rq), q01 = div_below20(q012, g1.rq), n = div_below20(q01, g0.rq);
      const int q2 = q - q012 * g2.nq, q1 = q012 - q01 * g1.nq, q0 = q01 - n * g0.nq;
      const int w0 = g0.out0 + q0 * g0.ostep, w1 = g1.out0 + q1 * g1.ostep, w2 = g2.out0 + q2 * g2.ostep;
      auto in = [](int v, int lo, int len) { return (uint32_t)(v - lo) < (uint32_t)len; };
      owned = MODE == 0 || (in(w0, g0.own_lo, g0.own_len) && in(w1, g1.own_lo, g1.own_len) && in(w2, g2.own_lo, g2.own_len));
      to = ((n * g0.out_ext + w0) * g1.out_ext + w1) * g2.out_ext + w2;
      // The cells that the position's taps meet, wherever they lie; the waves of a tile and a lane's four quarters share the taps
      const int p0 = g0.in0 + q0 * g0.step, p1 = g1.in0 + q1 * g1.step, p2 = g2.in0 + q2 * g2.step;
      if (it > 0) __syncthreads();
      // (the last step may go beyond the taps)
      const int entries = a.nch > 1 ? ntaps + 16 : ntaps + div_below20((-(ntaps * a.cb) & 15) + a.cb - 1, rcp(a.cb));
#pragma unroll 2
      for (int t = kg * 4 + kq; t < entries; t += 4 * a.wk) {
        const int4 d = steps_of[min(t, a.most_taps - 1)];
        const int c0 = p0 + d.x, c1 = p1 + d.y, c2 = p2 + d.z;
        const bool ok = t < ntaps && owned && in(c0, g0.vlo, g0.vlen) && in(c1, g1.vlo, g1.vlen) && in(c2, g2.vlo, g2.vlen);
        const int f0 = (c0 >= g0.lo) + (c0 >= g0.hi), f1 = (c1 >= g1.lo) + (c1 >= g1.hi), f2 = (c2 >= g2.lo) + (c2 >= g2.hi);
        const Neighbour nb = nbs[ok ? (f0 * 3 + f1) * 3 + f2 : 13];
        cells[t * 16 + i] = ok ? nb.base + (int64_t)(n * nb.sn + c0 * nb.s0 + c1 * nb.s1 + c2 * a.kc) * (int)sizeof(T) : nothing;
      }
    }
    Acc<BF16> acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t].clear();
    for (int chunk = 0; chunk < a.nch; ++chunk) {
      const int c0 = chunk * a.cb, cb = min(a.cb, a.kc - c0);
      if (a.nch > 1 || it == 0) {
        if (chunk > 0) {
          stage_load(c0, cb);
          __syncthreads();  // (the chunk before has been read)
        }
        stage_rest(c0, cb);
      }
      __syncthreads();
      if (tile * 16 >= total) continue;
      const int steps = (ntaps * cb + 15) / 16;
      const float rcb = rcp((VEC ? cb / 4 : cb));
      auto load = [&](int st) -> f32x4 {
        const int qd = st * 4 + kq;
        if constexpr (VEC) {
          const int t = div_below20(qd, rcb);
          return load4<BF16>(cells[t * 16 + i], c0 + (qd - t * (cb / 4)) * 4);
        } else {
          f32x4 v;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int k = qd * 4 + j, t = div_below20(k, rcb);
            v[j] = load1<BF16>(cells[t * 16 + i], c0 + k - t * cb);
          }
          return v;
        }
      };
      constexpr int U = 4;
      f32x4 x[U], next[U];
      // (the row of lane i: such that a lane's four sums are those of neighbouring channels)
      const float* const wrow = wl + (BF16 ? i : 4 * (i & 3) + (i >> 2)) * a.pitch + kq * 4;
      auto fetch = [&](f32x4 (&v)[U], int st) {
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (st + u * a.wk < steps) v[u] = load(st + u * a.wk);  // (uniform)
      };
      fetch(x, kg);
      for (int st = kg; st < steps; st += U * a.wk) {
        fetch(next, st + U * a.wk);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (st + u * a.wk < steps) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
              const f32x4 w4 = *(const f32x4*)(wrow + t * 16 * a.pitch + (st + u * a.wk) * 16);
#pragma unroll
              for (int j = 0; j < 4; ++j) acc[t].add(j & 1, w4[j], x[u][j]);
            }
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = next[u];
      }
    }
    Sum tot[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) tot[t] = acc[t].sum();
    if (a.wk > 1) {  // the waves that share a tile, in order
#pragma unroll
      for (int t = 0; t < NT; ++t) red[(wave * NT + t) * 64 + lane] = tot[t];
      __syncthreads();
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (t % a.wk != kg) continue;
        tot[t] = red[(pg * a.wk * NT + t) * 64 + lane];
        for (int u = 1; u < a.wk; ++u) tot[t] += red[((pg * a.wk + u) * NT + t) * 64 + lane];
      }
    }
    if (tile * 16 >= total || !live) continue;
    bool terms = false;
    if constexpr (MODE == 1) terms = *flag != 0;
    T* const out = (T*)out_bufs[worker] + (size_t)to * a.nc;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (a.wk > 1 && t % a.wk != kg) continue;
      const int ch = ch0 + 16 * t + 4 * kq;
      if (ch >= a.nc) continue;
      if constexpr (MODE == 0) {
        if (a.bias) {
#pragma unroll
          for (int e = 0; e < 4; ++e) tot[t][e] += ld((const T*)a.bias, min(ch + e, a.nc - 1));
        }
      }
      f32x4 v = __builtin_convertvector(tot[t], f32x4);
      if constexpr (MODE == 1) {
        if (!owned) v = f32x4{0.f, 0.f, 0.f, 0.f};
        if (terms && owned) {
          // A weight that is not finite met the zeros of taps whose output does not exist: term by term, without those
#pragma unroll 1
          for (int e = 0; e < 4 && ch + e < a.nc; ++e) {
            const float was = e == 0 ? v[0] : e == 1 ? v[1] : e == 2 ? v[2] : v[3];
            if (!not_finite(was)) continue;
            float s = 0.f;
#pragma unroll 1
            for (int m = 0; m < a.taps; ++m) {
              const int at = strided ? map[m] : m;
              if (at < 0) continue;
              const uint64_t cell = cells[at * 16 + i];
              if (cell == nothing) continue;
#pragma unroll 1
              for (int c = 0; c < a.kc; ++c) s = fmaf(load1<BF16>(cell, c), ld((const T*)a.w, ((size_t)c * a.ci + ch + e) * a.taps + m), s);
            }
            if (e == 0) v[0] = s;
            else if (e == 1) v[1] = s;
            else if (e == 2) v[2] = s;
            else v[3] = s;
          }
        }
      }
      if constexpr (VEC && !BF16) {
        *(f32x4*)(out + ch) = v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (ch + e < a.nc) st(out, ch + e, v[e]);
      }
    }
  }
}

// dw and db: 64 rows (tap, input channel) by 16 NT columns over a chunk of a worker's positions, or over all positions of all
// workers.  A lane reads 4 rows of one position (VEC: neighbours) and one column of NT; the waves share the positions.
template <bool BF16, bool VEC, int NT>
__device__ __forceinline__ void fused_wgrad(const WorkerDev* __restrict__ workers, int n_workers, void* const* x_bufs, void* const* dy_bufs,
                                            const FusedArgs& a, int b, char* smem) {
  typedef std::conditional_t<BF16, uint16_t, float> T;
  const int mt = b % a.dw_mt;
  int r = b / a.dw_mt;
  const int ntile = r % a.dw_nt;
  r /= a.dw_nt;
  const bool whole = a.dw_chunks == 0;
  const int chunk = whole ? 0 : r % a.dw_chunks, one = whole ? 0 : r / a.dw_chunks;
  const int tid = threadIdx.x, lane = tid & 63, i = lane & 15, kk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rows = a.taps * a.ci;
  // this lane's rows: tap and channel
  constexpr int NR = VEC ? 1 : 4;
  int t0[NR], t1[NR], t2[NR], cc[NR];
  const float rci = rcp(a.ci), rk2 = rcp(a.k[2]), rk1 = rcp(a.k[1]);
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    const int k = min(mt * 64 + (VEC ? 4 * i : 16 * j + i), rows - 1), tap = div_below20(k, rci), t01 = div_below20(tap, rk2);
    cc[j] = VEC ? (k - tap * a.ci) / 4 * 4 : k - tap * a.ci;
    t2[j] = tap - t01 * a.k[2];
    t0[j] = div_below20(t01, rk1);
    t1[j] = t01 - t0[j] * a.k[1];
  }
  int col[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) col[t] = (ntile * NT + t) * 16 + i;
  typedef typename Acc<BF16>::V Sum;
  typedef std::conditional_t<BF16, float, double> One;
  Acc<BF16> acc[4][NT];
  One bsum[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    bsum[t] = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j][t].clear();
  }
  // (all workers: they, or of one and two their halves and quarters, are dealt to the waves)
  const int cuts = whole ? max(4 / n_workers, 1) : 1;
  for (int share = whole ? wave : 0; share < (whole ? n_workers * cuts : 1); share += 4) {
    const int worker = whole ? share / cuts : one;
    const WorkerDev wd = workers[worker];
    const int s1 = wd.buf[2] * a.ci, s0 = wd.buf[1] * s1, sn = wd.buf[0] * s0;
    const int npos = a.n_b * wd.out[0] * wd.out[1] * wd.out[2];
    const __amdgpu_buffer_rsrc_t rx = rsrc_of(x_bufs[worker], (uint32_t)(a.n_b * sn) * (uint32_t)sizeof(T)),
                                 ry = rsrc_of(dy_bufs[worker], (uint32_t)(npos * a.co) * (uint32_t)sizeof(T));
    const float rq2 = rcp(wd.out[2]), rq1 = rcp(wd.out[1]), rq0 = rcp(wd.out[0]);
    // fours of positions, dealt to the chunks, and a chunk's to the waves
    const int fours = (npos + 3) / 4, parts = whole ? cuts : a.dw_chunks * 4, part = whole ? share % cuts : chunk * 4 + wave;
    const int begin = (int)((int64_t)fours * part / parts) * 4, end = min((int)((int64_t)fours * (part + 1) / parts) * 4, npos);
    int base[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j)
      base[j] = (wd.origin[0] + t0[j] * a.dil[0]) * s0 + (wd.origin[1] + t1[j] * a.dil[1]) * s1 + (wd.origin[2] + t2[j] * a.dil[2]) * a.ci + cc[j];
    // Batches of four times four positions, the next one on its way while one is multiplied
    constexpr int U = 4;
    f32x4 x[U], next_x[U];
    float y[U][NT], next_y[U][NT];
    int cell = 0;  // of position at + lane, of the 64 that the batch is one of
    auto fetch = [&](f32x4 (&x)[U], float (&y)[U][NT], int at, int s) {
      if (s == 0) {
        const int q = min(at + lane, npos - 1);
        const int q012 = div_below20(q, rq2), q01 = div_below20(q012, rq1), n = div_below20(q01, rq0);
        const int o2 = q - q012 * wd.out[2], o1 = q012 - q01 * wd.out[1], o0 = q01 - n * wd.out[0];
        cell = n * sn + o0 * a.s[0] * s0 + o1 * a.s[1] * s1 + o2 * a.s[2] * a.ci;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = at + (s + u) * 4 + kk;
        const bool ok = p < end;
        const int off = __shfl(cell, (s + u) * 4 + kk);
        if constexpr (VEC) {
          x[u] = load4<BF16>(rx, off + base[0], ok);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) x[u][j] = load1<BF16>(rx, off + base[j], ok);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) y[u][t] = load1<BF16>(ry, p * a.co + col[t], ok && col[t] < a.co);
      }
    };
    if (begin < end) fetch(x, y, begin, 0);
    for (int at = begin, s = 0; at + s * 4 < end;) {
      const int here = s + U < 16 ? at : at + 64, there = s + U < 16 ? s + U : 0;
      if (here + there * 4 < end) fetch(next_x, next_y, here, there);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          bsum[t] += y[u][t];
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[j][t].add(u & 1, x[u][j], y[u][t]);
        }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        x[u] = next_x[u];
#pragma unroll
        for (int t = 0; t < NT; ++t) y[u][t] = next_y[u][t];
      }
      at = here, s = there;
    }
  }
  constexpr int NB = 16 * NT;
  One* const red = (One*)smem;  // [wave][row][column]
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const Sum tot = acc[j][t].sum();
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int ri = Acc<BF16>::row(kk, e), row = VEC ? 4 * ri + j : 16 * j + ri;
        red[(wave * 64 + row) * NB + 16 * t + i] = tot[e];
      }
    }
  One* const bred = red + 4 * 64 * NB;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    One s = bsum[t];
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if (lane < 16) bred[wave * NB + 16 * t + lane] = s;
  }
  __syncthreads();
  float* const slot = whole ? nullptr : a.partial + ((size_t)one * a.dw_chunks + chunk) * a.slot;
#pragma unroll
  for (int u = 0; u < 64 * NB / 256; ++u) {
    const int e = tid + 256 * u, row = e / NB, c = e % NB, k = mt * 64 + row, ch = ntile * NB + c;
    const float s = (float)((red[e] + red[64 * NB + e]) + red[2 * 64 * NB + e] + red[3 * 64 * NB + e]);
    if (k >= rows || ch >= a.co) continue;
    if (whole) {
      const int tap = div_below20(k, rci);
      st((T*)a.dw, ((size_t)ch * a.ci + (k - tap * a.ci)) * a.taps + tap, s);
    } else {
      slot[(size_t)k * a.co + ch] = s;
    }
  }
  if (mt == 0 && tid < NB && ntile * NB + tid < a.co) {
    const float s = (float)(bred[tid] + bred[NB + tid] + bred[2 * NB + tid] + bred[3 * NB + tid]);
    if (!whole) slot[(size_t)rows * a.co + ntile * NB + tid] = s;
    else if (a.db) st((T*)a.db, ntile * NB + tid, s);
  }
}

template <bool BF16, bool VEC, int NT>
__global__ __launch_bounds__(256, NT == 4 ? 2 : 3) void fused_fwd_kernel(void* const* x_bufs, void* const* y_bufs, FusedArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int b = (int)blockIdx.x;
  if (b < a.blocks) return fused_corr<BF16, 0, VEC, NT>(x_bufs, y_bufs, a, b, smem);
  if constexpr (BF16) {
    if (a.wide) halo_fwd_box<BF16x8>(a.hblocks, a.htasks, x_bufs, b - a.blocks);
    else halo_fwd_box<BF16x1>(a.hblocks, a.htasks, x_bufs, b - a.blocks);
  } else {
    if (a.wide) halo_fwd_box<F32x4>(a.hblocks, a.htasks, x_bufs, b - a.blocks);
    else halo_fwd_box<F32x1>(a.hblocks, a.htasks, x_bufs, b - a.blocks);
  }
}

template <bool BF16, bool VEC, int NT>
__global__ __launch_bounds__(256, NT == 4 ? 2 : 3) void fused_bwd_kernel(const WorkerDev* __restrict__ workers, int n_workers, void* const* x_bufs,
                                                           void* const* dy_bufs, void* const* dx_bufs, FusedArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int b = (int)blockIdx.x;
  if (b < a.dw_blocks) fused_wgrad<BF16, VEC, 1>(workers, n_workers, x_bufs, dy_bufs, a, b, smem);
  else fused_corr<BF16, 1, VEC, NT>(dy_bufs, dx_bufs, a, b - a.dw_blocks, smem);
}

// ---- host side ------------------------------------------------------------------

struct Shape {
  FusedArgs a = {};
  int NT = 1, lds = 0;
  bool fits = false;
};
// What a plan keeps of one direction: the shapes of its launch without and with 16-byte accesses, and, once it is to run, its tables
struct FusedPlan {
  Shape shape[2];
  std::vector<FusedRec> recs;
  std::vector<FusedNear> nears;
  std::vector<int4> tap_steps;
  std::vector<int32_t> tap_index;
  FusedRec* d_recs = nullptr;
  FusedNear* d_nears = nullptr;
  int4* d_tap_steps = nullptr;
  int32_t* d_tap_index = nullptr;
  char* own = nullptr;  // their block, where it is not the plan's
  ~FusedPlan() {
    if (own) (void)hipFree(own);
  }
  void add_to(HostTables& t) { t.add(recs, &d_recs), t.add(nears, &d_nears), t.add(tap_steps, &d_tap_steps), t.add(tap_index, &d_tap_index); }
};

FusedDim dim_of(const distdl_plan* p, int mode, int w, int d, int par, int nt, int tf) {
  const WorkerDev& wd = p->workers[w];
  FusedDim g{};
  if (mode == 0) {
    g.step = p->stride[d], g.in0 = wd.origin[d];
    g.nq = g.out_ext = wd.out[d], g.out0 = 0, g.ostep = 1;
    g.lo = wd.bulk_off[d], g.hi = wd.bulk_off[d] + wd.in_size[d], g.vlo = wd.dom_lo[d], g.vlen = wd.dom_hi[d] - wd.dom_lo[d];
    g.own_lo = 0, g.own_len = wd.out[d];
  } else {
    const int s = p->stride[d], op = wd.origin[d] + par, first = op % s;
    g.step = 1, g.in0 = nt > 0 ? -(op / s) - (tf * p->dilation[d] - par) / s : 0;
    g.nq = first < wd.buf[d] ? (wd.buf[d] - 1 - first) / s + 1 : 0;
    g.out_ext = wd.buf[d], g.out0 = first, g.ostep = s;
    const int start = d < 3 - p->D ? 0 : (int)p->dims[d][p->coords(w, d)].out_start;
    g.lo = 0, g.hi = wd.out[d], g.vlo = -start, g.vlen = (int32_t)p->out_shape[d];
    g.own_lo = wd.bulk_off[d], g.own_len = wd.in_size[d];
  }
  g.rq = 1.0f / (float)std::max(g.nq, 1);
  return g;
}

// The classes of a direction: a stride's in the adjoint, one forward
struct Classes {
  int n = 1, taps = 1, most_taps = 1;
  std::vector<int> nt, tf, ts;  // [class][dimension]: taps, the first and the step between them
  int par(const distdl_plan* p, int mode, int cls, int d) const {
    if (mode == 0) return 0;
    return d == 0 ? cls / (p->stride[1] * p->stride[2]) : d == 1 ? cls / p->stride[2] % p->stride[1] : cls % p->stride[2];
  }
};
Classes classes_of(const distdl_plan* p, int mode) {
  Classes c;
  for (int d = 0; d < 3; ++d) {
    c.taps *= p->ksize[d];
    if (mode == 1) c.n *= p->stride[d];
  }
  c.nt.resize(c.n * 3), c.tf.resize(c.n * 3), c.ts.resize(c.n * 3);
  for (int cls = 0; cls < c.n; ++cls) {
    int all = 1;
    for (int d = 0; d < 3; ++d) {
      int &n = c.nt[cls * 3 + d] = p->ksize[d], &f = c.tf[cls * 3 + d] = 0, &s = c.ts[cls * 3 + d] = 1;
      if (mode == 1) class_taps(p->ksize[d], p->stride[d], p->dilation[d], c.par(p, mode, cls, d), n, f, s);
      all *= n;
    }
    c.most_taps = std::max(c.most_taps, all);
  }
  return c;
}

// The most positions of a worker and class: extents of a dimension depend on a worker's place in it and on the class's parity there
int64_t most_positions(const distdl_plan* p, int mode) {
  int64_t most = p->n_b;
  for (int d = 0; d < 3; ++d) {
    int32_t n = 0;
    const int step = d == 0 ? p->P[1] * p->P[2] : d == 1 ? p->P[2] : 1;  // from worker to worker along d
    for (int at = 0; at < p->P[d]; ++at)
      for (int par = 0; par < (mode == 0 ? 1 : p->stride[d]); ++par) n = std::max(n, dim_of(p, mode, at * step, d, par, 0, 0).nq);
    most *= n;
  }
  return std::max<int64_t>(most, 1);
}

// The tables of a direction
void make_tables(const distdl_plan* p, int mode, FusedPlan& f) {
  const Classes c = classes_of(p, mode);
  const int ncls = c.n, taps = c.taps, most_taps = c.most_taps;
  f.recs.resize((size_t)p->n_workers * ncls);
  f.tap_steps.assign((size_t)ncls * most_taps, int4{0, 0, 0, 0});
  f.tap_index.assign((size_t)ncls * taps, -1);
  for (int cls = 0; cls < ncls; ++cls) {
    const int *n = &c.nt[cls * 3], *first = &c.tf[cls * 3], *s = &c.ts[cls * 3];
    int at = 0;
    for (int i0 = 0; i0 < n[0]; ++i0)
      for (int i1 = 0; i1 < n[1]; ++i1)
        for (int i2 = 0; i2 < n[2]; ++i2, ++at) {
          const int i[3] = {i0, i1, i2};
          int step[3], tap = 0;
          for (int d = 0; d < 3; ++d) {
            step[d] = mode == 0 ? i[d] * p->dilation[d] : -i[d] * (s[d] * p->dilation[d] / p->stride[d]);
            tap = tap * p->ksize[d] + first[d] + i[d] * s[d];
          }
          f.tap_steps[(size_t)cls * most_taps + at] = int4{step[0], step[1], step[2], 0};
          f.tap_index[(size_t)cls * taps + tap] = at;
        }
    for (int w = 0; w < p->n_workers; ++w) {
      FusedRec& r = f.recs[(size_t)w * ncls + cls];
      r = FusedRec{};
      int64_t total = p->n_b;
      for (int d = 0; d < 3; ++d) {
        r.d[d] = dim_of(p, mode, w, d, c.par(p, mode, cls, d), n[0] * n[1] * n[2], first[d]);
        total *= r.d[d].nq;
      }
      r.total = (int32_t)total;
      r.ntaps = n[0] * n[1] * n[2];
    }
  }
  f.nears.resize((size_t)p->n_workers * 27);
  const int64_t kc = mode == 0 ? p->n_ci : p->n_co;
  for (int w = 0; w < p->n_workers; ++w)
    for (int e = 0; e < 27; ++e) {
      const int f3[3] = {e / 9 - 1, e / 3 % 3 - 1, e % 3 - 1};
      bool there = true;
      int to = 0;
      for (int d = 0; d < 3; ++d) {
        const int at = p->coords(w, d) + f3[d];
        there &= at >= 0 && at < p->P[d];
        to = to * p->P[d] + at;
      }
      if (!there) to = w;
      const WorkerDev &own = p->workers[w], &nb = p->workers[to];
      const int32_t* ext = mode == 0 ? nb.buf : nb.out;
      FusedNear& near = f.nears[(size_t)w * 27 + e];
      near = FusedNear{};
      near.to = to;
      near.s1 = (int32_t)(ext[2] * kc), near.s0 = ext[1] * near.s1, near.sn = ext[0] * near.s0;
      const int64_t stride[3] = {near.s0, near.s1, kc};
      for (int d = 0; there && d < 3; ++d) {
        if (f3[d] == 0) continue;
        const int below = mode == 0 ? nb.bulk_off[d] + nb.in_size[d] - own.bulk_off[d] : nb.out[d],
                  above = mode == 0 ? nb.bulk_off[d] - own.bulk_off[d] - own.in_size[d] : -own.out[d];
        near.shift += (f3[d] < 0 ? below : above) * stride[d];
      }
    }
}

Shape shape_of(const distdl_plan* p, int mode, bool vec, int taps, int64_t positions) {
  Shape sh;
  FusedArgs& a = sh.a;
  a.n_b = (int32_t)p->n_b, a.ci = (int32_t)p->n_ci, a.co = (int32_t)p->n_co;
  a.kc = mode == 0 ? a.ci : a.co, a.nc = mode == 0 ? a.co : a.ci;
  a.taps = a.ncls = 1;
  for (int d = 0; d < 3; ++d) {
    a.k[d] = p->ksize[d], a.s[d] = p->stride[d], a.dil[d] = p->dilation[d];
    a.taps *= a.k[d];
    if (mode == 1) a.ncls *= a.s[d];
  }
  const int64_t tiles = (positions + 15) / 16, each = tiles * p->n_workers * a.ncls;  // of 16 columns each
  // Columns of a wave's tile: as many as the channels fill, while there are two waves for every SIMD
  const int nts = (a.nc + 15) / 16;
  sh.NT = nts >= 3 && each * ((nts + 3) / 4) >= 2048 ? 4 : nts >= 2 && each * ((nts + 1) / 2) >= 1024 ? 2 : 1;
  a.ntn = (nts + sh.NT - 1) / sh.NT;
  // waves that share a tile's k where there are few tiles
  const int64_t K = (int64_t)taps * a.kc, waves = each * a.ntn;
  a.wk = waves < 1024 && K > 32 ? 4 : waves < 2048 && K > 16 ? 2 : 1;
  // chunk of channels: at most 96 KB of weights
  const int most = 1536 / sh.NT;
  int cb = a.kc;
  if ((int64_t)taps * cb > most) cb = std::max(vec ? 4 : 1, most / taps / (vec ? 4 : 1) * (vec ? 4 : 1));
  a.cb = cb;
  a.nch = (a.kc + cb - 1) / cb;
  const int quads = (taps * cb + 15) / 16 * 4;
  a.pitch = 4 * (quads | 1);
  const int per = 4 / a.wk;
  // Tiles a wave makes one after the other: the set-up and the weights serve all of them, where a launch is many rounds of workgroups
  a.tpw = a.nch > 1 ? 1 : (int)std::max<int64_t>(1, std::min<int64_t>(8, waves / (8 * 1024)));
  a.groups = (int32_t)((tiles + (int64_t)per * a.tpw - 1) / ((int64_t)per * a.tpw));
  const int64_t blocks = (int64_t)p->n_workers * a.ncls * a.ntn * a.groups;
  a.blocks = (int32_t)std::min<int64_t>(blocks, INT32_MAX);
  a.most_taps = taps;
  int at = 16 * sh.NT * a.pitch * 4;
  a.at_red = at, at += a.wk > 1 ? 4 * sh.NT * 64 * 32 : 0;
  a.at_cells = at, at += (taps + 16) * 16 * 8 * per;
  a.at_taps = at, at += taps * 16;
  a.at_map = at, at += a.ncls > 1 ? (a.taps * 4 + 15) / 16 * 16 : 0;
  a.at_nb = at, at += (27 * (int)sizeof(Neighbour) + 15) / 16 * 16;
  a.at_rec = at, at += (int)sizeof(FusedRec) / 16 * 16 + 16;
  a.at_flag = at, at += 16;
  sh.lds = at;
  // (indexes of weights are divided through a float: fewer than 2^20)
  sh.fits = at <= 128 * 1024 && a.kc <= kZeros && 16 * sh.NT * (int64_t)cb * a.taps < (1 << 20) && blocks < (1 << 22);
  return sh;
}

FusedPlan* plan_of(const distdl_plan* p, int mode) {
  std::shared_ptr<void>& kept = p->fused_plan[mode];
  if (!kept) {
    auto f = std::make_shared<FusedPlan>();
    if (const int64_t positions = most_positions(p, mode); positions < (1 << 20))  // (they are divided through a float)
      for (int vec = 0; vec < 2; ++vec) f->shape[vec] = shape_of(p, mode, vec != 0, classes_of(p, mode).most_taps, positions);
    kept = f;
  }
  return (FusedPlan*)kept.get();
}

}  // namespace

// (what an estimate asks for is in the shapes: tables are made for the directions that run)
void conv_fused_make_tables(const distdl_plan* p, bool backward) {
  if (FusedPlan* const f = plan_of(p, backward); f->recs.empty()) make_tables(p, backward, *f);
}
int conv_fused_records(const distdl_plan* p, bool backward) { return p->n_workers * (backward ? p->stride[0] * p->stride[1] * p->stride[2] : 1); }

namespace {

// the launch of a direction, its tables on the device
int shape_on_device(const distdl_plan* p, int mode, bool vec, Shape& sh) {
  FusedPlan* const f = plan_of(p, mode);
  if (!f->d_recs) {
    HostTables t;
    conv_fused_make_tables(p, mode != 0);
    f->add_to(t);
    if (int rc = t.to_device(&f->own)) return rc;
  }
  sh = f->shape[vec];
  sh.a.recs = f->d_recs, sh.a.nears = f->d_nears, sh.a.tap_steps = f->d_tap_steps, sh.a.tap_index = f->d_tap_index;
  return DISTDL_OK;
}

template <bool BF16, bool VEC, int NT>
int launch_fwd(distdl_plan* p, const Shape& sh, int halo_blocks, hipStream_t st) {
  if (sh.lds > 64 * 1024)
    if (int rc = allow_large_lds<fused_fwd_kernel<BF16, VEC, NT>>()) return rc;
  hipLaunchKernelGGL((fused_fwd_kernel<BF16, VEC, NT>), dim3((unsigned)(sh.a.blocks + halo_blocks)), dim3(256), sh.lds, st, p->tab_x.dev, p->tab_y.dev,
                     sh.a);
  return DISTDL_OK;
}
template <bool BF16, bool VEC, int NT>
int launch_bwd(distdl_plan* p, const Shape& sh, hipStream_t st) {
  const int lds = std::max(sh.lds, (4 * 64 + 4) * 16 * (BF16 ? 4 : 8));
  if (lds > 64 * 1024)
    if (int rc = allow_large_lds<fused_bwd_kernel<BF16, VEC, NT>>()) return rc;
  hipLaunchKernelGGL((fused_bwd_kernel<BF16, VEC, NT>), dim3((unsigned)(sh.a.blocks + sh.a.dw_blocks)), dim3(256), lds, st, p->d_workers, p->n_workers,
                     p->tab_x.dev, p->tab_dy.dev, p->tab_dx.dev, sh.a);
  return DISTDL_OK;
}
#define DISTDL_FUSED(F_, BF_, V_, NT_, ...)                                      \
  ((BF_) ? ((V_) ? DISTDL_FUSED_NT(F_, true, true, NT_, __VA_ARGS__)             \
                 : DISTDL_FUSED_NT(F_, true, false, NT_, __VA_ARGS__))           \
         : ((V_) ? DISTDL_FUSED_NT(F_, false, true, NT_, __VA_ARGS__)            \
                 : DISTDL_FUSED_NT(F_, false, false, NT_, __VA_ARGS__)))
#define DISTDL_FUSED_NT(F_, BF_, V_, NT_, ...) \
  ((NT_) == 1 ? F_<BF_, V_, 1>(__VA_ARGS__) : (NT_) == 2 ? F_<BF_, V_, 2>(__VA_ARGS__) : F_<BF_, V_, 4>(__VA_ARGS__))

bool small_tensors(const distdl_plan* p) {
  return !p->explicit_halo && (double)p->n_b * p->max_buf_cells * std::max(p->n_ci, p->n_co) < 5e8 && p->max_buf_cells * p->n_b < (1 << 20) && p->max_out_cells * p->n_b < (1 << 20) && p->n_workers <= 1024 &&
         (double)p->n_ci * p->n_co * p->ksize[0] * p->ksize[1] * p->ksize[2] < (1 << 22) &&
         (double)std::max(p->n_ci, p->n_co) * p->ksize[0] * p->ksize[1] * p->ksize[2] < (1 << 20) && p->stride[0] * p->stride[1] * p->stride[2] <= 64 &&
         (int64_t)p->ksize[0] * p->ksize[1] * p->ksize[2] <= 1024;
}

// positions of a wave where one workgroup sums over all of them
double wave_positions(const distdl_plan* p) {
  const int cuts = std::max(4 / p->n_workers, 1);
  return (double)((p->n_workers * cuts + 3) / 4) * p->n_b * p->max_out_cells / cuts;
}

// the weight gradient's part of an adjoint's launch
void add_wgrad(const distdl_plan* p, Shape& sh) {
  FusedArgs& a = sh.a;
  const int64_t pos = p->n_b * p->max_out_cells, rows = (int64_t)a.taps * a.ci;
  a.slot = rows * a.co + a.co;
  a.dw_mt = (int32_t)((rows + 63) / 64);
  a.dw_nt = (a.co + 15) / 16;
  const int64_t tiles = (int64_t)a.dw_mt * a.dw_nt;
  int64_t chunks = 0;
  if (wave_positions(p) > 256) {
    const int64_t room = (int64_t)(distdl_conv_bwd_workspace(p) / (a.slot * 4 * p->n_workers));
    chunks = std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(room, (pos + 127) / 128), (768 + tiles * p->n_workers - 1) / (tiles * p->n_workers)));
  }
  a.dw_chunks = (int32_t)chunks;
  a.dw_blocks = (int32_t)(tiles * (chunks == 0 ? 1 : chunks * p->n_workers));
}

}  // namespace

// Estimated time of a direction's call, launches and all (us); infinite where it is not taken.  A workgroup's time is that of its
// set-up, its weights, the positions and taps of its tiles and their steps of 16 k; compute units with several of them take longer
// for each; y leaves at 5 TB/s, or value by value at a million in 1.1 us.  Two terms joined by a fourth power: what the host takes to launch, more
// for each worker's arrays, and what the device does.  Fitted to 600 layers of 1 to 64 channels, one to three dimensions, up to
// 600 000 positions and 0.4 GFLOP; four fifths are within 12 % (forward) and 14 %.
double conv_fused_us(const distdl_plan* p, bool backward, bool vec) {
  if (!small_tensors(p)) return INFINITY;
  Shape& sh = plan_of(p, backward)->shape[vec];
  if (!sh.fits) return INFINITY;
  if (backward && sh.a.dw_blocks == 0) add_wgrad(p, sh);
  const FusedArgs& a = sh.a;
  const bool bf16 = p->dtype == DISTDL_BF16;
  const double stage = (double)std::min(16 * sh.NT, a.nc) * a.taps * a.kc / 2048, entries = (a.most_taps + 2) / (4.0 * a.wk),
               steps = std::max(1.0, std::ceil((double)a.most_taps * a.kc / 16)) / a.wk, load = a.blocks / 256.0;
  const double written = 1e-6 * p->n_workers * p->n_b * (backward ? p->max_buf_cells : p->max_out_cells) * a.nc * dtype_size(p->dtype);  // of y or dx, MB
  const int resident = std::min(160 * 1024 / sh.lds, sh.NT == 4 ? 2 : 3);
  if (!backward) {
    const double t = 1.2 + stage + a.tpw * (0.58 + 0.17 * entries + steps * ((vec ? 0.0 : 0.21) + 0.32 * sh.NT));
    const double store = vec && !bf16 ? 0.2 * written : 1.1 * written / (bf16 ? 2 : 4);
    return joined(6.2 + 0.2 * p->n_workers, 3.2 + t * std::max(1.0, load / resident) * (1 + 0.22 * std::min(load, 3.0)) + store);
  }
  const double t = 1.1 + 0.77 * stage + a.tpw * (0.69 + 0.077 * entries + steps * ((vec ? 0.08 : 0.2) + 0.11 * sh.NT));
  const bool whole = a.dw_chunks == 0;
  const double batches = std::max(1.0, whole ? wave_positions(p) / 16 : (double)p->n_b * p->max_out_cells / (a.dw_chunks * 64.0));
  const double tw = 1.6 + batches * (vec ? 0.91 : 1.5) * (bf16 ? 1.2 : 1.0), loadw = a.dw_blocks / 256.0;
  const double longest = std::max(t, tw), all = (t * load + tw * loadw) / resident * (1 + 0.27 * std::min(load + loadw, 3.0));
  const double reduce = whole ? 0 : 2.0 + 13e-6 * a.slot * p->n_workers * a.dw_chunks;
  return joined(7.8 + 0.25 * p->n_workers, 3.5 + std::max(longest, all) + 0.58 * std::min(longest, all) + reduce + 0.092 * written);
}

// (a call that is recorded cannot bring the tables to the device: where it is the plan's first, the general kernels take it)
bool conv_fused_ready(const distdl_plan* p, bool backward, hipStream_t st) {
  if (plan_of(p, backward)->d_recs) return true;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(st, &cs) == hipSuccess && cs == hipStreamCaptureStatusNone;
}

void conv_fused_add_tables(const distdl_plan* p, HostTables& t) {
  for (const auto& kept : p->fused_plan)
    if (FusedPlan* const f = (FusedPlan*)kept.get(); f && !f->d_recs && !f->recs.empty()) f->add_to(t);
}

int conv_fwd_fused(distdl_plan* p, const void* w, const void* bias, bool vec, bool wide, hipStream_t st) {
  Shape sh;
  if (int rc = shape_on_device(p, 0, vec, sh)) return rc;
  const TaskTable& tt = wide ? p->fwd16 : p->fwd1;
  sh.a.w = w, sh.a.bias = bias;
  sh.a.hblocks = tt.d_blocks, sh.a.htasks = tt.d_tasks, sh.a.wide = wide;
  ProfScope prof("conv_fwd_fused", st);
  return DISTDL_FUSED(launch_fwd, p->dtype == DISTDL_BF16, vec, sh.NT, p, sh, (int)tt.blocks.size(), st);
}

int conv_bwd_fused(distdl_plan* p, const void* w, void* dw, void* db, float* partial, bool vec, hipStream_t st, int* partials) {
  Shape sh;
  if (int rc = shape_on_device(p, 1, vec, sh)) return rc;
  if (sh.a.dw_blocks == 0) add_wgrad(p, sh);
  sh.a.w = w, sh.a.dw = dw, sh.a.db = db, sh.a.partial = partial;
  *partials = sh.a.dw_chunks * p->n_workers;
  ProfScope prof("conv_bwd_fused", st);
  return DISTDL_FUSED(launch_bwd, p->dtype == DISTDL_BF16, vec, sh.NT, p, sh, st);
}
#undef DISTDL_FUSED
#undef DISTDL_FUSED_NT

}  // namespace distdl
