// Local convolution of fp32 tensors on the bf16 matrix cores (split_bf16.h): forward and data gradient of the layers
// whose contraction channels are a multiple of 4, as an implicit GEMM over staged patches (Sec. 4, "Conv" and "[dConv]*").
//
//   out[q][n] = sum_taps sum_k W[tap][k][n] * in[base + q * step + tapoff][k]
//
// as in conv_mfma.hip: forward in = x^, out = y; data gradient once per stride-parity class of dx^, in = dy
// (the classes that take the same kernel variant are one launch).
// A workgroup of four waves owns a tr x tc window of 128 MT output positions and walks output planes.  A stage is
//   (kernel plane t0, tap group, 16 channels):
// the input cells that the group's taps read are loaded, split into three bf16 planes and written to LDS, as are the
// group's weights (split once per call, by a launch before: weight_job.h); then every tap multiplies 6 MT MFMAs per wave.
// The taps of a kernel plane are grouped by the residue of their input offset modulo the step: a group's cells are then
// the cells of one residue only, the cell of (position, tap) is position + constant, and a stage of a stride-2 layer is a
// quarter of the patch with a quarter of the taps.  Three planes of a whole 5 x 5 stride-2 stage would be 200 KB; the
// groups (9, 6, 6 and 4 taps) take 64 KB at most, so two workgroups share a compute unit and one's loads, splits and
// barriers run under the other's MFMAs.  Groups of more than 10 taps are cut by kernel rows.
// Layers of few channels (FEW).  A tile has 32 columns and an MFMA 16 k; an output tensor of 3 channels and a chunk of 4 or 8
// input channels leave most of both empty.  Two ways to fill them, each taken where the estimate of the launch's time says so:
//   fold: `fold` neighbouring cells along dimension 2 are one position with fold * channels columns (contiguous in memory); the
//     taps of the cells, those of one offset together, are the position's taps: k + fold - 1 of them instead of fold * k.
//     Data gradient: fold is a multiple of the stride, and the classes of dimension 2 are one launch.
//   a last chunk of at most 8 channels: the 16 k of an MFMA are those of two taps.
// us before and after: data gradient of 32 -> 3 channels, 7 x 7, stride 2, 8 x 224 x 224 (fold 4) 71 and 37; 4 -> 8, 3^3, stride 2,
// 6 x 28 x 30 x 45 (fold 2) 36.7 and 23.7; 20 -> 2, 1^3, stride 2, 7 x 58 x 62 x 60 52 and 37; forward of 28 -> 8, 3 x 3,
// 2 x 675 x 1013 (fold 3) 145 and 123.  (Whole layers of 24 and 40 channels gain nothing from the second way alone: three M-tiles
// do not fit its registers.)
// Error (2-norm, against 64 bits; fp32 MFMAs in brackets): 4000 products a sum 3.9e-7 (1.13e-6), 21952 with three M-tiles
// 1.9e-6 and two 8.5e-7 (2.4e-6), 72 products 5.7e-8 (1.5e-7).
// Bound: MFMAs (at the clock that the power limit leaves them with real data, about 2/3 of the peak) and LDS: with
// MT = 2 a tap reads 9 KB per 12 MFMAs and wave, 3/4 of what LDS can deliver in that time.
#include <algorithm>
#include <mutex>
#include <memory>

#include "buffer.h"
#include "common.h"
#include "conv_mfma.h"
#include "conv_split.h"
#include "profile.h"
#include "split_bf16.h"
#include "weight_job.h"

namespace distdl {

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kGroupTaps = 10, kFewTaps = 8, kMaxFewColumns = 0xffff;

template <class ArgsPtr>
__host__ __device__ inline PerWorker derive_of(const WorkerDev& wd, ArgsPtr a) {
  CorrArgs c;
  c.mode = a->c.mode;
#pragma unroll
  for (int d = 0; d < 3; ++d) c.s[d] = a->c.s[d], c.par[d] = a->c.par[d];
  PerWorker g = derive(wd, c);
  if (a->fold > 1) {  // position q2: cells out_base + fold * q2 ...; data gradient: all classes of dimension 2
    const int s = c.s[2], r = wd.origin[2] % s;
    g.out_base[2] = c.mode == 0 || r == 0 ? 0 : r - s;
    g.in_base[2] = c.mode == 0 ? wd.origin[2] : (g.out_base[2] - wd.origin[2]) / s;  // (a whole number)
    g.nq[2] = (g.out_ext[2] - g.out_base[2] + a->fold - 1) / a->fold;
    g.os[2] = a->fold;
  }
  return g;
}

// Bytes of half an LDS plane of the patch (8 channels of PA * 128 cells), of a plane.  The halves lie a multiple of 256
// bytes apart, as the two half-waves of an operand read want it (64 or 128 more bytes between them: 1.4 times the LDS
// cycles), and a half-wave writes one half of 32 cells.
constexpr uint32_t half_bytes(int PA) { return PA * 2048; }
constexpr uint32_t plane_bytes(int PA) { return 2 * half_bytes(PA); }
constexpr int split_lds_bytes(int PA, int taps) { return 3 * plane_bytes(PA) + taps * 3072 + 16; }

// MT: 32-position M-tiles per wave; PA: pairs of 16-byte pieces (8 channels of a cell) per thread and stage; PB: weight
// pieces per thread and stage; FEW: for layers of few channels,
// fold > 1 or a last chunk of one octet
template <int MT, int PA, int PB, bool FEW, class ArgsPtr>
__device__ __forceinline__ void corr_split(ArgsPtr a, const WorkerDev* __restrict__ workers, void* const* in_bufs,
                                           void* const* out_bufs, const u32x4* wt, const float* w, const float* bias_in) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const auto& c = a->c;
  constexpr uint32_t HB = half_bytes(PA), PS = plane_bytes(PA);
  // consecutive tiles (which share input rows) stay on one XCD, i.e. behind one L2
  const uint32_t nblk = gridDim.x, r = (blockIdx.x & 7u) * (nblk >> 3) + (blockIdx.x >> 3);
  const uint32_t worker = r / c.tiles_max;
  uint32_t tile = r - worker * c.tiles_max;
  if (worker >= (uint32_t)c.n_workers) return;
  const WorkerDev wd = workers[worker];
  const PerWorker g = derive_of(wd, a);
  const int nt2tiles = (g.nq[2] + c.tc - 1) / c.tc, nt1tiles = (g.nq[1] + c.tr - 1) / c.tr;
  const int nq0 = g.nq[0], ptotal = c.n_b * nq0, ngroups = (ptotal + c.g0 - 1) / c.g0;
  if ((int64_t)tile >= (int64_t)ngroups * nt1tiles * nt2tiles * c.ntn) return;
  const int q2_0 = (tile % nt2tiles) * c.tc; tile /= nt2tiles;
  const int q1_0 = (tile % nt1tiles) * c.tr; tile /= nt1tiles;
  const int ntile = tile % c.ntn; tile /= c.ntn;  // `tile` is now this workgroup's place among the plane groups

  const int si2 = c.kc, si1 = g.in_ext[2] * si2, si0 = g.in_ext[1] * si1;
  const uint32_t sin = (uint32_t)g.in_ext[0] * si0;
  const uint32_t so2 = FEW ? a->nch : c.nc, so1 = g.out_ext[2] * so2, so0 = g.out_ext[1] * so1, son = g.out_ext[0] * so0;
  const __amdgpu_buffer_rsrc_t rin = rsrc_of(in_bufs[worker], (uint32_t)c.n_b * sin * 4u);
  const __amdgpu_buffer_rsrc_t rout = rsrc_of(out_bufs[worker], (uint32_t)c.n_b * son * 4u);
  const int ncc = (c.kc + 15) / 16, nt0 = c.nt[0], ntaps = a->gbegin[a->ngroups];
  const int nfull = FEW ? a->nfull : ncc;
  const bool one_octet = FEW && nfull == 0;  // a cell is one piece
  const uint32_t wplane = (uint32_t)ntaps * 192u, wt0 = (uint32_t)nfull * wplane + (FEW ? a->npairs : 0) * 192u;  // weight pieces of one (t0, chunk), of t0
  const __amdgpu_buffer_rsrc_t rw = rsrc_of(wt + a->woff + (size_t)ntile * nt0 * wt0, (uint32_t)nt0 * wt0 * 16u);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, m = lane & 31;

  const FastDiv div_cw{c.div_cw.mul, c.div_cw.sh1, c.div_cw.sh2, c.div_cw.d}, div_tc{c.div_tc.mul, c.div_tc.sh1, c.div_tc.sh2, c.div_tc.d};
  // this thread's patch pieces: 8 channels (half ph) of cell `cell`; row and column in input steps
  int prow[PA], pcol[PA];
  uint32_t plin[PA];
#pragma unroll
  for (int i = 0; i < PA; ++i) {
    const int ph = one_octet ? 0 : (tid >> 5) & 1, cell = one_octet ? tid + 256 * i : (tid & 31) + 32 * (tid >> 6) + 128 * i;
    const int rr = (int)fd_div((uint32_t)cell, div_cw), cc = cell - rr * c.Cw;
    prow[i] = cell < c.R * c.Cw ? g.in_base[1] + q1_0 * c.is[1] + rr * c.is[1] : -0x40000000;  // never in range
    pcol[i] = g.in_base[2] + q2_0 * c.is[2] + cc * c.is[2];
    plin[i] = (uint32_t)(prow[i] * si1 + pcol[i] * si2 + ph * 8) * 4u;
  }
  // piece i lies 128 * i (256 * i) cells further
  const uint32_t pl0 = one_octet ? tid * 16u : (uint32_t)((tid >> 5) & 1) * HB + (uint32_t)((tid & 31) + 32 * (tid >> 6)) * 16u;
  const uint32_t pl1 = one_octet ? 4096u : 2048u;
  char* const wlds = smem + 3 * PS;

  // lane m of M-tile (wave, mt) multiplies window position (wave * MT + mt) * 32 + m.  The tile is accumulated transposed
  // (the weights are the first MFMA operand): register v of lane (h, m) is channel ntile * 32 + 8 (v / 4) + 4 h + v % 4 of
  // that position, so that a register quad is four consecutive channels and goes out as one 16-byte store.
  uint32_t abase[MT], soff[MT], live[FEW ? MT : 1];  // live: the columns of the position that are cells of the buffer, first and end
  const int ch0 = ntile * 32 + 4 * h;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int pidx = (wave * MT + mt) * 32 + m;
    int wr = (int)fd_div((uint32_t)pidx, div_tc), wc = pidx - wr * c.tc;
    const int q1 = q1_0 + wr, q2 = q2_0 + wc;
    soff[mt] = kOob;
    if (wr < c.tr && q1 < g.nq[1] && q2 < g.nq[2])
      soff[mt] = ((g.out_base[1] + g.os[1] * q1) * so1 + (g.out_base[2] + g.os[2] * q2) * so2 + ch0) * 4u;
    if constexpr (FEW) {
      const int cell = g.out_base[2] + g.os[2] * q2, lo = max(0, -cell * a->nch), hi = min(c.nc, (g.out_ext[2] - cell) * a->nch);
      live[mt] = soff[mt] == kOob ? 0u : (uint32_t)lo | (uint32_t)hi << 16;  // (at most kMaxFewColumns)
    }
    if (wr >= c.tr) wr = 0, wc = 0;  // idle position: multiplies something in range, never stored
    abase[mt] = (FEW ? 0u : (uint32_t)h * HB) + (uint32_t)(wr * c.Cw + wc) * 16u;
  }
  const uint32_t wread = (uint32_t)(h * 32 + m) * 16u;

  // stage order: output planes dealt to the groups in turn, kernel planes rotated so that neighbouring groups stand on
  // the same input plane at the same moment (see conv_mfma.hip)
  const int toff0 = c.tapoff[0][0], tstep = nt0 > 1 ? c.tapoff[0][1] - c.tapoff[0][0] : 0;
  auto plane_of = [&](int q0, int t0) { return g.in_base[0] + q0 * c.is[0] + toff0 + t0 * tstep; };
  const int rot_d = (nt0 > 1 && tstep != 0 && c.is[0] % tstep == 0) ? (c.is[0] / tstep) % nt0 : 0;
  const bool dealt = rot_d != 0 && ngroups > 1;
  const int pfirst = dealt ? (int)tile : (int)tile * c.g0, pstride = dealt ? ngroups : 1;
  const int pcnt = dealt ? (ptotal - (int)tile + ngroups - 1) / ngroups : min(c.g0, ptotal - (int)tile * c.g0);
  auto skew_of = [&](int q0) {
    const int s = (rot_d * q0) % nt0;
    return s == 0 ? 0 : (s > 0 ? nt0 - s : -s);  // (-d * q0) mod nt0
  };
  struct StagePos {
    int p, n, q0, t0, cc, gr, j, sk;
  };
  auto advance = [&](StagePos& sp) {  // next valid stage after sp, or sp.p == pcnt
    if (++sp.cc < ncc) return;
    sp.cc = 0;
    if (++sp.gr < a->ngroups) return;
    sp.gr = 0;
    ++sp.j;
    while (sp.p < pcnt) {
      while (sp.j < nt0) {
        sp.t0 = sp.j + sp.sk < nt0 ? sp.j + sp.sk : sp.j + sp.sk - nt0;
        const int i0 = plane_of(sp.q0, sp.t0);
        if (i0 >= 0 && i0 < g.in_ext[0] && a->ngroups > 0) return;
        ++sp.j;
      }
      ++sp.p;
      sp.j = 0;
      sp.q0 += pstride;
      while (sp.q0 >= nq0) sp.q0 -= nq0, ++sp.n;
      sp.sk = rot_d ? skew_of(sp.q0) : 0;
    }
  };

  u32x4 ra[PA][2], rb[PB];
  const uint32_t wave_u = (uint32_t)__builtin_amdgcn_readfirstlane(wave);
  uint32_t wpieces = 0;  // weight pieces of the stage in the registers
  auto load_cells = [&](const StagePos& sp) {
    const int b1 = a->gbase[sp.gr][0], b2 = a->gbase[sp.gr][1];
    const uint32_t shift = (uint32_t)(b1 * si1 + b2 * si2) * 4u;
    const uint32_t sbase = ((uint32_t)sp.n * sin + (uint32_t)plane_of(sp.q0, sp.t0) * si0 + sp.cc * 16) * 4u;
    const int left = c.kc - sp.cc * 16 - (one_octet ? 0 : ((tid >> 5) & 1) * 8);  // channels of this thread's half
#pragma unroll
    for (int i = 0; i < PA; ++i) {
      const bool ok = (uint32_t)(prow[i] + b1) < (uint32_t)g.in_ext[1] && (uint32_t)(pcol[i] + b2) < (uint32_t)g.in_ext[2];
      const uint32_t vo = plin[i] + shift;
      ra[i][0] = __builtin_amdgcn_raw_buffer_load_b128(rin, ok && left > 0 ? vo : kOob, sbase, 0);
      ra[i][1] = __builtin_amdgcn_raw_buffer_load_b128(rin, ok && left > 4 ? vo + 16u : kOob, sbase, 0);
    }
  };
  auto load_stage = [&](const StagePos& sp) {
    load_cells(sp);
    const bool pairs = FEW && sp.cc >= nfull;
    const int tb = pairs ? a->hbegin[sp.gr] : a->gbegin[sp.gr];
    const uint32_t np = (uint32_t)((pairs ? a->hbegin[sp.gr + 1] : a->gbegin[sp.gr + 1]) - tb) * 192u;
    const uint32_t wbase = ((uint32_t)sp.t0 * wt0 + (uint32_t)sp.cc * wplane + (uint32_t)tb * 192u) * 16u;
#pragma unroll
    for (int i = 0; i < PB; ++i)  // (a wave's 64 pieces are all there or all not)
      if (i * 256 + wave_u * 64 < np) rb[i] = __builtin_amdgcn_raw_buffer_load_b128(rw, tid * 16u, wbase + i * 4096u, 0);
    wpieces = np;
  };
  auto write_stage = [&](float scale) {
#pragma unroll
    for (int i = 0; i < PA; ++i) {
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = __uint_as_float(ra[i][e >> 2][e & 3]);
      u32x4 hi, mid, lo;
      split_eight(v, scale, hi, mid, lo);
      char* const at = smem + pl0 + i * (FEW ? pl1 : 2048u);
      *(u32x4*)at = hi;
      *(u32x4*)(at + PS) = mid;
      *(u32x4*)(at + 2 * PS) = lo;
    }
#pragma unroll
    for (int i = 0; i < PB; ++i)
      if (i * 256 + wave_u * 64 < wpieces) *(u32x4*)(wlds + (tid + i * 256) * 16) = rb[i];
  };

  union Frag {
    u32x4 u;
    bf16x8 v;
  };
  // Two accumulators, or (three M-tiles: 48 more registers do not fit) one whose sign changes from pair to pair of stages,
  // and that of the cells with it: either keeps the bias of the small products out of the sums (split_bf16.h).
  constexpr bool TWO = MT < 3;
  floatx16 acc[MT], low[TWO ? MT : 1];
  auto zero_acc = [&]() {
#pragma unroll
    for (int t = 0; t < MT; ++t)
      for (int v = 0; v < 16; ++v) {
        acc[t][v] = 0.f;
        if constexpr (TWO) low[t][v] = 0.f;
      }
  };
  // One set of operand registers: a tap's six products are ordered so that every operand of the next tap is read right
  // after the last product that needs its register, two to four products before its own first use.
  Frag fw[3], fx[3][MT];
  auto read_w = [&](int p, int t) { fw[p].u = *(const u32x4*)(wlds + t * 3072 + p * 1024 + wread); };
  auto read_x = [&](int p, uint32_t cell16) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) fx[p][mt].u = *(const u32x4*)(smem + abase[mt] + cell16 + p * PS);
  };
  auto mm = [&](int pw, int px) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      floatx16& c = TWO && pw + px > 0 ? low[TWO ? mt : 0] : acc[mt];
      c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[pw].v, fx[px][mt].v, c, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  const int my_cell = lane < ntaps ? a->tapcell[lane] * 16 : 0;  // lane t keeps the patch offset of tap t
  const uint32_t half = (uint32_t)h * HB;
  // A chunk of at most 8 channels: the k of an MFMA are those of two taps, one for each half of the wave (the weights of a
  // tap that there is not are zero).
  auto compute = [&](int gr, bool pairs) {
    const int tb = a->gbegin[gr], ntap = a->gbegin[gr + 1] - tb, nt = FEW && pairs ? (ntap + 1) / 2 : ntap;
    auto cell_of = [&](int t) -> uint32_t {
      if constexpr (!FEW) return (uint32_t)__builtin_amdgcn_readlane(my_cell, tb + t);
      if (!pairs) return (uint32_t)__builtin_amdgcn_readlane(my_cell, tb + t) + half;
      const uint32_t c0 = (uint32_t)__builtin_amdgcn_readlane(my_cell, tb + 2 * t),
                     c1 = (uint32_t)__builtin_amdgcn_readlane(my_cell, tb + min(2 * t + 1, ntap - 1));
      return h ? c1 : c0;
    };
    uint32_t cell = cell_of(0);
    read_w(2, 0);
    read_x(0, cell);
    read_w(1, 0);
    read_w(0, 0);
    read_x(2, cell);
    read_x(1, cell);
    for (int t = 0; t < nt; ++t) {
      const int tn = t + 1 < nt ? t + 1 : t;  // (past the last tap: its own operands again)
      cell = cell_of(tn);
      mm(2, 0);
      read_w(2, tn);
      mm(1, 0);
      mm(0, 0);
      read_x(0, cell);
      mm(0, 2);
      read_x(2, cell);
      mm(1, 1);
      read_w(1, tn);
      mm(0, 1);
      read_w(0, tn);
      read_x(1, cell);
    }
  };

  StagePos sp{0, pfirst / nq0, pfirst % nq0, 0, ncc - 1, a->ngroups - 1, -1, 0};  // the stage whose loads are in flight
  sp.sk = rot_d ? skew_of(sp.q0) : 0;
  advance(sp);
  int on = pfirst / nq0, oq0 = pfirst % nq0;  // the output plane that is stored next
  const FastDiv div_nch{a->div_nch.mul, a->div_nch.sh1, a->div_nch.sh2, a->div_nch.d};
  auto store_plane = [&]() {
    float bias[4][4] = {};
    if (bias_in) {
      // 16 loads of some channel of the layer, all in flight (with a branch and a wait for each of them the forward pass of 8 -> 44
      // channels, 1^3, 9 x 53 x 29 x 52, took 86 us instead of 73).  Indexes and address are not kept from plane to plane: the
      // registers are few, and what the scalar ones cannot hold is moved about in the loop over the taps.
      int first = ch0;
      const float* b = bias_in;
      asm volatile("" : "+v"(first), "+s"(b));
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t col = (uint32_t)(first + 8 * q + e);  // (beyond the channels: any of them, it is not stored)
          bias[q][e] = b[FEW ? col - fd_div(col, div_nch) * (uint32_t)a->nch : min(col, (uint32_t)c.nc - 1u)];
        }
    }
    const uint32_t obase = ((uint32_t)on * son + (uint32_t)(g.out_base[0] + g.os[0] * oq0) * so0) * 4u;
    // (the plane's offset is added into the per-lane offset: with a scalar offset the compiler leaves out the wait states
    // a 16-byte store needs before its data registers are written again)
    if constexpr (FEW) {
      // The columns of a position are contiguous in memory: 16-byte stores (of any alignment) of whole quads, single ones at the
      // ends of a row.
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int n0 = ch0 + 8 * q, lo = (int)(live[mt] & 0xffffu), hi = (int)(live[mt] >> 16);
          const bool whole = n0 >= lo && n0 + 4 <= hi, some = !whole && n0 + 4 > lo && n0 < hi;
          const uint32_t off = soff[mt] + (uint32_t)(8 * q) * 4u + obase;
          u32x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = __float_as_uint(acc[mt][4 * q + e] + bias[q][e]);
          __builtin_amdgcn_raw_buffer_store_b128(o, rout, whole ? off : kOob, 0, 0);
          if (__builtin_amdgcn_ballot_w64(some)) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              __builtin_amdgcn_raw_buffer_store_b32(o[e], rout, some && n0 + e >= lo && n0 + e < hi ? off + 4u * e : kOob, 0, 0);
          }
        }
    } else if (c.nc & 3) {  // (uniform) quads need not be whole, nor aligned
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int e = 8 * (v >> 2) + (v & 3);
          const bool live = ch0 + e < c.nc;
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[mt][v] + bias[v >> 2][v & 3]), rout,
                                                (live ? soff[mt] + (uint32_t)e * 4u : kOob) + obase, 0, 0);
        }
    } else
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool live = ch0 + 8 * q < c.nc;  // a quad is whole or absent
        const uint32_t off = (live ? soff[mt] + (uint32_t)(8 * q) * 4u : kOob) + obase;
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          o[e] = __float_as_uint(acc[mt][4 * q + e] + bias[q][e]);
        }
        __builtin_amdgcn_raw_buffer_store_b128(o, rout, off, 0, 0);
      }
    oq0 += pstride;
    while (oq0 >= nq0) oq0 -= nq0, ++on;
  };
  int* const redo = (int*)(wlds + c.ck * 3072);  // set if a sum of the plane is not finite; if a weight is not
  if (tid == 0) redo[0] = redo[1] = 0;
  __syncthreads();
  if (sp.p < pcnt) load_stage(sp);
  for (int po = 0; po < pcnt; ++po) {  // output planes of this workgroup
    zero_acc();
    uint32_t turn = 1;  // stages of the plane so far, and one; bit 1: the sign of the accumulator (+ - - + + - - ...)
    while (sp.p == po) {  // the stages that feed output plane po
      const int gr = sp.gr;
      const bool pairs = FEW && sp.cc >= nfull;
      if constexpr (!TWO) {
        if (turn > 1 && (turn & 1) == 0) {
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[mt] = -acc[mt];
        }
      }
      write_stage(!TWO && (turn & 2) ? -kSplitScale : kSplitScale);
      __syncthreads();
      advance(sp);
      if (sp.p < pcnt) load_stage(sp);  // in flight while this stage multiplies
      compute(gr, pairs);
      if (sp.p != po) {
        float seen = 0.f;
        const float scale = !TWO && (turn & 2) ? -kUnsplit : kUnsplit;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          if constexpr (TWO) acc[mt] += low[mt];
#pragma unroll
          for (int v = 0; v < 16; ++v) seen = note_not_finite(acc[mt][v] *= scale, seen);
        }
        if (any_not_finite(seen)) *redo = 1;
      }
      ++turn;
      __syncthreads();
    }
    if (__builtin_amdgcn_readfirstlane(*redo)) {  // (uniform, rare) the plane once more in fp32, its weights from the caller's
      StagePos rp{po, on, oq0, 0, ncc - 1, a->ngroups - 1, -1, rot_d ? skew_of(oq0) : 0};
      zero_acc();
      __syncthreads();  // every wave has read the word
      if (tid == 0) redo[0] = redo[1] = 0;
      __syncthreads();
      for (advance(rp); rp.p == po; advance(rp)) {
        load_cells(rp);
        const int tb = a->gbegin[rp.gr], nt = a->gbegin[rp.gr + 1] - tb;
#pragma unroll
        for (int i = 0; i < PA; ++i) {
          float v[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = __uint_as_float(ra[i][e >> 2][e & 3]);
          u32x4 u, l;
          halve_eight(v, u, l);
          char* const at = smem + pl0 + i * (FEW ? pl1 : 2048u);
          *(u32x4*)at = u;
          *(u32x4*)(at + PS) = l;
        }
#pragma unroll 1
        for (int i = tid; i < nt * 64; i += 256) {  // [tap][h][nn]
          float v[8];
          split_weight_octet(a, w, rp.t0, rp.cc * 16 + ((i >> 5) & 1) * 8, tb + (i >> 6), ntile * 32 + (i & 31), v);
          u32x4 u, l;
          halve_eight(v, u, l);
          char* const at = wlds + (i >> 6) * 3072 + (i & 63) * 16;
          *(u32x4*)at = u;
          *(u32x4*)(at + 1024) = l;
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (not_finite(v[e])) redo[1] = 1;
        }
        __syncthreads();
        // A cell of dx lacks the taps whose output does not exist.  They read zeros, which do not cancel a weight that is not
        // finite: once there is one, lane by lane and without those terms.  Ditto where zeros fill up the weights: the taps that
        // a cell of a position lacks, the second octet of a chunk that has one.
        const int octets = FEW && rp.cc >= nfull ? 1 : 2;
        const bool lanes = (FEW && (a->fold > 1 || octets == 1)) || (c.mode == 1 && __builtin_amdgcn_readfirstlane(redo[1]));
#pragma unroll 1
        for (int t = 0; lanes && t < nt; ++t) {
          const uint32_t cell = (uint32_t)__builtin_amdgcn_readlane(my_cell, tb + t) - (FEW ? 0u : half);
          bool there[MT];
          int first = ch0;
          asm volatile("" : "+v"(first));
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            const int pidx = (wave * MT + mt) * 32 + m, wr = (int)fd_div((uint32_t)pidx, div_tc), wc = pidx - wr * c.tc;
            const int i1 = g.in_base[1] + (q1_0 + wr) * c.is[1] + c.tapoff[1][a->tap12[tb + t][0]],
                      i2 = g.in_base[2] + (q2_0 + wc) * c.is[2] + a->off2[a->tap12[tb + t][1]];
            there[mt] = (uint32_t)i1 < (uint32_t)g.in_ext[1] && (uint32_t)i2 < (uint32_t)g.in_ext[2];
          }
#pragma unroll 1
          for (int o = 0; o < octets; ++o) {  // of the chunk
            Eight xx[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
              const char* const xp = smem + abase[mt] + cell + o * HB;
              xx[mt] = join_halves(*(const u32x4*)xp, *(const u32x4*)(xp + PS));
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              const char* const wp = wlds + t * 3072 + (o * 32 + 8 * (v >> 2) + 4 * h + (v & 3)) * 16;
              const Eight xw = join_halves(*(const u32x4*)wp, *(const u32x4*)(wp + 1024));
              if constexpr (FEW) {
                if (tap2_of(a, a->tap12[tb + t][1], (int)fd_div((uint32_t)(first + 8 * (v >> 2) + (v & 3)), div_nch)) < 0) continue;
              }
#pragma unroll
              for (int mt = 0; mt < MT; ++mt) {
                float sum = acc[mt][v];
#pragma unroll
                for (int e = 0; e < 8; ++e) sum = fmaf(xw.v[e], xx[mt].v[e], sum);
                acc[mt][v] = there[mt] ? sum : acc[mt][v];
              }
            }
          }
        }
#pragma unroll 1
        for (int t = 0; !lanes && t < nt; ++t) {
          const uint32_t cell = (uint32_t)__builtin_amdgcn_readlane(my_cell, tb + t) + (FEW ? half : 0u);
          const char* const wp = wlds + t * 3072 + wread;
          const Eight xw = join_halves(*(const u32x4*)wp, *(const u32x4*)(wp + 1024));
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            const char* const xp = smem + abase[mt] + cell;
            acc[mt] = multiply_fp32(xw, join_halves(*(const u32x4*)xp, *(const u32x4*)(xp + PS)), acc[mt]);
          }
        }
        __syncthreads();
      }
      if (sp.p < pcnt) load_cells(sp);  // the next plane's cells again: their registers were used
    }
    store_plane();
  }
}

// One class, its arguments in the kernel's (their loads cost nothing to repeat, where those of the table stay in registers:
// 0.48 against 1.3 ms per class on the 5^3 stride-2 layer), and several, blockIdx.y, from the table: small layers, where
// it is launches that count (8 -> 64 channels, 3^3, stride 2, 3 x 5 x 6 x 7: 205 us with 16 launches, 71 with 2).
template <int MT, int PA, int PB, bool FEW>
__global__ __launch_bounds__(256, 2) void corr_split_kernel(const WorkerDev* __restrict__ workers, void* const* in_bufs,
                                                            void* const* out_bufs, SplitArgs a, const u32x4* wt,
                                                            const float* w, const float* bias) {
  corr_split<MT, PA, PB, FEW, const SplitArgs*>(&a, workers, in_bufs, out_bufs, wt, w, bias);
}
template <int MT, int PA, int PB, bool FEW>
__global__ __launch_bounds__(256, 2) void corr_split_classes_kernel(const WorkerDev* __restrict__ workers, void* const* in_bufs,
                                                                    void* const* out_bufs, const SplitArgs* tab, int first,
                                                                    const u32x4* wt, const float* w, const float* bias) {
  corr_split<MT, PA, PB, FEW, TablePtr>(args_at(tab, first + (int)blockIdx.y), workers, in_bufs, out_bufs, wt, w, bias);
}

// ---- host side ------------------------------------------------------------------

// Tap groups of a launch; false when there are more than the arguments hold.
bool group_taps(SplitArgs& a, bool octet, int group) {
  const CorrArgs& c = a.c;
  if (c.nt[1] * c.nt[2] > kMaxTaps) return false;
  int at = 0, most = 0;
  a.ngroups = 0;
  a.gbegin[0] = 0;
  int span1 = 0, span2 = 0;
  // first the groups with their tap indices, then the patch they need
  for (int r1 = 0; r1 < c.is[1]; ++r1)
    for (int r2 = 0; r2 < c.is[2]; ++r2) {
      int i1[8], n1 = 0, i2[kMaxOff2], n2 = 0;
      for (int t = 0; t < c.nt[1]; ++t)
        if (((c.tapoff[1][t] - r1) % c.is[1] + c.is[1]) % c.is[1] == 0) i1[n1++] = t;
      for (int t = 0; t < c.nt[2]; ++t)
        if (((a.off2[t] - r2) % c.is[2] + c.is[2]) % c.is[2] == 0) i2[n2++] = t;
      if (n1 == 0 || n2 == 0) continue;
      const int rows = std::max(1, group / n2), parts = (n1 + rows - 1) / rows, per = (n1 + parts - 1) / parts;
      for (int b = 0; b < n1; b += per) {
        if (a.ngroups >= kMaxGroups) return false;
        const int e = std::min(n1, b + per);
        int lo1 = INT32_MAX, hi1 = INT32_MIN, lo2 = INT32_MAX, hi2 = INT32_MIN;
        for (int i = b; i < e; ++i) lo1 = std::min(lo1, c.tapoff[1][i1[i]]), hi1 = std::max(hi1, c.tapoff[1][i1[i]]);
        for (int j = 0; j < n2; ++j) lo2 = std::min(lo2, a.off2[i2[j]]), hi2 = std::max(hi2, a.off2[i2[j]]);
        a.gbase[a.ngroups][0] = lo1;
        a.gbase[a.ngroups][1] = lo2;
        span1 = std::max(span1, (hi1 - lo1) / c.is[1]);
        span2 = std::max(span2, (hi2 - lo2) / c.is[2]);
        for (int i = b; i < e; ++i)
          for (int j = 0; j < n2; ++j) {
            a.tap12[at][0] = (uint8_t)i1[i];
            a.tap12[at][1] = (uint8_t)i2[j];
            ++at;
          }
        most = std::max(most, at - a.gbegin[a.ngroups]);
        a.hbegin[a.ngroups + 1] = a.hbegin[a.ngroups] + (at - a.gbegin[a.ngroups] + 1) / 2;
        a.gbegin[++a.ngroups] = at;
      }
    }
  a.c.tapspan[1] = span1;
  a.c.tapspan[2] = span2;
  a.c.ck = most;
  const int last = a.c.kc % 16;
  a.nfull = a.c.kc / 16 + (octet ? 0 : last > 0);
  a.npairs = octet ? a.hbegin[a.ngroups] : 0;
  return true;
}

// window tr x tc of 128 mt positions and the patch of its groups
void set_window(SplitArgs& a, int mt, int tc) {
  CorrArgs& c = a.c;
  const int cap = 128 * mt;
  c.tc = std::max(1, std::min(tc, cap));
  c.tr = std::max(1, cap / c.tc);
  c.R = c.tr + c.tapspan[1];
  c.Cw = c.tc + c.tapspan[2];
  c.div_cw = make_fastdiv((uint32_t)c.Cw);
  c.div_tc = make_fastdiv((uint32_t)c.tc);
  for (int gr = 0; gr < a.ngroups; ++gr)
    for (int t = a.gbegin[gr]; t < a.gbegin[gr + 1]; ++t)
      a.tapcell[t] = ((c.tapoff[1][a.tap12[t][0]] - a.gbase[gr][0]) / c.is[1] * c.Cw +
                                (a.off2[a.tap12[t][1]] - a.gbase[gr][1]) / c.is[2]);
}

double window_share(int cap, int tc, int nq1, int nq2) {  // fraction of the multiplied positions that are outputs
  const int tr = std::max(1, cap / tc);
  return (double)nq1 * nq2 / ((double)((nq2 + tc - 1) / tc) * ((nq1 + tr - 1) / tr) * cap);
}

bool one_octet(const SplitArgs& a) { return a.nfull == 0; }
int patch_cells(const SplitArgs& a, int tr, int tc) { return (tr + a.c.tapspan[1]) * (tc + a.c.tapspan[2]); }
int pieces_of(const SplitArgs& a, int cells) { return (cells * (one_octet(a) ? 1 : 2) + 255) / 256; }  // per thread
bool few_channels(const SplitArgs& a) { return a.fold > 1 || a.npairs > 0; }

// The window of a launch: M-tiles per wave (0: none fits).  The window that wastes the fewest multiplied positions; of
// equal ones the one with the smallest patch per position.  Of widths that give as many rows and as many windows side by side
// only the smallest is tried: the others share its positions and have larger patches (some 60 of 768 widths; a plan is searched
// in its first call, and asks for every way to fold: 4 -> 4 channels, 5 x 5, 6 x 528 x 776, 2800 us with all widths).
int choose_window(const distdl_plan* p, SplitArgs& a, double& used, int64_t& tried) {
  int nq1 = 1, nq2 = 1;
  for (const WorkerDev& wd : p->workers) {
    const PerWorker g = derive_of(wd, &a);
    nq1 = std::max(nq1, g.nq[1]);
    nq2 = std::max(nq2, g.nq[2]);
  }
  double best = -1;
  used = 0;
  int best_mt = 0, best_tc = 0;
  for (int mt : {3, 2, 1}) {
    // Three M-tiles have one accumulator for large and small products, which rounds it six times for 16 channels, where fp32
    // MFMAs do so eight times.  4 and 20 channels fill their last chunk by a quarter and would be further off than with those
    // (3 x 3, 4 channels: 1.32e-7 and 1.10e-7; 8 channels 1.34 and 1.54, 36 channels 2.99 and 3.22); two M-tiles: 4.9e-8.
    if (mt == 3 && (a.c.kc == 4 || a.c.kc == 20 || a.c.ck > 9 || few_channels(a))) continue;
    if (best * 1.001 >= (mt == 1 ? 0.75 : 1.0) / 1.05) break;  // (a patch has a cell for every position)
    const int cap = 128 * mt, widest = std::min(cap, nq2);
    for (int tc = 1, next; tc <= widest; tc = next) {
      const int tr = cap / tc, across = (nq2 + tc - 1) / tc;
      next = cap / tr + 1;  // fewer rows
      if (across > 1) next = std::min(next, (nq2 + across - 2) / (across - 1));  // fewer windows side by side
      ++tried;
      const int cells = patch_cells(a, tr, tc), pa = pieces_of(a, cells);
      if (pa > 4 || split_lds_bytes(pa <= 3 && mt == 2 ? 3 : 4, a.c.ck) > 80 * 1024) continue;
      // a tap costs a wave 6 mt MFMAs and 3 mt + 3 operand reads: fewer M-tiles pay relatively more for the weights
      const double share = window_share(cap, tc, nq1, nq2), patch = (double)cells / cap;
      const double score = share * (mt == 1 ? 0.75 : 1.0) / (1.0 + 0.05 * patch);
      if (score > best * 1.001) best = score, best_mt = mt, best_tc = tc, used = share;
    }
  }
  if (best_mt) set_window(a, best_mt, best_tc);
  return best_mt;
}

// fold = 1: the launch as `c` has it; else one that makes `fold` neighbouring cells along dimension 2 in one position, a
// multiple of the stride where `c` is a class of the data gradient (then of any parity along that dimension)
SplitArgs split_args(const distdl_plan* p, const CorrArgs& c, int fold, bool octet, bool& ok) {
  SplitArgs a{};
  a.c = c;
  a.ci = (int32_t)p->n_ci;
  a.co = (int32_t)p->n_co;
  a.taps = p->ksize[0] * p->ksize[1] * p->ksize[2];
  a.k1 = p->ksize[1];
  a.k2 = p->ksize[2];
  a.dil2 = p->dilation[2];
  a.fold = fold;
  a.nch = c.nc;
  a.div_nch = make_fastdiv((uint32_t)a.nch);
  if (fold == 1) {
    for (int t = 0; t < c.nt[2]; ++t) a.off2[t] = c.tapoff[2][t];
  } else {
    const int s = p->stride[2];
    a.c.nc = fold * a.nch;
    a.c.ntn = (a.c.nc + 31) / 32;
    a.c.is[2] = c.mode == 0 ? fold * s : fold / s;
    std::vector<int> off;
    for (int j = 0; j < fold; ++j)
      for (int t = 0; t < a.k2; ++t) {
        const int at = c.mode == 0 ? j * s + t * a.dil2 : j - t * a.dil2;
        if (c.mode == 0) off.push_back(at);
        else if (at % s == 0) off.push_back(at / s);
      }
    std::sort(off.begin(), off.end());
    off.erase(std::unique(off.begin(), off.end()), off.end());
    a.c.nt[2] = (int32_t)off.size();
    if (off.size() > kMaxOff2) return ok = false, a;
    std::copy(off.begin(), off.end(), a.off2);
  }
  ok = group_taps(a, octet, fold > 1 || octet ? kFewTaps : kGroupTaps);
  return a;
}

int64_t weight_pieces(const SplitArgs& a) {
  return (int64_t)a.c.ntn * a.c.nt[0] * (a.nfull * a.gbegin[a.ngroups] + a.npairs) * 192;
}

int64_t tiles_of_worker(const PerWorker& g, const CorrArgs& c) {
  return (((int64_t)c.n_b * g.nq[0] + c.g0 - 1) / c.g0) * ((g.nq[1] + c.tr - 1) / c.tr) * ((g.nq[2] + c.tc - 1) / c.tc) * c.ntn;
}

// The launches of one direction (forward: one; data gradient: one per class), sorted by kernel variant; kept in the plan.
struct Launch {
  SplitArgs a;
  int variant = 0;  // index into the switch of launch_variants
  unsigned blocks = 0;
  int64_t pieces = 0;  // of weights
  double clocks = 0, share = 1;  // estimates: time alone; part of the chip that it fills
  double used = 1;               // part of the multiplied positions that are outputs
};
struct Launches {
  std::vector<Launch> v;
  int64_t pieces = 0;  // all of them
  double clocks = 0;   // estimate
  double used = 1;     // of the launch that uses its windows least
};
struct SplitPlan {
  Launches dir[2];
  bool ok[2] = {false, false};
  int64_t tried = 0;         // windows
  SplitArgs* dev = nullptr;  // forward, then the classes
  ~SplitPlan() {
    if (dev) (void)hipFree(dev);
  }
};

constexpr double kFewSetup = 20.0e3;  // clocks
// `limit`: launches that take more clocks are not wanted
bool plan_launch(const distdl_plan* p, const CorrArgs& c, int fold, bool octet, double limit, Launch& l, int64_t& tried) {
  bool ok;
  l.a = split_args(p, c, fold, octet, ok);
  SplitArgs& a = l.a;
  if (!ok) return false;
  const double setup = few_channels(a) ? kFewSetup : 12.0e3;
  {  // set-up, and what the matrix cores take with no position idle
    double positions = 0;
    for (const WorkerDev& wd : p->workers) {
      const PerWorker g = derive_of(wd, &a);
      positions = std::max(positions, (double)p->n_b * g.nq[0] * g.nq[1] * g.nq[2]);
    }
    const double tiles = positions * p->n_workers * a.c.ntn / (128.0 * 256);
    if (setup + tiles * a.c.nt[0] * (a.nfull * a.gbegin[a.ngroups] + a.npairs) * 6 * 32.0 * 1.4 > limit) return false;
  }
  const int mt = choose_window(p, a, l.used, tried);
  if (mt == 0) return false;
  l.variant = (mt == 3 ? 3 : mt == 1 ? 0 : pieces_of(a, a.c.R * a.c.Cw) <= 3 ? 1 : 2) + (few_channels(a) ? 4 : 0);
  l.pieces = weight_pieces(a);
  // Output planes per workgroup: a fixed set-up (its address tables, about 8 * 10^3 clocks) against the number of rounds
  // of 512 workgroups; at least four groups per worker where neighbouring planes share input planes (conv_mfma.hip).
  int64_t planes_max = 0, per_plane = 0;
  for (const WorkerDev& wd : p->workers) {
    const PerWorker g = derive_of(wd, &a);
    planes_max = std::max<int64_t>(planes_max, p->n_b * g.nq[0]);
    per_plane = std::max<int64_t>(per_plane, (int64_t)((g.nq[1] + a.c.tr - 1) / a.c.tr) * ((g.nq[2] + a.c.tc - 1) / a.c.tc) * a.c.ntn);
  }
  per_plane *= p->n_workers;
  const int ncc = a.nfull + (a.npairs > 0), mfmas = a.nfull * a.gbegin[a.ngroups] + a.npairs;
  const double stage = (double)a.c.nt[0] * (mfmas * mt * 6 * 32.0 * 2 * 1.4 + ncc * a.ngroups * 1500.0);
  const int tstep0 = a.c.nt[0] > 1 ? a.c.tapoff[0][1] - a.c.tapoff[0][0] : 0;
  const bool shares = tstep0 != 0 && a.c.is[0] % tstep0 == 0 && (a.c.is[0] / tstep0) % a.c.nt[0] != 0;
  const int64_t g0_max = shares ? std::max<int64_t>(1, planes_max / 4) : std::max<int64_t>(1, planes_max);
  double best = 1e300;
  a.c.g0 = 1;
  for (int64_t g0 = 1, next; g0 <= g0_max; g0 = next) {
    const int64_t groups = (planes_max + g0 - 1) / g0, wgs = groups * per_plane;
    next = groups > 1 ? (planes_max + groups - 2) / (groups - 1) : g0_max + 1;  // (more planes in as many groups take longer)
    const double cost = (double)((wgs + 511) / 512) * (8.0e3 + g0 * stage);
    if (cost < best * 0.97) best = cost, a.c.g0 = (int32_t)g0;
  }
  {  // stages of a workgroup that is alone on its compute unit are longer than what the matrix cores need
    const int64_t wgs = (planes_max + a.c.g0 - 1) / a.c.g0 * per_plane;
    const double one = (double)a.c.nt[0] * (mfmas * mt * 6 * 32.0 * 1.4 * (wgs > 256 ? 2 : 1) + ncc * a.ngroups * 2500.0);
    l.share = std::min(1.0, wgs / 512.0);
    l.clocks = (double)((wgs + 511) / 512) * (setup + a.c.g0 * one);
  }
  int64_t tiles = 0;
  for (const WorkerDev& wd : p->workers) tiles = std::max(tiles, tiles_of_worker(derive_of(wd, &a), a.c));
  const int64_t blocks = (tiles * p->n_workers + 7) / 8 * 8;
  if (blocks >= kMaxBlocks256) return false;
  a.c.tiles_max = (int32_t)tiles;
  l.blocks = (unsigned)blocks;
  return true;
}

// launches v[0 ... count) of one variant, which lie at tab[first] ... in the plan's table
template <int MT, int PA, int PB, bool FEW>
int launch_variant(distdl_plan* p, const SplitArgs* tab, int first, const Launch* v, int count, const u32x4* wt, const float* w,
                   const float* bias, void** in_tab, void** out_tab, const char* name, hipStream_t st) {
  unsigned blocks = 0;
  int lds = 0;
  for (int i = 0; i < count; ++i) blocks = std::max(blocks, v[i].blocks), lds = std::max(lds, split_lds_bytes(PA, v[i].a.c.ck));
  if (count > 1 && blocks <= 2048) {
    if (blocks == 0) return DISTDL_OK;
    if (lds > 64 * 1024)
      if (int rc = allow_large_lds<corr_split_classes_kernel<MT, PA, PB, FEW>>()) return rc;
    ProfScope prof(name, st);
    hipLaunchKernelGGL((corr_split_classes_kernel<MT, PA, PB, FEW>), dim3(blocks, (unsigned)count), dim3(256), lds, st, p->d_workers,
                       in_tab, out_tab, tab, first, wt, w, bias);
    return DISTDL_OK;
  }
  if (lds > 64 * 1024)
    if (int rc = allow_large_lds<corr_split_kernel<MT, PA, PB, FEW>>()) return rc;
  for (int i = 0; i < count; ++i) {
    if (v[i].blocks == 0) continue;
    ProfScope prof(name, st);
    hipLaunchKernelGGL((corr_split_kernel<MT, PA, PB, FEW>), dim3(v[i].blocks), dim3(256), split_lds_bytes(PA, v[i].a.c.ck), st,
                       p->d_workers, in_tab, out_tab, v[i].a, wt, w, bias);
  }
  return DISTDL_OK;
}

int table_of(SplitPlan& sp) {
  if (sp.dev) return DISTDL_OK;
  std::vector<SplitArgs> all;
  for (const Launches& d : sp.dir)
    for (const Launch& l : d.v) all.push_back(l.a);
  SplitArgs* dev = nullptr;
  DISTDL_HIP_TRY(hipMalloc((void**)&dev, all.size() * sizeof(SplitArgs)));
  if (hipError_t e = hipMemcpy(dev, all.data(), all.size() * sizeof(SplitArgs), hipMemcpyHostToDevice); e != hipSuccess) {
    (void)hipFree(dev);
    DISTDL_HIP_TRY(e);
  }
  sp.dev = dev;
  return DISTDL_OK;
}

// One direction, its weights laid out: one launch per kernel variant.
int run_split(distdl_plan* p, int dir, const float* w, const float* bias, void** in_tab, void** out_tab, const char* name,
              hipStream_t st) {
  SplitPlan& sp = *(SplitPlan*)p->corr_split_plan.get();
  const Launches& d = sp.dir[dir];
  const int first = dir == 0 ? 0 : (int)sp.dir[0].v.size();
  const u32x4* const wt = (const u32x4*)p->d_wt;
  constexpr int kPb = (kGroupTaps * 192 + 255) / 256, kPb3 = (9 * 192 + 255) / 256,
                kPbFew = (kFewTaps * 192 + 255) / 256;
  for (size_t i = 0; i < d.v.size();) {
    size_t e = i;
    while (e < d.v.size() && d.v[e].variant == d.v[i].variant) ++e;
    const Launch* const v = &d.v[i];
    const int at = first + (int)i, n = (int)(e - i);
    int rc;
    switch (v->variant) {
#define DISTDL_SPLIT(MT_, PA_, PB_, FEW_) \
  rc = launch_variant<MT_, PA_, PB_, FEW_>(p, sp.dev, at, v, n, wt, w, bias, in_tab, out_tab, name, st)
      case 0: DISTDL_SPLIT(1, 4, kPb, false); break;
      case 1: DISTDL_SPLIT(2, 3, kPb, false); break;
      case 2: DISTDL_SPLIT(2, 4, kPb, false); break;
      case 3: DISTDL_SPLIT(3, 4, kPb3, false); break;
      case 4: DISTDL_SPLIT(1, 4, kPbFew, true); break;
      case 5: DISTDL_SPLIT(2, 3, kPbFew, true); break;
      default: DISTDL_SPLIT(2, 4, kPbFew, true);
#undef DISTDL_SPLIT
    }
    if (rc) return rc;
    i = e;
  }
  return DISTDL_OK;
}

SplitPlan* split_plan(const distdl_plan* p) {
  static std::mutex lock;
  std::lock_guard<std::mutex> hold(lock);
  if (p->corr_split_plan) return (SplitPlan*)p->corr_split_plan.get();
  auto sp = std::make_shared<SplitPlan>();
  p->corr_split_plan = sp;
  if (p->explicit_halo || p->dtype != DISTDL_F32) return sp.get();
  // buffer instructions address one worker's tensor with 31-bit byte offsets
  const double most = (double)p->n_b * std::max(p->n_ci, p->n_co) * 4.0;
  if (most * p->max_buf_cells >= 2147480000.0 || most * p->max_out_cells >= 2147480000.0) return sp.get();
  for (int d = 0; d < 3; ++d)
    if (p->ksize[d] > 8 || p->stride[d] > 4) return sp.get();
  for (int dir = 0; dir < 2; ++dir) {
    if ((dir == 0 ? p->n_ci : p->n_co) % 4) continue;  // the tensor that is read comes in 16-byte pieces
    Launches& d = sp->dir[dir];
    // The launches with `fold` cells to a position (data gradient: a class per residue of the dimensions that are not folded), of
    // all folds those that are estimated to take the least time.  One cell to a position and no shared products unless another form
    // takes less than 0.9 of that (737 directions of 370 layers: at 0.97 11 of them took 1.04 to 1.33 times as long as in the
    // general form, 24 -> 4, 5^3, 8 x 45 x 44 x 46, forward 985 us and 741; at 0.9 three).  0.97 for the data gradient with a stride
    // and cells of at most 96 bytes, which the classes of the general form write apart: 8 <- 48, 2 taps, stride 2, 7 x 392639, 172 us
    // in two classes, 123 folded.  0.65 for a forward pass of three dimensions whose cells are folded under a dilation: the cells of a
    // position share few offsets, and of eight such layers with estimates between that and 0.9 five took up to 1.3 times as long, 1.10 in
    // the mean (32 -> 10, 5^3, dilation 2, 4 x 29 x 29 x 38, estimate 0.76: 299 us and 231; 48 -> 5, 7 x 24 x 46 x 47, 0.79: 563 and 653).
    const int nch = (int)(dir == 0 ? p->n_co : p->n_ci), kc = (int)(dir == 0 ? p->n_ci : p->n_co), s2 = dir == 0 ? 1 : p->stride[2];
    const double margin = s2 > 1 && nch <= 24 ? 0.97 : 0.9;
    double limit = 1e300, general = 1e300;
    for (int fold = 1; fold <= 32; fold = fold < s2 ? s2 : fold + s2) {
      // (one class instead of several along dimension 2 pays for any columns; FEW keeps the bounds of a position's in 16 bits)
      if (fold > 1 && (int64_t)fold * nch > (fold == s2 ? kMaxFewColumns : 32)) break;
      for (const bool octet : {false, true}) {
        if (octet && (kc % 16 == 0 || kc % 16 > 8 || nch > kMaxFewColumns)) continue;
        if (kFewSetup >= limit) continue;  // (the general form comes first)
        const bool spread = dir == 0 && fold > 1 && !octet && p->dilation[2] > 1 && p->ksize[0] > 1;
        Launches l;
        double sum = 0, most = 0;  // (classes that fill the chip together only are one launch)
        bool ok = true;
        auto add = [&](const CorrArgs& c) {
          if (!ok) return;
          l.v.emplace_back();
          ok = plan_launch(p, c, fold, octet, limit, l.v.back(), sp->tried);
          sum += l.v.back().clocks * l.v.back().share;
          l.used = std::min(l.used, l.v.back().used);
          most = std::max(most, l.v.back().clocks);
          ok = ok && std::max(sum, most) < (spread ? std::min(limit, 0.65 * general) : limit);
        };
        if (dir == 0) add(forward_args(p));
        else
          for (int p0 = 0; p0 < p->stride[0]; ++p0)
            for (int p1 = 0; p1 < p->stride[1]; ++p1)
              for (int p2 = 0; p2 < (fold == 1 ? p->stride[2] : 1); ++p2) {
                const int par[3] = {p0, p1, p2};
                add(class_args(p, par));
              }
        if (!ok) continue;
        l.clocks = std::max(sum, most);
        if (fold == 1 && !octet) general = l.clocks;
        limit = l.clocks * (fold == 1 && !octet ? margin : 0.97);
        d = std::move(l);
      }
    }
    if (d.v.empty()) continue;
    std::stable_sort(d.v.begin(), d.v.end(), [](const Launch& x, const Launch& y) { return x.variant < y.variant; });
    for (Launch& l : d.v) {
      l.a.woff = d.pieces;
      d.pieces += l.pieces;
    }
    sp->ok[dir] = true;
  }
  return sp.get();
}

}  // namespace

bool corr_split_supported(const distdl_plan* p, bool backward) { return split_plan(p)->ok[backward ? 1 : 0]; }

// Estimated time: that of the clocks that chose the launches (fitted to 144 directions, nine tenths within a fifth where the
// tensors are small), and the tensors.
double corr_split_used(const distdl_plan* p, bool backward) { return split_plan(p)->dir[backward ? 1 : 0].used; }
double corr_split_us(const distdl_plan* p, bool backward) {
  const double cells = (double)p->n_workers * p->n_b * (backward ? p->max_buf_cells : p->max_out_cells);
  return 2.7 + split_plan(p)->dir[backward ? 1 : 0].clocks / 2240 + cells * (double)(p->n_ci + p->n_co) * 0.65e-6;
}

void corr_split_shape(const distdl_plan* p, bool backward, int32_t out[5]) {
  const Launches& d = split_plan(p)->dir[backward ? 1 : 0];
  out[0] = (int32_t)d.v.size();
  out[1] = out[2] = out[3] = 0;
  out[4] = (int32_t)std::min<int64_t>(split_plan(p)->tried, INT32_MAX);
  for (const Launch& l : d.v) {
    out[1] = l.a.fold;
    out[2] = std::max(out[2], l.a.c.nc);
    out[3] = std::max(out[3], l.a.npairs);
  }
}

int split_weight_job(distdl_plan* p, bool backward, const float* w, hipStream_t st, WeightJob& job) {
  SplitPlan& sp = *(SplitPlan*)p->corr_split_plan.get();
  if (int rc = table_of(sp)) return rc;
  if (int rc = ensure_wscratch(p, (size_t)std::max(sp.dir[0].pieces, sp.dir[1].pieces) * 4, st)) return rc;
  const Launches& d = sp.dir[backward ? 1 : 0];
  int64_t most = 0;
  for (const Launch& l : d.v) most = std::max(most, l.pieces / 3);  // threads: three pieces each
  job.kind = most > 0 ? 1 : 0;
  job.per_class = (int32_t)((most + 255) / 256);
  job.blocks = job.per_class * (int32_t)d.v.size();
  job.tab = sp.dev;
  job.first = backward ? (int32_t)sp.dir[0].v.size() : 0;
  job.w = w;
  job.dst = (split_u32x4*)p->d_wt;
  return DISTDL_OK;
}

int conv_fwd_split(distdl_plan* p, const float* w, const float* bias, hipStream_t st) {
  return run_split(p, 0, w, bias, p->tab_x.dev, p->tab_y.dev, "conv_fwd_split", st);
}

int conv_bwd_data_split(distdl_plan* p, const float* w, hipStream_t st) {
  return run_split(p, 1, w, nullptr, p->tab_dy.dev, p->tab_dx.dev, "conv_bwd_data_split", st);
}

}  // namespace distdl
