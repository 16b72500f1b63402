// Weight gradient of fp32 convolutions on the bf16 matrix cores (split_bf16.h): dW[tap][ci][co] and db, one partial per
// worker and chunk of its output positions.
//
// A workgroup holds one kernel plane t0, a chunk of cc input channels and NT * 16 output channels.  The rows of its
// product are (tap of the plane, input channel) without padding between taps, in tiles of 16; the columns are output
// channels; the sum runs over output positions, 32 of one output row (a step) at a time.  The waves walk the output rows
// together: the input rows that a step reads lie in LDS as a ring of span + s1 rows, each step fetches its s1 new rows
// and the dy row one step ahead through registers, splits them into three bf16 planes once, and writes them; as the ring
// has s1 spare rows and dy two buffers, one barrier a step is enough.
//
// MFMA operands need eight consecutive positions per lane, from rows whose channels are consecutive:
// ds_read_b64_tr_b16 (in a group of 16 lanes, lane 4 b + a receives as element v the a-th of the four 16-bit elements
// that lane b + 4 v addresses).  Lane s of group g addresses four rows, 4 (s % 4) ..., of position 4 g + s / 4 (and
// 16 more): which rows is each lane's own matter, so a tile may hold rows of several taps.  k slot (g, v) is position
// 4 g + v on both sides.
//
// LDS of a ring row: [plane][channel group][cell][channel], cells of a stride-2 row by residue, so that consecutive
// positions are consecutive in LDS for every tap; groups of 16 channels where cc allows: a read of 16 positions x 16 channels
// is then 512 contiguous bytes and free of bank conflicts.
//
// A step takes tiles * NT * 6 MFMAs of 16 clocks; a tile's operand (6 reads, 3 KiB) serves all NT columns, those of dy stay in
// registers over the tiles.  At 32 -> 32 channels, 5^3, stride 2, 256^3 on 64 workers the matrix pipes issue in 47 % of the
// cycles (at 2.03 GHz: 1.04 PFLOP/s in bf16) and LDS is active in 27 %; what bounds it is vector instructions, 3.3 of 4
// clocks beside each MFMA of 16: splitting the staged pieces, the addresses of six reads a tile, the sums' additions.
//
// The sums of a step start from zero and join the running sums by a vector instruction.  A bf16 MFMA drops the bits of its
// products that lie below its largest operand, towards minus infinity: over 10^3 steps in one accumulator that bias made an
// error of 6.7e-6 (fp32 MFMAs: 1.1e-6), 1.6e-6 with a fresh start each step.  So every other step multiplies by -dy and
// subtracts: the biases cancel, 3.1e-7.
//
// Against fp32 MFMAs with a tap a tile (us, fp32, this kernel alone):
//   32 -> 32, 5^3, stride 2, 256^3, 64 workers:       4480 -> 3070
//   24 -> 40, 3^3, 2 x 61 x 75 x 58, 12 workers:       515 -> 235
//   56 -> 44, 3 x 3 with dilation 2, 3 x 291 x 355:    258 -> 120
//   4 -> 4, 5 x 5, 6 x 528 x 776:                     1303 -> 140
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "buffer.h"
#include "conv_wsplit.h"
#include "profile.h"
#include "split_bf16.h"

namespace distdl {

namespace {

constexpr int kNx = 4;                  // input pieces per thread and step
// Row tiles of a workgroup: seven for each of eight waves, five with three columns and three with four (more sums than
// that leave a lane's 256 registers).
constexpr int max_tiles(int nt) { return nt == 4 ? 24 : nt == 3 ? 40 : 56; }
constexpr int kLds = 160 * 1024;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16* lds_v4;

struct Args {
  int32_t n_b, ci, co;
  int32_t k[3], s[3], dil[3];
  int32_t nchunks, ob;         // chunks of units per worker; output rows per unit
  int32_t r, lc;               // a step is r output rows by 2^lc columns: 32 positions
  int32_t ncell, half, cells;  // cells a row segment reads; of one residue; places for cells (half * s2)
  int32_t span, ring;          // input rows an output row reads; rows in LDS
  int32_t cc, nci, gw, ncob;   // input channels per workgroup, chunks of them, channels per group; blocks of output channels
  int32_t tiles;               // of 16 rows
  int64_t slot;                // floats of a partial
};

__device__ inline bf16x8 operand(const char* first, const char* second) {
  union {
    v4i16 half[2];
    bf16x8 v;
  } f;
  f.half[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)first);
  f.half[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)second);
  return f.v;
}

// the operand's numbers, from its upper and lower halves
__device__ inline Eight halves(const char* first, const char* second, uint32_t plane) {
  return join_halves(__builtin_bit_cast(u32x4, operand(first, second)), __builtin_bit_cast(u32x4, operand(first + plane, second + plane)));
}

// four channels of a cell or position; RAW: as they are, for fp32 MFMAs
template <bool RAW>
__device__ inline void put_split(char* at, uint32_t plane, u32x4 v, float scale = kSplitScale) {
  u32x2 hi, mid, lo;
  if constexpr (RAW) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      uint32_t a, b;
      halve_pair(v[2 * j], v[2 * j + 1], a, b);
      hi[j] = a, mid[j] = b;
    }
    *(u32x2*)at = hi;
    *(u32x2*)(at + plane) = mid;
    return;
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    uint32_t a, b, c;
    split_pair(__uint_as_float(v[2 * j]), __uint_as_float(v[2 * j + 1]), scale, a, b, c);
    hi[j] = a, mid[j] = b, lo[j] = c;
  }
  *(u32x2*)at = hi;
  *(u32x2*)(at + plane) = mid;
  *(u32x2*)(at + 2 * plane) = lo;
}

// grid: (kernel planes, channel chunks x column blocks, workers x chunks)
template <int NW, int MT, int NT>
__global__ __launch_bounds__(64 * NW, 2) void wgrad_split_kernel(const WorkerDev* __restrict__ workers, void* const* x_bufs,
                                                                 void* const* dy_bufs, float* __restrict__ partial, Args a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int TH = 64 * NW, NY = (NT * 128 + TH - 1) / TH;
  constexpr uint32_t kYPlane = NT * 1024, kYBuf = 3 * kYPlane;
  const int tid = threadIdx.x, lane = tid & 63, lg = lane >> 4, ls = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // The workgroups of the k0 planes of one (worker, chunk, channels) read the same input planes: they take consecutive
  // places on one XCD and walk their units rotated, so that at one moment they are on the same plane.
  uint32_t bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
  {
    const uint32_t nblk = gridDim.x * gridDim.y * gridDim.z;
    if ((nblk & 7u) == 0) {
      const uint32_t lin = bx + gridDim.x * (by + gridDim.y * bz);
      const uint32_t r = (lin & 7u) * (nblk >> 3) + (lin >> 3);
      bx = r % gridDim.x;
      const uint32_t rest = r / gridDim.x;
      by = rest % gridDim.y;
      bz = rest / gridDim.y;
    }
  }
  const int t0 = (int)bx, cic = (int)by / a.ncob, cob = (int)by - cic * a.ncob;
  const int worker = (int)bz / a.nchunks, chunk = (int)bz - worker * a.nchunks;
  const WorkerDev wd = workers[worker];
  const int cols = 1 << a.lc, nr = a.r * a.s[1];  // columns of a step, and its new input rows
  const int s1 = a.s[1], T = a.k[1] * a.k[2], quads = a.cc >> 2;
  const int ci0 = cic * a.cc, co0 = cob * NT * 16;
  const uint32_t cellb = (uint32_t)a.gw * 2u, groupb = (uint32_t)a.cells * cellb, planeb = (uint32_t)a.cells * a.cc * 2u,
                 rowb = 3u * planeb, ringb = (uint32_t)a.ring * rowb;
  char* const ys = smem + ((ringb + 15u) & ~15u);

  const uint32_t sx2 = a.ci, sx1 = wd.buf[2] * sx2, sx0 = wd.buf[1] * sx1, sxn = wd.buf[0] * sx0;
  const uint32_t sy2 = a.co, sy1 = wd.out[2] * sy2, sy0 = wd.out[1] * sy1, syn = wd.out[0] * sy0;
  const __amdgpu_buffer_rsrc_t rx = rsrc_of(x_bufs[worker], (uint32_t)a.n_b * sxn * 4u);
  const __amdgpu_buffer_rsrc_t ry = rsrc_of(dy_bufs[worker], (uint32_t)a.n_b * syn * 4u);

  // place in a ring row of the channel c (a multiple of 4) of cell `cell`
  auto place = [&](int cell, int c) -> uint32_t {
    const int r = cell % a.s[2], at = r * a.half + cell / a.s[2];
    const int grp = c / a.gw;
    return (uint32_t)grp * groupb + (uint32_t)at * cellb + (uint32_t)(c - grp * a.gw) * 2u;
  };

  // this wave's tiles: first, first + 1, ...; at least MT - 1 of them are multiplied (repeated if need be, and not stored)
  const int tbase = a.tiles / NW, trem = a.tiles - tbase * NW;
  const int first = wave * tbase + min(wave, trem), ntw = tbase + (wave < trem ? 1 : 0);
  const int rows = T * a.cc;
  uint32_t toff[MT];  // ring place of the lane's four rows of tile i and position, without the ring row
  int trow[MT];       // window row of that tap
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    int r = (first + max(0, min(i, ntw - 1))) * 16 + 4 * (ls & 3);
    if (r >= rows) r = 0;  // never stored
    const int tap = r / a.cc, c = r - tap * a.cc, t1 = tap / a.k[2], t2 = tap - t1 * a.k[2];
    const int pos = 4 * lg + (ls >> 2);
    toff[i] = place(t2 * a.dil[2], c) + (uint32_t)(pos & (cols / 2 - 1)) * cellb;
    trow[i] = t1 * a.dil[1] + (pos >> (a.lc - 1)) * s1;
  }
  floatx4 acc[MT][NT];

  const int row_cells = wd.buf[2] - wd.origin[2];
  const int O1 = wd.out[1], O2 = wd.out[2], nseg = (O2 + cols - 1) >> a.lc;
  const int nblk1 = (O1 + a.ob - 1) / a.ob;
  const int nunits = a.n_b * wd.out[0] * nblk1;
  const int per = (nunits + a.nchunks - 1) / a.nchunks;
  const int unit_end = min(nunits, (chunk + 1) * per);

  // pieces of four channels: of the new input rows, and of the dy positions
  const int rowp = a.ncell * quads, npieces = nr * rowp;
  uint32_t pdst[kNx], pvo[kNx], psrc[kNx];
  int pcell[kNx], prr[kNx];
#pragma unroll
  for (int i = 0; i < kNx; ++i) {
    const int idx = i * TH + tid, rr = idx / rowp, rest = idx - rr * rowp, cell = rest / quads, c = (rest - cell * quads) * 4;
    prr[i] = rr;
    pcell[i] = idx < npieces && ci0 + c < a.ci ? cell : 0x40000000;
    pdst[i] = (uint32_t)rr * rowb + place(cell, c);
    psrc[i] = ((uint32_t)rr * sx1 + (uint32_t)cell * sx2 + ci0 + c) * 4u;
  }
  uint32_t yvo[NY];
  auto setup_pieces = [&](int seg) {
#pragma unroll
    for (int i = 0; i < kNx; ++i) pvo[i] = seg * cols * a.s[2] + pcell[i] < row_cells ? psrc[i] : kOob;
#pragma unroll
    for (int i = 0; i < NY; ++i) {
      const int u = i * TH + tid, pos = u / (4 * NT), c = co0 + u % (4 * NT) * 4;
      const int row = (pos & 15) >> (a.lc - 1), col = seg * cols + (pos & (cols / 2 - 1)) + (pos >> 4) * (cols / 2);
      yvo[i] = pos < 32 && col < O2 && c < a.co ? ((uint32_t)row * sy1 + (uint32_t)col * sy2 + c) * 4u : kOob;
    }
  };
  u32x4 rp[kNx], rpy[NY];
  auto fetch = [&](int n, int o0, int o1, int o1_end, int seg) {
    const int c0 = wd.origin[0] + o0 * a.s[0] + t0 * a.dil[0];
    const int r_first = wd.origin[1] + o1 * s1 + a.span - s1;  // buffer row of new row 0
    const uint32_t xb = ((uint32_t)n * sxn + (uint32_t)c0 * sx0 + (uint32_t)r_first * sx1 +
                         (uint32_t)(wd.origin[2] + seg * cols * a.s[2]) * sx2) * 4u;
#pragma unroll
    for (int i = 0; i < kNx; ++i)
      if (i * TH < npieces)  // (uniform)
        rp[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, r_first + prr[i] < wd.buf[1] ? pvo[i] : kOob, xb, 0);
    const uint32_t yb = ((uint32_t)n * syn + (uint32_t)o0 * sy0 + (uint32_t)o1 * sy1) * 4u;
#pragma unroll
    for (int i = 0; i < NY; ++i)
      rpy[i] = __builtin_amdgcn_raw_buffer_load_b128(ry, o1 + (((i * TH + tid) / (4 * NT) & 15) >> (a.lc - 1)) < o1_end ? yvo[i] : kOob, yb, 0);
  };
  // db of this chunk: the workgroups of plane 0 and channel chunk 0 see each dy element of their columns once
  const bool bias_wg = t0 == 0 && cic == 0;
  // (a unit's sums on their own first: one running sum over all steps is further off)
  float bsum[NY][4], btotal[NY][4];
#pragma unroll
  for (int i = 0; i < NY; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) bsum[i][j] = btotal[i][j] = 0.f;
  uint32_t nslot = 0;  // ring place of the step's new row 0
  auto wrap = [&](uint32_t at) { return min(at, at - ringb); };  // at < 2 ringb
  auto stash = [&](auto raw, uint32_t odd) {
    constexpr bool RAW = decltype(raw)::value;
    // All loads are in.  (Said here because on the paths that skip a piece the compiler cannot see it, and would wait for the
    // next step's loads before it multiplies.)
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
#pragma unroll
    for (int i = 0; i < kNx; ++i)
      if (i * TH < npieces) {
        if (i * TH + tid < npieces) put_split<RAW>(smem + wrap(pdst[i] + nslot), planeb, rp[i]);
      }
#pragma unroll
    for (int i = 0; i < NY; ++i) {
      const int u = i * TH + tid, pos = u / (4 * NT), q = u % (4 * NT);
      if (pos < 32)
        put_split<RAW>(ys + odd * kYBuf + (q >> 2) * 1024 + pos * 32 + (q & 3) * 8, kYPlane, rpy[i], odd ? -kSplitScale : kSplitScale);
      if (bias_wg && !RAW)
#pragma unroll
        for (int j = 0; j < 4; ++j) bsum[i][j] += __uint_as_float(rpy[i][j]);
    }
  };
  const uint32_t lane_y = (uint32_t)((4 * lg + (ls >> 2)) * 32 + (ls & 3) * 8);
  const uint32_t more = (uint32_t)(cols / 2) * cellb;  // to the other sixteen positions
  const uint32_t tstep = (uint32_t)nr * rowb;
  const int unit_begin = chunk * per, unit_cnt = unit_end - unit_begin;
  const int skew = unit_cnt > 0 ? (((a.k[0] - 1 - t0) * a.dil[0]) / a.s[0] * nblk1) % unit_cnt : 0;
  // All units of this workgroup, with operands that are split, or (RAW) multiplied as they are.
  auto pass = [&](auto raw) __attribute__((always_inline)) {
  constexpr bool RAW = decltype(raw)::value;
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  uint32_t odd = 0;  // which dy buffer, and sign, the next step takes
  for (int uj = 0; uj < unit_cnt; ++uj) {
    const int unit = unit_begin + (uj + skew < unit_cnt ? uj + skew : uj + skew - unit_cnt);
    const int plane = unit / nblk1, o1_begin = (unit - plane * nblk1) * a.ob, o1_end = min(O1, o1_begin + a.ob);
    const int o0 = plane % wd.out[0], n = plane / wd.out[0];
    if (bias_wg && !RAW)
#pragma unroll
      for (int i = 0; i < NY; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) btotal[i][j] += bsum[i][j], bsum[i][j] = 0.f;
    for (int seg = 0; seg < nseg; ++seg) {
      setup_pieces(seg);
      nslot = (uint32_t)((o1_begin * s1 + a.span - s1) % a.ring) * rowb;
      uint32_t taddr[MT];
#pragma unroll
      for (int i = 0; i < MT; ++i) taddr[i] = (uint32_t)((o1_begin * s1 + trow[i]) % a.ring) * rowb + toff[i];
      __syncthreads();  // previous unit / segment fully consumed
      fetch(n, o0, o1_begin, o1_end, seg);
      {  // the first span - s1 window rows of step o1_begin
        const int c0 = wd.origin[0] + o0 * a.s[0] + t0 * a.dil[0];
        const uint32_t xb = ((uint32_t)n * sxn + (uint32_t)c0 * sx0 + (uint32_t)(wd.origin[2] + seg * cols * a.s[2]) * sx2 + ci0) * 4u;
        const int total = (a.span - s1) * rowp;
        for (int base = 0; base < total; base += 4 * TH) {
          u32x4 v[4];
          uint32_t at[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int idx = base + i * TH + tid, rr = idx / rowp, rest = idx - rr * rowp, cell = rest / quads, c = (rest - cell * quads) * 4;
            const int wrow = o1_begin * s1 + rr, row = wd.origin[1] + wrow;
            const bool ok = idx < total && row < wd.buf[1] && seg * cols * a.s[2] + cell < row_cells && ci0 + c < a.ci;
            v[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, ok ? ((uint32_t)row * sx1 + (uint32_t)cell * sx2 + c) * 4u : kOob, xb, 0);
            at[i] = (uint32_t)(wrow % a.ring) * rowb + place(cell, c);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (base + i * TH + tid < total) put_split<RAW>(smem + at[i], planeb, v[i]);
        }
      }
      for (int o1 = o1_begin; o1 < o1_end; o1 += a.r, odd ^= 1u) {
        stash(raw, odd);
        __syncthreads();  // step o1 staged; every wave has finished step o1 - 1
        if (o1 + a.r < o1_end) fetch(n, o0, o1 + a.r, o1_end, seg);  // in flight while this step multiplies
        const char* const yb = ys + odd * kYBuf + lane_y;
        if constexpr (RAW) {
          Eight xb[NT];
#pragma unroll
          for (int j = 0; j < NT; ++j) xb[j] = halves(yb + j * 1024, yb + j * 1024 + 512, kYPlane);
          // a position beyond the output has a dy of zero, which does not cancel a cell that is not finite
          bool there[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int pos = 4 * lg + (e & 3), row = pos >> (a.lc - 1), col = seg * cols + (pos & (cols / 2 - 1)) + (e >> 2) * (cols / 2);
            there[e] = o1 + row < o1_end && col < O2;
          }
#pragma unroll
          for (int i = 0; i < MT; ++i) {
            Eight xa = halves(smem + taddr[i], smem + taddr[i] + more, planeb);
#pragma unroll
            for (int e = 0; e < 8; ++e) xa.v[e] = there[e] ? xa.v[e] : 0.f;
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
              for (int e = 0; e < 8; ++e) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa.v[e], xb[j].v[e], acc[i][j], 0, 0, 0);
          }
        } else {
        const float sign = odd ? -kUnsplit : kUnsplit;
        bf16x8 fb[NT][3];
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
          for (int pl = 0; pl < 3; ++pl)
            fb[j][pl] = operand(yb + j * 1024 + pl * kYPlane, yb + j * 1024 + pl * kYPlane + 512);
        // Tile by tile: the operands of the next one are read, and the sums of the last one added, while one is multiplied.
        // (Left alone the compiler keeps the sums of all tiles to the end of the step, and runs out of registers.)
        bf16x8 fa[2][3];
        floatx4 sum[2][NT];
        auto read = [&](int i) {
          const char* const at = smem + taddr[i];
#pragma unroll
          for (int pl = 0; pl < 3; ++pl) fa[i & 1][pl] = operand(at + pl * planeb, at + pl * planeb + more);
        };
        auto multiply = [&](int i) {
          constexpr int pa[6] = {2, 1, 0, 1, 0, 0}, pb[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
          for (int j = 0; j < NT; ++j) sum[i & 1][j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int j = 0; j < NT; ++j)
              sum[i & 1][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i & 1][pa[q]], fb[j][pb[q]], sum[i & 1][j], 0, 0, 0);
        };
        auto add = [&](int i) {
#pragma unroll
          for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][e] = fmaf(sum[i & 1][j][e], sign, acc[i][j][e]);
#pragma unroll
          for (int j = 0; j < NT; ++j) asm volatile("" : "+v"(acc[i][j]));  // here, and no later
        };
        read(0);
#pragma unroll
        for (int i = 0; i < MT - 1; ++i) {
          read(i + 1);
          multiply(i);
          if (i > 0) add(i - 1);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (ntw == MT) {  // (uniform)
          multiply(MT - 1);
          if constexpr (MT > 1) add(MT - 2);
          add(MT - 1);
        } else if constexpr (MT > 1) {
          add(MT - 2);
        }
        }
        nslot = wrap(nslot + tstep);
#pragma unroll
        for (int i = 0; i < MT; ++i) taddr[i] = wrap(taddr[i] + tstep);
      }
    }
  }
  };
  pass(std::false_type{});
  {
    int* const redo = (int*)ys;  // set if a sum of this workgroup's is not finite
    __syncthreads();  // the last step is consumed
    if (tid == 0) *redo = 0;
    __syncthreads();
    float seen = 0.f;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) seen = note_not_finite(acc[i][j][e], seen);
    if (any_not_finite(seen)) *redo = 1;
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(*redo)) pass(std::true_type{});  // (uniform, rare)
  }
  float* const slot = partial + (size_t)bz * a.slot;
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int r = (first + i) * 16 + 4 * lg;  // four rows of one tap
    const int tap = r / a.cc, c = ci0 + r - tap * a.cc;
    if (i < ntw && r < rows && c < a.ci) {
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const int ch = co0 + 16 * j + ls;
        if (ch < a.co) {
#pragma unroll
          for (int e = 0; e < 4; ++e) slot[((size_t)(t0 * T + tap) * a.ci + c + e) * a.co + ch] = acc[i][j][e];
        }
      }
    }
  }
  if (bias_wg) {  // each column's positions of a row, in order
    float* const red = (float*)smem;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NY; ++i) {
      const int u = i * TH + tid;
      if (u < NT * 128)
#pragma unroll
        for (int j = 0; j < 4; ++j) red[u / (4 * NT) * (16 * NT) + u % (4 * NT) * 4 + j] = btotal[i][j] + bsum[i][j];
    }
    __syncthreads();
    if (tid < 16 * NT && co0 + tid < a.co) {
      float sum[4] = {0.f, 0.f, 0.f, 0.f};
      for (int pos = 0; pos < 32; pos += 4)
#pragma unroll
        for (int q = 0; q < 4; ++q) sum[q] += red[(pos + q) * (16 * NT) + tid];
      slot[(size_t)a.k[0] * T * a.ci * a.co + co0 + tid] = (sum[0] + sum[1]) + (sum[2] + sum[3]);
    }
  }
}

struct Shape {
  Args a;
  int nw, mt, nt, lds;
  double us;  // estimated time
  bool ok;
};

// Everything that follows from the columns of a step: as few channel chunks as fit (tiles, LDS, pieces).
bool layout_of(Shape& s, int lc) {
  Args& a = s.a;
  const int T = a.k[1] * a.k[2], cols = 1 << lc;
  a.lc = lc;
  a.r = 32 >> lc;
  a.ring = a.span + (2 * a.r - 1) * a.s[1];
  a.ncell = (cols - 1) * a.s[2] + (a.k[2] - 1) * a.dil[2] + 1;
  a.half = (a.ncell + a.s[2] - 1) / a.s[2];
  a.cells = a.half * a.s[2];
  for (a.nci = 1; a.nci <= a.ci / 4; ++a.nci) {
    a.cc = (int32_t)(((a.ci + a.nci - 1) / a.nci + 3) / 4 * 4);
    a.tiles = (T * a.cc + 15) / 16;
    if (a.tiles > max_tiles(s.nt)) continue;
    a.gw = a.cc % 16 == 0 ? 16 : a.cc;
    s.nw = a.tiles > (s.nt == 4 ? 12 : 16) ? 8 : 4;
    const int64_t ring = (int64_t)a.ring * a.cells * a.cc * 6;
    if (ring + 16 + s.nt * 6144 > kLds) continue;
    if ((int64_t)a.r * a.s[1] * a.ncell * (a.cc / 4) > (int64_t)kNx * 64 * s.nw) continue;
    s.lds = std::max((int)((ring + 15) / 16 * 16) + s.nt * 6144, s.nt * 2048);
    a.nci = (a.ci + a.cc - 1) / a.cc;
    const int mt = (a.tiles + s.nw - 1) / s.nw;
    s.mt = s.nw == 4 ? mt : mt <= 3 ? 3 : mt <= 5 ? 5 : 7;
    return true;
  }
  return false;
}

bool find_shape(const distdl_plan* p, Shape& s) {
  if (p->explicit_halo || p->dtype != DISTDL_F32 || p->n_ci % 4 || p->n_co % 4) return false;
  if ((double)p->n_b * p->max_buf_cells * p->n_ci * 4.0 >= 2147480000.0 ||
      (double)p->n_b * p->max_out_cells * p->n_co * 4.0 >= 2147480000.0)
    return false;
  Args& a = s.a;
  a = Args{};
  a.n_b = (int32_t)p->n_b;
  a.ci = (int32_t)p->n_ci;
  a.co = (int32_t)p->n_co;
  for (int d = 0; d < 3; ++d) {
    a.k[d] = p->ksize[d];
    a.s[d] = p->stride[d];
    a.dil[d] = p->dilation[d];
  }
  const int T = a.k[1] * a.k[2];
  a.span = (a.k[1] - 1) * a.dil[1] + 1;
  if (a.s[1] > a.span) return false;
  a.slot = (int64_t)a.k[0] * T * a.ci * a.co + a.co;
  const int cols16 = (a.co + 15) / 16;
  int64_t o1 = 1, o2 = 1, planes = 0;
  for (const WorkerDev& wd : p->workers) {
    planes = std::max<int64_t>(planes, p->n_b * wd.out[0]);
    o1 = std::max<int64_t>(o1, wd.out[1]);
    o2 = std::max<int64_t>(o2, wd.out[2]);
  }
  // The shape of a step, chunks, and rows per unit: rounds of workgroups that the chip holds at once, times what one
  // takes (clocks): its steps, the start of each unit, its set-up and its partial's way to memory and back.
  const Shape base = s;
  double best = 1e300;
  for (int q = 0; q < 6; ++q) {  // columns of a step; whole blocks of up to four columns, or half of that
    const int lc = 5 - q / 2;
    Shape t = base;
    t.a.ncob = (cols16 + 3) / 4 * (1 + q % 2);
    if (t.a.ncob > cols16) continue;
    t.nt = (cols16 + t.a.ncob - 1) / t.a.ncob;
    if (lc < 5 && (32 >> lc) > 2 * o1) continue;
    if (!layout_of(t, lc)) continue;
    const Args& b = t.a;
    const int64_t nseg = (o2 + (1 << lc) - 1) >> lc, blocks = (int64_t)b.k[0] * b.nci * b.ncob * p->n_workers;
    if ((int64_t)b.nci * b.ncob > 65535) continue;
    const int resident = t.nw == 8 ? 1 : std::min(2, kLds / t.lds);
    const double step = std::max(1200.0, (double)((b.tiles + 3) / 4) * t.nt * 96.0 * 1.3 * resident);
    const double part = (double)blocks * b.tiles * 16 * t.nt * 16 * 8.0 / 2000.0;  // written and read, about 2 KB a clock
    const double start = 3000.0 + 700.0 * ((b.span - b.s[1]) * b.ncell * (b.cc / 4) / (4 * 64 * t.nw));
    for (int64_t nb1 = 1; nb1 <= std::max<int64_t>(1, o1 / 2); nb1 += std::max<int64_t>(1, nb1 / 4)) {
      const int64_t ob = ((o1 + nb1 - 1) / nb1 + b.r - 1) / b.r * b.r, units = planes * ((o1 + ob - 1) / ob);
      const double unit = (double)nseg * (ob / b.r * step + start);
      for (int64_t c = 1; c <= std::min<int64_t>(units, 512) && c * p->n_workers <= 65535; ++c) {
        const int64_t per = (units + c - 1) / c;
        if (c > 1 && (units + per - 1) / per != c) continue;  // an empty chunk
        const int64_t rounds = (blocks * c + 256 * resident - 1) / (256 * resident);
        const double cost = rounds * (per * unit + 8000.0) + part * c;
        if (cost < best * 0.99) best = cost, s = t, s.a.nchunks = (int32_t)c, s.a.ob = (int32_t)ob;
      }
    }
  }
  s.us = best / 2100.0;  // clocks in a microsecond under load
  return best < 1e300;
}

const Shape& shape_of(const distdl_plan* p) {
  static std::mutex lock;  // a workspace may be asked for from any thread
  std::lock_guard<std::mutex> hold(lock);
  if (!p->wgrad_split_plan) {
    auto s = std::make_shared<Shape>();
    s->ok = find_shape(p, *s);
    if (!s->ok) s->us = 1e300;
    p->wgrad_split_plan = s;
  }
  return *(const Shape*)p->wgrad_split_plan.get();
}

template <int NW, int MT, int NT>
int launch(distdl_plan* p, const Shape& s, float* partial, hipStream_t st) {
  if (s.lds > 64 * 1024)
    if (int rc = allow_large_lds<wgrad_split_kernel<NW, MT, NT>>()) return rc;
  const dim3 grid((unsigned)s.a.k[0], (unsigned)(s.a.nci * s.a.ncob), (unsigned)(p->n_workers * s.a.nchunks));
  hipLaunchKernelGGL((wgrad_split_kernel<NW, MT, NT>), grid, dim3(64 * NW), s.lds, st, p->d_workers, p->tab_x.dev, p->tab_dy.dev,
                     partial, s.a);
  return DISTDL_OK;
}
template <int NW, int MT>
int launch_nt(distdl_plan* p, const Shape& s, float* partial, hipStream_t st) {
  switch (s.nt) {
    case 1: return launch<NW, MT, 1>(p, s, partial, st);
    case 2: return launch<NW, MT, 2>(p, s, partial, st);
    case 3: return launch<NW, MT, 3>(p, s, partial, st);
    default: return launch<NW, MT, 4>(p, s, partial, st);
  }
}

}  // namespace

bool wgrad_split_supported(const distdl_plan* p) { return shape_of(p).ok; }

int wgrad_split_chunks(const distdl_plan* p) { return shape_of(p).ok ? shape_of(p).a.nchunks : 0; }

double wgrad_split_us(const distdl_plan* p) { return shape_of(p).us; }

int conv_wgrad_split(distdl_plan* p, float* partial, hipStream_t st) {
  const Shape& s = shape_of(p);
  if (!s.ok) return set_error(DISTDL_ERR_UNSUPPORTED, "conv: weight gradient shape");
  ProfScope prof("conv_bwd_weight_split", st);
  if (s.nw == 4) {
    if (s.mt == 1) return launch_nt<4, 1>(p, s, partial, st);
    if (s.mt == 2) return launch_nt<4, 2>(p, s, partial, st);
    if (s.mt == 3) return launch_nt<4, 3>(p, s, partial, st);
    if (s.nt == 1) return launch<4, 4, 1>(p, s, partial, st);
    if (s.nt == 2) return launch<4, 4, 2>(p, s, partial, st);
    return launch<4, 4, 3>(p, s, partial, st);
  }
  if (s.mt == 3) return launch_nt<8, 3>(p, s, partial, st);
  if (s.mt == 5 && s.nt == 1) return launch<8, 5, 1>(p, s, partial, st);
  if (s.mt == 5 && s.nt == 2) return launch<8, 5, 2>(p, s, partial, st);
  if (s.mt == 5) return launch<8, 5, 3>(p, s, partial, st);
  return s.nt == 1 ? launch<8, 7, 1>(p, s, partial, st) : launch<8, 7, 2>(p, s, partial, st);
}

}  // namespace distdl
