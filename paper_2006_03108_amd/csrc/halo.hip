// Halo exchange H and adjoint H* (Sec. 3 "Halo exchange") as one-pass box
// kernels over all workers, dimensions, faces, edges and corners.
//
// The nested per-dimension exchange of the paper leaves every in-domain
// non-owned cell equal to its owner's bulk value; since all partitions share
// one address space that end state is written directly: each box of halo
// cells is one strided copy from the owner's buffer (pack + exchange + unpack
// collapsed, exchange buffers never materialised), each box of padding cells
// a zero fill.  The adjoint runs in gather form: the thread that owns a bulk
// cell reads every halo copy of it (fixed ascending worker order), adds them
// and clears them -- the "add into the bulk" of C* = K_b S_{b->a} without
// atomics, so results are run-to-run identical.
#include "common.h"
#include "halo_box.h"
#include "profile.h"
#include "weight_job.h"

namespace distdl {

extern const int kHaloUnitsPerBlock = 1024;  // 256 threads x 4 vector units

template <class E, bool JOB>
__global__ __launch_bounds__(kThreads) void halo_fwd_kernel(const BlockRef* __restrict__ blocks,
                                                            const HaloTaskDev* __restrict__ tasks,
                                                            void* const* __restrict__ bufs, JobArg<JOB> job) {
  using S = typename E::Store;
  if constexpr (JOB) {
    if ((int)blockIdx.x >= job.at) return run_weight_job(job, (int)blockIdx.x - job.at);
  }
  halo_fwd_box<E>(blocks, tasks, bufs, (int)blockIdx.x);
}

// Adjoint: bulk boxes gather-add their halo copies and clear them; padding
// boxes are cleared.  Per source, the loads of all kUnroll units are issued
// before the clears, and the destination is loaded together with the first
// source, so that a thread has 2 * kUnroll requests in flight.
template <class E>
__global__ __launch_bounds__(kThreads) void halo_adj_kernel(const BlockRef* __restrict__ blocks,
                                                            const HaloTaskDev* __restrict__ tasks,
                                                            const HaloView* __restrict__ views,
                                                            void* const* __restrict__ bufs) {
  using S = typename E::Store;
  const BlockRef br = blocks[blockIdx.x];
  const HaloTaskDev t = tasks[br.task];  // by value: the record is read once into scalar registers
  const uint32_t total = t.total;
  S* dst = (S*)bufs[t.dst.worker];
  if (t.nsrc == 0) {
#pragma unroll
    for (int i = 0; i < kUnroll; ++i) {
      uint32_t u = br.unit0 + threadIdx.x + i * kThreads;
      if (u < total) nt_store(dst + view_offset(t.dst, decode(u, t)), E::zero());
    }
    return;
  }
  UnitPos pos[kUnroll];
  bool live[kUnroll];
  S dv[kUnroll], sv[kUnroll];
  float acc[kUnroll][E::N];
  S* src = (S*)bufs[t.src0.worker];
#pragma unroll
  for (int i = 0; i < kUnroll; ++i) {
    uint32_t u = br.unit0 + threadIdx.x + i * kThreads;
    live[i] = u < total;
    pos[i] = decode(live[i] ? u : total - 1, t);  // clamped: loads need no branch
    dv[i] = nt_load(dst + view_offset(t.dst, pos[i]));
    sv[i] = nt_load(src + view_offset(t.src0, pos[i]));
  }
#pragma unroll
  for (int i = 0; i < kUnroll; ++i) {
    float v[E::N];
    E::unpack(dv[i], acc[i]);
    E::unpack(sv[i], v);
    if (live[i]) nt_store(src + view_offset(t.src0, pos[i]), E::zero());
#pragma unroll
    for (int e = 0; e < E::N; ++e) acc[i][e] += v[e];
  }
  for (int s = 1; s < t.nsrc; ++s) {  // ascending source-worker order
    const HaloView sr = views[t.src_begin + s];
    src = (S*)bufs[sr.worker];
#pragma unroll
    for (int i = 0; i < kUnroll; ++i) sv[i] = nt_load(src + view_offset(sr, pos[i]));
#pragma unroll
    for (int i = 0; i < kUnroll; ++i) {
      float v[E::N];
      E::unpack(sv[i], v);
      if (live[i]) nt_store(src + view_offset(sr, pos[i]), E::zero());
#pragma unroll
      for (int e = 0; e < E::N; ++e) acc[i][e] += v[e];
    }
  }
#pragma unroll
  for (int i = 0; i < kUnroll; ++i)
    if (live[i]) plain_store(dst + view_offset(t.dst, pos[i]), E::pack(acc[i]));
}

int plan_prepare_device(distdl_plan* p);

__global__ __launch_bounds__(kThreads) void weight_job_kernel(WeightJob job) {
  run_weight_job(job, (int)(blockIdx.y * gridDim.x + blockIdx.x));
}

int launch_weight_job(const WeightJob& job, hipStream_t st) {
  if (job.kind == 0) return DISTDL_OK;
  ProfScope prof("conv_relayout_w", st);
  // (a class a row: 64 of them may have more blocks than a launch has along one dimension)
  hipLaunchKernelGGL(weight_job_kernel, dim3((unsigned)job.per_class, (unsigned)(job.blocks / job.per_class)), dim3(kThreads), 0, st, job);
  DISTDL_HIP_TRY(hipGetLastError());
  return DISTDL_OK;
}

template <class E>
static void launch(bool adjoint, const TaskTable& tt, void* const* bufs, WeightJob* job, hipStream_t st) {
  dim3 grid((unsigned)tt.blocks.size()), block(kThreads);
  ProfScope prof(adjoint ? "halo_adj" : "halo_fwd", st);
  if (adjoint) {
    hipLaunchKernelGGL(halo_adj_kernel<E>, grid, block, 0, st, tt.d_blocks, tt.d_tasks, tt.d_views, bufs);
  } else if (job && job->kind != 0 && (int64_t)grid.x + job->blocks < kMaxBlocks256) {
    job->at = (int32_t)grid.x;
    grid.x += (unsigned)job->blocks;
    hipLaunchKernelGGL((halo_fwd_kernel<E, true>), grid, block, 0, st, tt.d_blocks, tt.d_tasks, bufs, *job);
    job->kind = 0;
  } else {
    hipLaunchKernelGGL((halo_fwd_kernel<E, false>), grid, block, 0, st, tt.d_blocks, tt.d_tasks, bufs, NoJob{});
  }
}

// Copy boxes between arbitrary buffers with the forward kernel (used by the generalized repartition): the
// tasks' views index one pointer table that holds sources and destinations; unit_bytes is 16, 4 or 2.
int run_box_copy(int unit_bytes, const BlockRef* d_blocks, const HaloTaskDev* d_tasks, size_t nblocks, void* const* d_bufs,
                 const char* name, hipStream_t st) {
  if (nblocks == 0) return DISTDL_OK;
  dim3 grid((unsigned)nblocks), block(kThreads);
  ProfScope prof(name, st);
  if (unit_bytes == 16) hipLaunchKernelGGL((halo_fwd_kernel<F32x4, false>), grid, block, 0, st, d_blocks, d_tasks, d_bufs, NoJob{});
  else if (unit_bytes == 4) hipLaunchKernelGGL((halo_fwd_kernel<F32x1, false>), grid, block, 0, st, d_blocks, d_tasks, d_bufs, NoJob{});
  else if (unit_bytes == 2) hipLaunchKernelGGL((halo_fwd_kernel<BF16x1, false>), grid, block, 0, st, d_blocks, d_tasks, d_bufs, NoJob{});
  else return set_error(DISTDL_ERR_INVALID_ARG, "internal: box copy unit of %d bytes", unit_bytes);
  DISTDL_HIP_TRY(hipGetLastError());
  return DISTDL_OK;
}

// Shared by the public halo calls and by conv_fwd / conv_bwd.
int run_halo(distdl_plan* p, bool adjoint, PtrTable& tab, void* const* bufs_host, hipStream_t st) {
  return run_halo_with(p, adjoint, tab, bufs_host, nullptr, st);
}
int run_halo_with(distdl_plan* p, bool adjoint, PtrTable& tab, void* const* bufs_host, WeightJob* job, hipStream_t st) {
  int rc = plan_prepare_device(p);
  if (rc) return rc;
  const size_t esz = dtype_size(p->dtype);
  bool aligned16 = true;
  for (int w = 0; w < p->n_workers; ++w) {
    if (!bufs_host[w]) return set_error(DISTDL_ERR_NULL, "buffer of worker %d is null", w);
    if ((uintptr_t)bufs_host[w] % esz) return set_error(DISTDL_ERR_INVALID_ARG, "buffer of worker %d is misaligned", w);
    aligned16 &= ((uintptr_t)bufs_host[w] % 16) == 0;
  }
  const bool wide = aligned16 && !p->fwd16.tasks.empty();
  const TaskTable& tt = adjoint ? (wide ? p->adj16 : p->adj1) : (wide ? p->fwd16 : p->fwd1);
  if (tt.blocks.empty()) return DISTDL_OK;  // a single worker with no padding: H is the identity
  if ((rc = tab.upload((const void* const*)bufs_host, p->n_workers, st))) return rc;
  if (p->dtype == DISTDL_F32) {
    if (wide) launch<F32x4>(adjoint, tt, tab.dev, job, st);
    else launch<F32x1>(adjoint, tt, tab.dev, job, st);
  } else {
    if (wide) launch<BF16x8>(adjoint, tt, tab.dev, job, st);
    else launch<BF16x1>(adjoint, tt, tab.dev, job, st);
  }
  DISTDL_HIP_TRY(hipGetLastError());
  return DISTDL_OK;
}

}  // namespace distdl

using namespace distdl;

extern "C" {

int distdl_halo_fwd(distdl_plan* plan, void* const bufs_dev[], void* stream) {
  if (!plan || !bufs_dev) return set_error(DISTDL_ERR_NULL, "halo_fwd: null argument");
  return run_halo(plan, false, plan->tab_x, bufs_dev, (hipStream_t)stream);
}

int distdl_halo_adj(distdl_plan* plan, void* const gbufs_dev[], void* stream) {
  if (!plan || !gbufs_dev) return set_error(DISTDL_ERR_NULL, "halo_adj: null argument");
  return run_halo(plan, true, plan->tab_dx, gbufs_dev, (hipStream_t)stream);
}

}  // extern "C"
