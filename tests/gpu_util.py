"""Helpers for the GPU parity tests: layout marshalling between the oracle's
logical [n_b, n_c, spatial...] numpy arrays and the library's channels-last
device buffers, and the parity norms."""
import itertools

import numpy as np
import torch

import paper_2006_03108_amd as dd
from oracle import geometry as geo


def require_gpu():
    assert torch.cuda.is_available(), "GPU tests need a HIP device (run them with -m gpu on the GPU box)"
    return torch.device("cuda:0")


def to_cl(arr, dtype=torch.float32):
    """numpy [n, c, s...] -> contiguous device tensor [n, s..., c]."""
    t = torch.from_numpy(np.ascontiguousarray(np.moveaxis(arr, 1, -1)))
    return t.to(dtype).cuda().contiguous()


def from_cl(t):
    """device tensor [n, s..., c] -> numpy [n, c, s...] (float64 for parity math)."""
    return np.moveaxis(t.detach().to(torch.float32).cpu().numpy(), -1, 1)


def w_to_dev(w):
    return torch.from_numpy(np.ascontiguousarray(w)).float().cuda()


def oracle_partition(cfg):
    return geo.Partition.for_kernel(cfg["in_shape"], cfg["P"], cfg["ksize"], cfg["stride"], cfg["padding"],
                                    cfg["dilation"])


def rel_errors(got, want):
    got = np.asarray(got, dtype=np.float64)
    want = np.asarray(want, dtype=np.float64)
    l2 = np.linalg.norm((got - want).ravel()) / max(np.linalg.norm(want.ravel()), 1e-300)
    mx = np.abs(got - want).max() / max(np.abs(want).max(), 1e-300)
    return l2, mx


def assert_close(got, want, tol, what=""):
    l2, mx = rel_errors(got, want)
    assert l2 <= tol and mx <= tol, f"{what}: rel l2 {l2:.3e}, rel max {mx:.3e} > {tol:.1e}"


def split_forms(plan):
    """Forward and data gradient of aligned tensors: (cells to a position, products that two taps share) where the split kernels
    run, else None."""
    kernels = dd.distdl_debug_conv_kernels(plan)
    forms = [dd.distdl_debug_conv_split(plan, backward) for backward in (False, True)]
    return tuple((f[1], f[3]) if k == 3 else None for k, f in zip(kernels, forms))


class ConvLayer:
    """A convolution layer on one worker, its tensors padded and channels-last, N(0, 1) values; exact() gives the same in
    fp64 on the device, tap by tap.  offset: the tensors start that many elements into an allocation."""

    def __init__(self, n_b, c_in, c_out, shape, k, s, dtype=torch.float32, p=None, dil=None, offset=0, seed=11):
        g = torch.Generator(device="cuda").manual_seed(seed)
        D = len(shape)
        each = lambda v: list(v) if isinstance(v, (list, tuple)) else [v] * D
        self.k, self.s, self.D, self.aligned = each(k), each(s), D, offset == 0
        self.dil = each(1 if dil is None else dil)
        p = [v // 2 for v in self.k] if p is None else each(p)

        def new(*sizes, random=True):
            n = int(np.prod(sizes))
            flat = torch.zeros(n + offset, device="cuda", dtype=dtype)
            if random:
                flat.copy_(torch.randn(n + offset, generator=g, device="cuda"))
            return flat[offset:].view(sizes)

        self.plan = dd.distdl_plan_create(D, n_b, c_in, c_out, shape, (1,) * D, self.k, self.s, p, self.dil, dtype)
        geo_ = self.plan.query(0)
        self.bulk = (slice(None), *(slice(a, a + n) for a, n in zip(geo_["bulk_off"], shape)))
        self.x = new(n_b, *geo_["buf_shape"][:D], c_in, random=False)
        self.x[self.bulk] = new(n_b, *shape, c_in)
        self.w, self.dy = new(c_out, c_in, *self.k), new(n_b, *geo_["out_size"][:D], c_out)
        self.y, self.dx, self.dw, self.db = (new(*t, random=False) for t in (self.dy.shape, self.x.shape, self.w.shape, (c_out,)))
        self.ws = torch.empty(max(dd.distdl_conv_bwd_workspace(self.plan), 16), dtype=torch.uint8, device="cuda")

    def run(self):
        """y, dx (of the owned cells), dw; db stays in self.db"""
        dd.distdl_conv_fwd(self.plan, [self.x], self.w, None, [self.y])
        dd.distdl_conv_bwd(self.plan, [self.x], self.w, [self.dy], [self.dx], self.dw, self.db, self.ws)
        return self.y, self.dx[self.bulk], self.dw

    def run_apart(self):
        """The same with the halo exchange in calls of its own: on the kernels that distdl_debug_conv_kernels names, whatever the size."""
        dd.distdl_halo_fwd(self.plan, [self.x])
        dd.distdl_conv_local_fwd(self.plan, [self.x], self.w, None, [self.y])
        dd.distdl_conv_local_bwd(self.plan, [self.x], self.w, [self.dy], [self.dx], self.dw, self.db, self.ws)
        dd.distdl_halo_adj(self.plan, [self.dx])
        return self.y, self.dx[self.bulk], self.dw

    def ways(self):
        """run, and run_apart where run takes a direction in one launch"""
        return [self.run] + [self.run_apart] * any(dd.distdl_debug_conv_fused(self.plan, self.aligned))

    def exact(self):
        x, w, dy = self.x.double(), self.w.double(), self.dy.double()
        y, dx, dw = torch.zeros_like(dy), torch.zeros_like(x), torch.zeros_like(w)
        rows = dy.reshape(-1, dy.shape[-1])
        for t in itertools.product(*[range(k) for k in self.k]):
            at = (slice(None), *(slice(i * d, i * d + (n - 1) * s + 1, s) for i, d, n, s in zip(t, self.dil, dy.shape[1:], self.s)))
            wt = w[(slice(None), slice(None), *t)]
            cells = x[at].reshape(-1, x.shape[-1])
            y += (cells @ wt.t()).view_as(dy)
            dx[at] += (rows @ wt).view_as(x[at])
            dw[(slice(None), slice(None), *t)] = rows.t() @ cells
        return y, dx[self.bulk], dw
