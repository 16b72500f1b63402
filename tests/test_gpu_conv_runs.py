"""Convolutions on the gather kernel whose channel count is no multiple of 4, or whose arrays are not aligned: k in octets of the
channels of neighbouring taps, which lie one behind the other in memory."""
import pytest
import torch

import paper_2006_03108_amd as dd
from tests.gpu_util import ConvLayer, require_gpu

pytestmark = pytest.mark.gpu

# n_b, c_in, c_out, shape, kernel, stride, dilation, offset: runs of whole octets and with 1 ... 7 more; of one tap (dilation, or the data
# gradient) and of several; k beyond the last octet; tiles of 64 rows and of 256 with one and two column tiles; classes without taps
RUNS = [
    (2, 17, 11, (67,), 3, 1, 1, 0), (3, 3, 33, (40, 41), 7, 2, 1, 0), (1, 13, 70, (9, 10, 11), 3, 1, (1, 1, 2), 0),
    (2, 20, 24, (33, 30), 2, 1, 1, 1), (5, 25, 41, (40, 41), 3, 1, 1, 0), (64, 9, 42, (50, 50), 3, 1, 1, 0), (70, 27, 14, (48, 48), 3, 1, 1, 0),
    (2, 18, 22, (9, 10, 11), (3, 1, 2), 2, (2, 1, 2), 0), (1, 31, 9, (300,), 1, 1, 1, 0), (2, 50, 50, (20, 20), (1, 5), (1, 3), 1, 3),
    (2, 20, 36, (33, 30), 3, 1, 1, 0),  # (bf16)
]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layer", RUNS, ids=lambda c: f"c{c[1]}-{c[2]}k{c[4]}s{c[5]}d{c[6]}x{c[3][-1]}o{c[7]}".replace(" ", ""))
def test_runs_against_fp64(layer, dtype):
    """A sum of K <= 400 split products is off by at most K / 16 + 2 roundings of 2^-24 of its running sum, about sqrt of that many as a
    random walk: 1e-6 in the 2-norm is four times as much.  bf16: 2^-8 for the result's rounding.  With an infinity in x and in dy, what does not read it stays finite."""
    require_gpu()
    n_b, c_in, c_out, shape, k, s, dil, offset = layer
    L, tol = ConvLayer(n_b, c_in, c_out, shape, k, s, dtype, dil=dil, offset=offset), 1e-6 if dtype == torch.float32 else 2.0 ** -8
    kernels = dd.distdl_debug_conv_kernels(L.plan, offset == 0)
    if c_in % 4 or offset or dtype == torch.bfloat16:
        assert kernels[0] == 4 and kernels[1] == 4

    def run():
        dd.distdl_conv_local_fwd(L.plan, [L.x], L.w, None, [L.y])
        dd.distdl_conv_local_bwd(L.plan, [L.x], L.w, [L.dy], [L.dx], L.dw, L.db, L.ws)
        return L.y, L.dx[L.bulk]

    for got, want in zip(run(), L.exact()):
        assert float((got.double() - want).norm()) <= tol * float(want.norm())
    middle = tuple(n // 2 for n in L.x.shape[1:-1])
    L.x[(0, *middle, c_in - 1)] = float("inf")
    L.dy[(0, *[n // 2 for n in L.dy.shape[1:-1]], 0)] = float("-inf")
    for got, want in zip(run(), L.exact()):
        sure = torch.isfinite(want)
        assert torch.equal(torch.isfinite(got), sure)
        assert float((got[sure].double() - want[sure]).norm()) <= tol * float(want[sure].norm())
