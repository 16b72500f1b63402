"""Host code of the library under a check of array bounds: its sources once more without their device code, every access beyond a
fixed array a trap.  A call is made up to its first HIP call, which fails without a device; pointers are numbers that nobody follows."""
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2006_03108_amd", "csrc")

AFFINE = """
import ctypes as C, sys
lib, ptr = C.CDLL(sys.argv[1]), C.c_void_p
P_fo, P_fi, dtype, first = map(int, sys.argv[2:])
plan = ptr()
assert lib.distdl_affine_plan_create(C.byref(plan), C.c_int64(5), C.c_int64(72), C.c_int64(63), P_fo, P_fi, dtype) == 0
some = lambda n: (ptr * n)(*[0x100000 * (i + 1) + first for i in range(n)])
x, W, f = some(P_fi), some(P_fo * P_fi), some(P_fo)
assert lib.distdl_affine_fwd(plan, x, W, f, f, None) != 0
assert lib.distdl_affine_bwd(plan, x, W, f, x, W, f, None) != 0
lib.distdl_affine_plan_destroy(plan)
"""


@pytest.fixture(scope="module")
def checked(tmp_path_factory):
    at = str(tmp_path_factory.mktemp("checked"))
    run = lambda cmd: subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True).stdout

    def one(name):
        obj = os.path.join(at, name + ".o")
        run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "-c", "-fPIC", "-O0", "-std=c++17", "--offload-arch=gfx950",
             "--offload-host-only", "-w", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-Xarch_host", "-fsanitize=array-bounds",
             "-Xarch_host", "-fsanitize-trap=array-bounds", os.path.join(CSRC, name), "-o", obj])
        return obj

    with ThreadPoolExecutor(8) as pool:
        objs = list(pool.map(one, sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))))
    images = sorted(set(re.findall(r"__hip_fatbin_[0-9a-f]+", run(["nm", *objs]))))
    with open(os.path.join(at, "none.c"), "w") as f:  # (in the place of the device code)
        f.write("".join(f"__attribute__((aligned(4096))) char {name}[64];\n" for name in images))
    lib = os.path.join(at, "libchecked.so")
    run(["gcc", "-c", "-fPIC", os.path.join(at, "none.c"), "-o", os.path.join(at, "none.o")])
    run(["g++", "-shared", "-o", lib, *objs, os.path.join(at, "none.o"), "-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib", "-lamdhip64"])
    return lib


@pytest.mark.parametrize("first", [0, 4], ids=["aligned", "odd"])
@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "bf16"])
@pytest.mark.parametrize("P_fo,P_fi", [(1, 8), (8, 1), (1, 9), (9, 1), (9, 9)])
def test_affine_layer_of_many_workers(checked, P_fo, P_fi, dtype, first):
    """A GEMM block has room for eight segments; a layer with more workers along its sum is not one for the estimates."""
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1")
    r = subprocess.run([sys.executable, "-c", AFFINE, checked, str(P_fo), str(P_fi), str(dtype), str(first)], env=env,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stdout[-500:])
