"""The scratch array of vector_route_static is as large as the header and vector_route_static_scratch_bytes() say, and shapes
whose routing needs more than that (heads are independent: they go a group at a time) get what vector_route gives."""
import os
import subprocess

import pytest

torch = pytest.importorskip("torch")

from paper_2605_23258_amd import binding as vb
from paper_2605_23258_amd import build
from test_zz_no_alloc import _route_both

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.mark.skipif(not (os.path.exists(build.HIPCC) and os.path.exists(READELF)), reason="needs the ROCm toolchain")
def test_the_device_array_has_the_reported_size(tmp_path):
    obj = str(tmp_path / "route_static.o")
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "--no-gpu-bundle-output", "-c", os.path.join(build.CSRC, "route_static.hip"), "-o", obj],
                   check=True, capture_output=True)
    symbols = subprocess.run([READELF, "-sW", obj], check=True, capture_output=True, text=True).stdout.splitlines()
    sizes = {int(line.split()[2]) for line in symbols if " OBJECT " in line and "scratch" in line.split()[-1]}
    assert sizes == {vb.lib().vector_route_static_scratch_bytes()}


@pytest.mark.gpu
@pytest.mark.parametrize("heads,n,n_pool,n_approx", [
    (10, 131072, 9000, 4000),            # 16 MiB and a little: two groups of five
    (13, 131072, 20000, 0),              # seven heads, then six
    (1, 1 << 20, 5000, 2000), (2, 950000, 3000, 3000),          # one head fills most of the array
    (11, 131072, 0, 0),
    (80, 16384, 2000, 900)])             # heads that need no scratch go at once
def test_more_heads_than_the_array_holds_at_once(heads, n, n_pool, n_approx):
    _route_both(heads, n, n_pool, n_approx, seed=heads)
