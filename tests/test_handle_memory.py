"""What a differentiable handle allocates, on a stand-in for the HIP runtime (no GPU):
the segment buffers past the fourth are optional, and never take what the handle cannot
do without, or more than a small share of the memory that is left."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = "/opt/rocm"
N, K, H = 20000, 16, 160      # ten segments; overlap off, so up to eight buffers
RB = (N + 63) // 64 * 64
RECORD = (K * 171 + (32 + K) * 4) * RB * 4


@pytest.fixture(scope="module")
def create(tmp_path_factory):
    if not (shutil.which("g++") and os.path.exists(f"{ROCM}/include/hip/hip_runtime_api.h")):
        pytest.skip("needs g++ and the HIP headers")
    from paper_2311_13081_amd import _lib
    d = tmp_path_factory.mktemp("fake_hip")
    src, shim, exe = os.path.join(HERE, "fake_hip.cpp"), str(d / "shim.so"), str(d / "driver")
    cc = ["g++", "-std=c++17", "-w"]
    subprocess.check_call(cc + ["-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", "-shared", "-fPIC", src,
                                "-o", shim])
    subprocess.check_call(cc + ["-DFAKE_HIP_DRIVER", f"-I{ROOT}/include", src, "-o", exe, "-ldl"])

    def run(**env):
        e = dict(os.environ, LD_PRELOAD=shim, LD_LIBRARY_PATH=f"{ROCM}/lib", **env)
        out = subprocess.run([exe, _lib.LIB_PATH, str(N), str(K), str(H)], env=e, text=True,
                             capture_output=True, timeout=60)
        assert out.returncode == 0, out.stdout + out.stderr
        lines = [x.split() for x in out.stdout.splitlines()]
        return (int(next(x[1] for x in lines if x[0] == "rc")),
                [int(x[1]) for x in lines if x[0] == "malloc"])

    return run


def test_optional_buffers_with_memory_to_spare(create):
    rc, sizes = create()
    assert rc == 0 and sizes.count(RECORD) == 8


def test_optional_buffers_do_not_take_required_memory(create):
    rc, least = create(FAKE_HIP_FREE="0")  # nothing to spare: none of them
    assert rc == 0 and least.count(RECORD) == 4
    need = sum(least)
    # any amount that is enough for the handle without them: it is created
    for extra in (0, RECORD, 2 * RECORD, 3 * RECORD, 5 * RECORD):
        rc, sizes = create(FAKE_HIP_BYTES=str(need + extra))
        assert rc == 0, extra
        assert sizes.count(RECORD) >= 4


def test_optional_buffers_leave_memory_to_the_caller(create):
    _, least = create(FAKE_HIP_FREE="0")
    for free in (RECORD * 4, RECORD * 40, RECORD * 120):
        rc, sizes = create(FAKE_HIP_BYTES=str(sum(least) + free))
        taken = sum(sizes) - sum(least)
        assert rc == 0 and taken <= free / 4, (free, taken)
