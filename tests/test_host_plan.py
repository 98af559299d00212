"""The planner and the executor's host side, checked by a C++ program linked
with the built library (tests/host/plan_host_check.cpp); no GPU is needed."""
import importlib.util
import os
import subprocess
from types import SimpleNamespace

import pytest

from paper_1505_01998_amd import build as b

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    if not os.path.exists(b.hipcc()) or not os.path.exists(b.LIB):
        pytest.skip("hipcc or library missing")
    d = tmp_path_factory.mktemp("plan")
    obj, exe = str(d / "check.o"), str(d / "check")
    # no device code: the host half alone
    subprocess.run([b.hipcc(), "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-w",
                    "-I", os.path.join(b.ROOT, "include"), "-I", b.CSRC, "-c", "-o", obj,
                    os.path.join(HERE, "host", "plan_host_check.cpp")], check=True)
    subprocess.run([b.hipcc(), "--offload-arch=gfx950", "-o", exe, obj, b.LIB,
                    "-Wl,-rpath," + os.path.dirname(b.LIB)], check=True)
    return exe


def test_planner_host_checks(check):
    r = subprocess.run([check], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip() == "OK"


def test_bench_names_the_kernel_that_runs(check):
    spec = importlib.util.spec_from_file_location("bench_names", os.path.join(b.ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    r = subprocess.run([check, "launch_evals"], capture_output=True, text=True, timeout=120, check=True)
    assert bench.LAUNCH_EVALS == float(r.stdout)
    args = SimpleNamespace(precision="mixed", prune=-1, autotune=1, mfma=-1, hc=-1, tj=-1, persistent=-1)
    ctx = SimpleNamespace(autotune=lambda n, n_h: ((32, 512), {}, {}))
    assert bench._lscv_kernel(ctx, args, 1_000_000, 512) == "k_lscv_units_f32_queue<32, 512>"
    assert bench._lscv_kernel(ctx, args, 20_000, 128) == "k_lscv_units_f32<16>"
    assert bench._lscv_kernel(ctx, args, 20_000, 128, 5e12) == "k_lscv_units_f32_queue<32, 512>"
    args.autotune = -1
    assert bench._lscv_kernel(ctx, args, 1_000_000, 512) == "k_lscv_units_f32_queue<16, 512>"
    args.persistent = 0
    assert bench._lscv_kernel(ctx, args, 1_000_000, 512) == "k_lscv_units_f32<16>"
