"""The host side of lagom_overlap_run on a model of the runtime (tests/runner_host.cpp): what is queued when, and what is left behind a failure."""
import json
import os
import shutil
import subprocess

import pytest

from paper_2602_20656_amd import binding as lg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_2602_20656_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def runner(tmp_path_factory):
    lg.lib()                       # built
    exe = str(tmp_path_factory.mktemp("runner") / "runner_host")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROCM, "include"),
                           os.path.join(ROOT, "tests", "runner_host.cpp"), lg.LIB_PATH, "-Wl,-rpath," + PACKAGE, "-Wl,--allow-shlib-undefined", "-o", exe])
    def run(fail=0, comm_us=1.0, comp_us=1.0, warmup=0, iters=1, mode=lg.LAGOM_CORUN):
        r = subprocess.run([exe, *map(str, (fail, comm_us, comp_us, warmup, iters, mode))], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stdout + r.stderr
        return json.loads(r.stdout)
    return run


@pytest.mark.parametrize("mode", [lg.LAGOM_CORUN, lg.LAGOM_ALONE_COMM, lg.LAGOM_ALONE_COMP])
def test_a_failed_read_out_leaves_nothing_in_flight(runner, mode):
    """Whatever is queued when a time cannot be read has ended before its events go and the call returns."""
    reads = runner(warmup=1, iters=3, mode=mode)["reads"]
    for fail in range(1, reads + 1):
        r = runner(fail=fail, warmup=1, iters=3, mode=mode)
        assert r["rc"] == lg.LAGOM_EHIP and "made to fail" in r["error"]
        assert r["destroyed_in_flight"] == 0 and r["in_flight"] == 0 and r["alive"] == 0, (fail, r)


@pytest.mark.parametrize("comm_us,comp_us", [(100.0, 3.0), (3.0, 100.0), (50.0, 40.0)])
@pytest.mark.parametrize("warmup,iters", [(0, 1), (1, 1), (2, 4)])
@pytest.mark.parametrize("mode", [lg.LAGOM_CORUN, lg.LAGOM_ALONE_COMM, lg.LAGOM_ALONE_COMP])
def test_repetitions_do_not_reach_into_each_other(runner, comm_us, comp_us, warmup, iters, mode):
    """A repetition begins when the one before has ended on both streams, however much longer one of them takes, and is not queued before: streams that
    wait for each other on the device are released 1.7 us apart."""
    r = runner(comm_us=comm_us, comp_us=comp_us, warmup=warmup, iters=iters, mode=mode)
    comm, comp = mode != lg.LAGOM_ALONE_COMP, mode != lg.LAGOM_ALONE_COMM
    assert r["rc"] == lg.LAGOM_OK and r["early"] == 0 and r["ahead"] == 0 and r["in_flight"] == 0 and r["alive"] == 0
    assert (r["comms"], r["comps"]) == ((warmup + iters) * comm, (warmup + iters) * comp)
    assert (r["X"], r["Y"], r["Z"]) == pytest.approx((comm_us * comm, comp_us * comp, max(comm_us * comm, comp_us * comp)), abs=0.01)
