"""Which kernel lagom_comm_steps launches, on a model of the runtime (tests/steps_host.cpp): loads carry the non-temporal hint or not."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2602_20656_amd import binding as lg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_2602_20656_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
REDUCE, COPY = "%d:" % lg.LAGOM_REDUCE_COPY, "%d:" % lg.LAGOM_GATHER_COPY
MiB = 1 << 20


@pytest.fixture(scope="module")
def streamed(tmp_path_factory):
    lg.lib()                       # built
    exe = str(tmp_path_factory.mktemp("steps") / "steps_host")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROCM, "include"),
                           os.path.join(ROOT, "tests", "steps_host.cpp"), lg.LIB_PATH, "-Wl,-rpath," + PACKAGE, "-Wl,--allow-shlib-undefined", "-o", exe])
    def run(steps, dtype=lg.LAGOM_F32, nbytes=32 * MiB, nc=128, nt=256, chunk=65536):
        count = nbytes // (4 if dtype == lg.LAGOM_F32 else 2)
        r = subprocess.run([exe, *map(str, (dtype, count, nc, nt, chunk)), *steps], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stdout + r.stderr
        m = re.fullmatch(r"\S*comm_steps_kernelILi(\d)ELb(\d)ELb(\d)E\S* (\d+) (\d+)\n", r.stdout)
        assert m and (int(m[1]), int(m[4]), int(m[5])) == (dtype, nc, nt), r.stdout
        return m[2] == "1"
    return run


@pytest.mark.parametrize("dtype", [lg.LAGOM_F32, lg.LAGOM_BF16])
@pytest.mark.parametrize("steps,again", [
    ([REDUCE + "ab-e", REDUCE + "cd-f"], False),                        # nothing touched twice
    ([REDUCE + "ab-e", COPY + "c-e"], False),                           # a buffer that is written twice
    ([REDUCE + "aa-e", COPY + "c-f"], False),                           # twice by one step
    ([REDUCE + "ab-a", COPY + "c-f"], False),                           # read and written by one step
    ([REDUCE + "ab-e", REDUCE + "ad-f"], True),                         # a source read twice
    ([REDUCE + "ab-e", COPY + "e-f"], True),                            # a destination read by a later step
    ([REDUCE + "ab-e", COPY + "c-b"], True),                            # a source written by a later step
    ([REDUCE + "ab-ef", COPY + "c-gh", COPY + "h-i"], True)])           # the last pointer of a step in between
def test_steps_that_read_again_load_without_the_hint(streamed, steps, again, dtype):
    assert streamed(steps, dtype) == (not again)
    assert not streamed(steps, dtype, nc=64) and not streamed(steps, dtype, nbytes=127 * 65536)      # fewer than 128 channels have work


@pytest.mark.parametrize("nbytes,hint", [(224 * MiB - 16, False), (224 * MiB, True), (1 << 30, True)])
def test_buffers_that_fill_the_last_level_cache_are_streamed_all_the_same(streamed, nbytes, hint):
    assert streamed([REDUCE + "ab-e", REDUCE + "ad-f"], nbytes=nbytes) == hint
    assert streamed([REDUCE + "ab-e", REDUCE + "cd-f"], nbytes=nbytes)
