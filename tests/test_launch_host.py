"""Which kernels lagom_comm_steps and lagom_gemm launch, on a model of the runtime (tests/launch_host.cpp): loads with the non-temporal hint or without,
and the names that the benchmark gives."""
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
def launched(tmp_path_factory):
    lg.lib()                       # built
    exe = str(tmp_path_factory.mktemp("launch") / "launch_host")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROCM, "include"),
                           os.path.join(ROOT, "tests", "launch_host.cpp"), lg.LIB_PATH, "-Wl,-rpath," + PACKAGE, "-Wl,--allow-shlib-undefined", "-o", exe])
    def run(*args):
        r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stdout + r.stderr
        return r.stdout.splitlines()
    return run


@pytest.fixture(scope="module")
def streamed(launched):
    def run(steps, dtype=lg.LAGOM_F32, nbytes=32 * MiB, nc=128, nt=256, chunk=65536):
        count = nbytes // (4 if dtype == lg.LAGOM_F32 else 2)
        (line,) = launched("steps", dtype, count, nc, nt, chunk, *steps)
        m = re.fullmatch(r"\S*comm_steps_kernelILi(\d)ELb(\d)ELb(\d)E\S* (\d+) (\d+)", line)
        assert m and (int(m[1]), int(m[4]), int(m[5])) == (dtype, nc, nt), line
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


def test_the_benchmark_names_the_kernels_that_are_launched(launched):
    """Both layouts of B, on either side of every line of the dispatch, and products anywhere."""
    import random
    import bench
    rng = random.Random(3)
    shapes = [(512, 512, 512), (512, 512, 56), (1200, 1288, 320), (1200, 1288, 72), (2048, 4096, 4096), (4096, 4096, 4096), (4096, 4096, 4104), (4096, 4352, 4096), (4100, 4200, 2056),
              (4096, 4352, 256), (4096, 6144, 72), (4096, 6400, 4096), *((1200, 1288, k) for k in (632, 640, 648, 1272, 1280, 1288)), *((2100, 2056, k) for k in (1528, 1536, 1544))]
    shapes += [tuple(int(2 ** rng.uniform(5, 13.3)) // 8 * 8 for _ in range(3)) for _ in range(200)]
    asked = [(*s, nk, out) for s in shapes for nk in (True, False) for out in (lg.LAGOM_BF16, lg.LAGOM_F32)]
    lines = launched("gemm", *("%d,%d,%d,%d,%d" % a for a in asked))
    assert len(lines) == len(asked)
    for (M, N, K, nk, out), line in zip(asked, lines):
        name = re.search(r"\d(gemm_bf16_\w+?_kernel)[IE]", line)[1]
        assert bench.gemm_kernel_name(lg.lagom_gemm_describe(M, N, K, out), M, N, K, nk, out) == name, (M, N, K, nk, out)


@pytest.mark.parametrize("M,N,name,first,alike_nk,alike_kn", [(1200, 1288, "lines128", {True: 640, False: 1280}, 64, 32), (2100, 2056, "lines256x128", {True: 1536, False: 1536}, 32, 16)])
def test_tiles_in_lines_where_rows_start_differently(launched, M, N, name, first, alike_nk, alike_kn):
    """Rows of every class of K modulo 64: tiles hold lines where few enough rows start at one, from the size on where that pays."""
    asked = [(M, N, K, nk) for nk in (True, False) for base in (first[nk] - 64, first[nk], 4096) for K in range(base, base + 64, 8)]
    lines = launched("gemm", *("%d,%d,%d,%d,%d" % (*a, lg.LAGOM_BF16) for a in asked))
    for (_, _, K, nk), line in zip(asked, lines):
        assert ("_%s_kernel" % name in line) == (K >= first[nk] and K % (alike_nk if nk else alike_kn) != 0), (K, nk, line)
