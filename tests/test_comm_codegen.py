"""Registers of the communication kernels against what a product leaves them, checked on the gfx950 assembly.

A large-tile product runs one wavefront per SIMD, and a channel shares the compute unit with it only if the wavefronts that
the channel puts on a SIMD fit into the registers that are left of the SIMD's 512 per lane.  A channel that does not fit
takes the compute unit from the product for as long as it runs.  (No GPU needed: hipcc cross-compiles.)
"""
import re

import pytest

from paper_2602_20656_amd import build as lb

LARGE = re.compile(r"gemm_bf16_(nk|kn)(_mixed|_pieces)?(_tail)?_kernel")
REGISTERS = 512     # per lane of a SIMD, given out in blocks of 8


def _kernels(src, tmp):
    text = open(lb.device_assembly(src, str(tmp))).read()
    entries = re.split(r"\n  - (?=\.)", text[text.index("amdhsa.kernels:"):])[1:]
    return {m.group(1): dict(re.findall(r"\.(\w+):\s+(\S+)", e)) for e in entries for m in [re.search(r"\.name:\s+(\S+)", e)]}


def _allocated(meta):
    return (int(meta["vgpr_count"]) + 7) // 8 * 8


@pytest.fixture(scope="module")
def left_by_product(tmp_path_factory):
    """Registers per lane that a large-tile product leaves on its SIMD, by the layout of B."""
    left = {"nk": REGISTERS, "kn": REGISTERS}
    found = 0
    for name, meta in _kernels("gemm.hip", tmp_path_factory.mktemp("asm")).items():
        m = LARGE.search(name)
        if m:
            found += 1
            left[m.group(1)] = min(left[m.group(1)], REGISTERS - _allocated(meta))
    assert found == 2 * 3 * 2 * 2           # layouts; plain, with quadrants, with pieces; K's rest; results' types
    return left


@pytest.fixture(scope="module")
def comm(tmp_path_factory):
    kernels = _kernels("comm_kernel.hip", tmp_path_factory.mktemp("asm"))
    for name, meta in kernels.items():
        assert meta["vgpr_spill_count"] == "0" and meta["sgpr_spill_count"] == "0" and meta["private_segment_fixed_size"] == "0", name
    return kernels


def _fits(meta, nt, left):
    """Whether the wavefronts of a workgroup of nt threads that share a SIMD fit into `left` registers."""
    return -(-nt // 256) * _allocated(meta) <= left


@pytest.mark.parametrize("layout", ["nk", "kn"])
def test_fused_steps_fit_beside_a_product_up_to_512_threads(comm, left_by_product, layout):
    kernels = {n: m for n, m in comm.items() if "comm_steps_kernel" in n}
    bounds = {int(m["max_flat_workgroup_size"]) for m in kernels.values()}
    assert bounds == {256, 1024}
    for name, meta in kernels.items():
        nt = min(int(meta["max_flat_workgroup_size"]), 512)
        assert _fits(meta, nt, left_by_product[layout]), (name, nt, meta["vgpr_count"], left_by_product)


@pytest.mark.parametrize("layout", ["nk", "kn"])
def test_reduces_and_gathers_fit_beside_a_product_up_to_512_threads(comm, left_by_product, layout):
    kernels = {n: m for n, m in comm.items() if "reduce_copy_kernel" in n or "gather_copy_kernel" in n}
    assert len(kernels) == 2 * (2 * 16 * 2 + 2 * 4)         # loads streamed or not; types, sources and depths; a gather's kinds and units per batch
    for name, meta in kernels.items():
        nt = min(int(meta["max_flat_workgroup_size"]), 512)
        assert _fits(meta, nt, left_by_product[layout]), (name, nt, meta["vgpr_count"], left_by_product)


@pytest.mark.parametrize("layout", ["nk", "kn"])
def test_gathers_of_shifted_shards_fit_beside_a_product_up_to_512_threads(comm, left_by_product, layout):
    kernels = {n: m for n, m in comm.items() if "gather_halves_kernel" in n}
    assert len(kernels) == 2 * 2           # loads streamed or not; batches of four and of eight units
    for name, meta in kernels.items():
        assert _fits(meta, min(int(meta["max_flat_workgroup_size"]), 512), left_by_product[layout]), (name, meta["vgpr_count"], left_by_product)


def test_walks_keep_to_scalar_registers(tmp_path):
    """A store whose buffer the compiler holds in vector registers becomes a loop over that buffer's values, and scalars that do not fit
    are written to lanes of vector registers: either costs a wavefront more instructions than the unit it moves."""
    text = open(lb.device_assembly("comm_kernel.hip", str(tmp_path))).read()
    bodies = re.findall(r"^(_ZN\S*(?:reduce_copy|gather_copy|gather_halves|comm_steps)_kernel\S*):(.*?)s_endpgm", text, re.S | re.M)
    assert len(bodies) == 2 * (2 * 16 * 2 + 2 * 4) + 2 * 2 + 2 * 2 * 2
    for name, body in bodies:
        assert "v_writelane" not in body, name
        assert "s_xor_b64 exec, exec" not in body, name          # how such a loop takes its lanes off


def test_streamed_gathers_of_whole_shards_read_nothing_behind_the_end(tmp_path):
    """Their walks are short, and the batches behind the end a large part of them: loads are bounded by the chunk, like the stores."""
    text = open(lb.device_assembly("comm_kernel.hip", str(tmp_path))).read()
    bodies = re.findall(r"^_ZN\S*gather_copy_kernelILNS_8WalkKindE1ELb([01])ELi(\d+)E\S*:(.*?)s_endpgm", text, re.S | re.M)
    assert sorted((s, int(u)) for s, u, _ in bodies) == [(s, u) for s in "01" for u in (1, 2, 4, 8)]
    for streamed, units, body in bodies:
        assert ("global_load_dwordx4" in body) == (streamed == "0"), (streamed, units)
        assert ("buffer_load_dwordx4" in body) == (streamed == "1"), (streamed, units)
