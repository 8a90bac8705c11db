"""What the fast GEMM kernel relies on in the generated code, checked on the gfx950 assembly.

Its MFMAs are inline asm, so the compiler knows neither their latency nor the wait states an
accumulator read needs after one.  The kernel is only correct if nothing but an MFMA touches an
accumulator register between the first MFMA and the wait states that follow the last one:
no spill, no copy, no early read.  (No GPU needed: hipcc cross-compiles.)
"""
import re

import pytest

from paper_2602_20656_amd import build as lb

KERNELS = tuple("gemm_bf16_%s_kernelILb%dE" % (k, o) for k in ("nk", "kn", "nk_tail", "kn_tail") for o in (1, 0))
SMALL = tuple("gemm_bf16_%s128%s_kernelILb%dE" % (k, t, o) for k in ("nk", "kn") for t in ("", "_tail") for o in (1, 0))   # 128 x 128 tiles, 64 accumulators
MEDIUM = tuple("gemm_bf16_%s256x128%s_kernelILb%dE" % (k, t, o) for k in ("nk", "kn") for t in ("", "_tail") for o in (1, 0))   # 256 x 128 tiles, 128 accumulators
ACCS = {**{k: 256 for k in KERNELS}, **{k: 64 for k in SMALL}, **{k: 128 for k in MEDIUM}}
AGPR = re.compile(r"\ba(\[\d+:\d+\]|\d+)\b")


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    path = lb.device_assembly("gemm.hip", str(tmp_path_factory.mktemp("asm")))
    return open(path).read()


def _body(text, name):
    m = re.search(r"^(\S*%s\S*):.*\n" % re.escape(name), text, re.M)
    assert m, name
    end = text.index("s_endpgm", m.end())
    return m.group(1), [l.split(";")[0].strip() for l in text[m.end():end].splitlines()]


def _metadata(text, sym):
    """The amdhsa.kernels entry of one kernel as a dict of its scalar fields."""
    kernels = text[text.index("amdhsa.kernels:"):]
    for entry in re.split(r"\n  - (?=\.)", kernels):
        if re.search(r"\.name:\s+%s\b" % re.escape(sym), entry):
            return dict(re.findall(r"\.(\w+):\s+(\S+)", entry))
    raise AssertionError(sym)


@pytest.mark.parametrize("name", KERNELS + SMALL + MEDIUM)
def test_no_spills_and_all_agprs_for_accumulators(assembly, name):
    sym, _ = _body(assembly, name)
    meta = _metadata(assembly, sym)
    assert meta["vgpr_spill_count"] == "0" and meta["sgpr_spill_count"] == "0", meta
    assert meta["agpr_count"] == str(ACCS[name]), meta
    assert meta["private_segment_fixed_size"] == "0", meta


def _blocks(lines):
    """Basic blocks in text order: (falls_in, [instructions]); falls_in is False after an unconditional branch."""
    blocks, cur, falls_in = [], [], True
    for l in lines:
        if not l:
            continue
        if l.endswith(":") and not l.startswith("s_") and not l.startswith("v_"):
            prev = cur[-1] if cur else ""
            blocks.append((falls_in, cur))
            falls_in, cur = not prev.startswith("s_branch"), []
        else:
            cur.append(l)
    blocks.append((falls_in, cur))
    return blocks


@pytest.mark.parametrize("name", KERNELS + SMALL + MEDIUM)
def test_only_mfmas_touch_accumulators_until_the_wait_states(assembly, name):
    _, lines = _body(assembly, name)
    mfma = [i for i, l in enumerate(lines) if l.startswith("v_mfma_f32_16x16x32_bf16")]
    assert len(mfma) >= 3 * ACCS[name] // 2        # the steady-state step and at least two peeled steps
    nop = next(i for i in range(mfma[-1], len(lines)) if lines[i].startswith("s_nop 7"))
    assert lines[nop + 1].startswith("s_nop 7") and lines[nop + 2].startswith("s_nop 7")
    for falls_in, block in _blocks(lines[mfma[0]:nop]):
        has_mfma = any(l.startswith("v_mfma") for l in block)
        for l in block:
            if l.startswith("v_mfma_f32_16x16x32_bf16"):
                continue
            assert not l.startswith("scratch_"), l
            if AGPR.search(l):
                # the one exception: the zero fill of the accumulators on the path that skips the
                # steady-state loop, a block of its own that is only jumped to and holds no MFMA
                assert not has_mfma and not falls_in and l.startswith(("v_accvgpr_mov_b32", "v_accvgpr_write_b32")), l


@pytest.mark.parametrize("name", KERNELS)
def test_steady_state_step_is_branch_free_with_one_side_instruction_per_mfma(assembly, name):
    _, lines = _body(assembly, name)
    lines = [l for l in lines if l]
    # the loop: from its label to the first backward scalar branch behind the first MFMA
    first = next(i for i, l in enumerate(lines) if l.startswith("v_mfma"))
    back = next(i for i in range(first, len(lines)) if lines[i].startswith("s_cbranch"))
    label = lines[back].split()[-1] + ":"
    head = max(i for i in range(first) if lines[i].startswith(label))
    body = [l for l in lines[head + 1:back] if not l.endswith(":")]
    assert sum(l.startswith("v_mfma") for l in body) == 128
    assert sum(l.startswith("global_load_lds_dwordx4") for l in body) == 16
    if "_nk_" in name:
        assert sum(l.startswith("ds_read_b128") for l in body) == 32
    else:   # B stored [K,N]: 16 reads of A, 2 x 16 transposing reads of B
        assert sum(l.startswith("ds_read_b128") for l in body) == 16
        assert sum(l.startswith("ds_read_b64_tr_b16") for l in body) == 32
        assert not any(l.startswith(("v_mov_b32", "v_perm_b32")) for l in body)   # fragment halves land in place
    assert sum(l.startswith("s_barrier") for l in body) == 1
    run, worst, lead = 0, 0, None
    for l in body:      # side instructions between two MFMAs
        if l.startswith("v_mfma"):
            if lead is None:
                lead = run          # in front of the first MFMA: the loop's own bookkeeping
            else:
                worst = max(worst, run)
            run = 0
        elif not l.startswith(("s_waitcnt", "s_barrier")):
            run += 1
    assert worst <= 2, worst        # an M0 write, a load or a fragment read; nothing longer
    # slot rotation, two running pointers, the counter ([K,N]: and the slot's base added to 8 fragment addresses)
    assert lead + run <= 24, (lead, run)


@pytest.mark.parametrize("name", SMALL + MEDIUM)
def test_small_tile_step_has_one_side_instruction_per_mfma(assembly, name):
    ni = 4 if name in SMALL else 8          # A fragments per wavefront and k-slice; 4 B fragments
    _, lines = _body(assembly, name)
    lines = [l for l in lines if l]
    first = next(i for i, l in enumerate(lines) if l.startswith("v_mfma"))
    back = next(i for i in range(first, len(lines)) if lines[i].startswith("s_cbranch"))
    label = lines[back].split()[-1] + ":"
    head = max(i for i in range(first) if lines[i].startswith(label))
    body = [l for l in lines[head + 1:back] if not l.endswith(":")]
    assert sum(l.startswith("v_mfma") for l in body) == 2 * ni * 4
    assert sum(l.startswith("global_load_lds_dwordx4") for l in body) == ni + 4
    assert sum(l.startswith("s_barrier") for l in body) == 1
    if "_nk" in name:
        assert sum(l.startswith("ds_read_b128") for l in body) == 2 * (ni + 4)
    else:   # B stored [K,N]: reads of A, 2 x 8 transposing reads of B
        assert sum(l.startswith("ds_read_b128") for l in body) == 2 * ni
        assert sum(l.startswith("ds_read_b64_tr_b16") for l in body) == 16
    run, worst, seen = 0, 0, False
    for l in body:
        if l.startswith("v_mfma"):
            if seen:
                worst = max(worst, run)
            seen, run = True, 0
        elif not l.startswith(("s_waitcnt", "s_barrier")):
            run += 1
    assert worst <= 4, worst   # an address add or two with a read; an offset add with an M0 write


MIXED = tuple("gemm_bf16_%s_mixed%s_kernelILb%dE" % (k, t, o) for k in ("nk", "kn") for t in ("", "_tail") for o in (1, 0))   # both bodies in one kernel


@pytest.mark.parametrize("name", MIXED)
def test_both_bodies_of_a_mixed_kernel_keep_their_accumulators(assembly, name):
    sym, _ = _body(assembly, name)
    start = assembly.index("\n" + sym + ":")
    lines = [l.split(";")[0].strip() for l in assembly[start:assembly.index(".Lfunc_end", start)].splitlines()[2:]]   # past the early ends
    lines = [l for l in lines if l]
    meta = _metadata(assembly, sym)
    assert meta["vgpr_spill_count"] == "0" and meta["sgpr_spill_count"] == "0", meta
    assert meta["agpr_count"] == "256" and meta["private_segment_fixed_size"] == "0", meta
    waits = [i for i in range(len(lines) - 2) if all(l.startswith("s_nop 7") for l in lines[i:i + 3])]
    assert len(waits) == 2
    start = 0
    for nop in waits:
        mfma = [i for i in range(start, nop) if lines[i].startswith("v_mfma_f32_16x16x32_bf16")]
        assert len(mfma) >= 3 * 64 // 2
        for falls_in, block in _blocks(lines[mfma[0]:nop]):
            has_mfma = any(l.startswith("v_mfma") for l in block)
            for l in block:
                if not l.startswith("v_mfma_f32_16x16x32_bf16") and AGPR.search(l):
                    assert not has_mfma and not falls_in and l.startswith(("v_accvgpr_mov_b32", "v_accvgpr_write_b32")), l
        start = nop + 3
    assert not any(l.startswith("v_mfma") for l in lines[start:])


PIECES = tuple("gemm_bf16_%s_pieces%s_kernelILb%dE" % (k, t, o) for k in ("nk", "kn") for t in ("", "_tail") for o in (1, 0))


@pytest.mark.parametrize("name", PIECES)
def test_large_body_of_a_kernel_with_split_pieces_keeps_its_accumulators(assembly, name):
    """The pieces' MFMAs are the compiler's own, in a body of their own."""
    sym, _ = _body(assembly, name)
    start = assembly.index("\n" + sym + ":")
    lines = [l.split(";")[0].strip() for l in assembly[start:assembly.index(".Lfunc_end", start)].splitlines()[2:]]
    lines = [l for l in lines if l]
    meta = _metadata(assembly, sym)
    assert meta["vgpr_spill_count"] == "0" and meta["sgpr_spill_count"] == "0" and meta["private_segment_fixed_size"] == "0", meta
    waits = [i for i in range(len(lines) - 2) if all(l.startswith("s_nop 7") for l in lines[i:i + 3])]
    assert len(waits) == 1
    begin = max(i for i in range(waits[0]) if lines[i].startswith("s_setprio"))          # either body begins with it
    first = next(i for i in range(begin, waits[0]) if lines[i].startswith("v_mfma"))
    blocks = _blocks(lines[first:waits[0]])
    assert sum(l.startswith("v_mfma") for _, b in blocks for l in b) >= 3 * 128
    for falls_in, block in blocks:
        has_mfma = any(l.startswith("v_mfma") for l in block)
        for l in block:
            if not l.startswith("v_mfma_f32_16x16x32_bf16") and AGPR.search(l):
                assert not has_mfma and not falls_in and l.startswith(("v_accvgpr_mov_b32", "v_accvgpr_write_b32")), l


def test_results_go_past_the_l2(assembly):
    """Whole vectors of C carry the non-temporal hint in every tiled kernel: what the last-level cache holds for kernels beside a product stays there."""
    names = set(re.findall(r"^(\S*gemm_bf16_(?:nk|kn)\S*_kernel\S*):", assembly, re.M))
    assert len(names) == 8 * (3 + 2)               # large tiles, with quadrants, with pieces; 256 x 128 and 128 x 128; K's rest, results' types
    for sym in names:
        body = assembly[assembly.index("\n" + sym + ":"):]
        body = body[:body.index(".Lfunc_end")]
        hinted = len(re.findall(r"^\s*global_store_dwordx4 .* nt\b", body, re.M))
        assert hinted >= (8 if "128" in sym else 32), (sym, hinted)


@pytest.mark.parametrize("M,N,K,name", [
    (512, 512, 512, "split"), (512, 512, 56, "general"), (1200, 1288, 320, "nk128"), (1200, 1288, 72, "nk128_tail"), (2048, 4096, 4096, "nk256x128"),
    (4096, 4096, 4096, "nk"), (4096, 4096, 4104, "nk_tail"), (4096, 4352, 4096, "nk_pieces"), (4100, 4200, 2056, "nk_pieces_tail"),
    (4096, 4352, 256, "nk_mixed"), (4096, 6144, 72, "nk_mixed_tail"), (4096, 6400, 4096, "nk")])
def test_bench_names_the_kernel_that_runs(assembly, M, N, K, name):
    import bench
    from paper_2602_20656_amd import binding as lg
    got = bench.gemm_kernel_name(lg.lagom_gemm_describe(M, N, K, lg.LAGOM_BF16), M, N, K)
    assert got == f"gemm_bf16_{name}_kernel"
    assert re.search(r"^\S*\d%sI?\S*:" % got, assembly, re.M)


LINES = tuple("gemm_bf16_lines%s_kernelILb%dELb%dE" % (t, k, o) for t in ("128", "256x128") for k in (0, 1) for o in (1, 0))


@pytest.mark.parametrize("name", LINES)
def test_tiles_in_lines_keep_their_accumulators_and_one_side_instruction_per_mfma(assembly, name):
    sym, lines = _body(assembly, name)
    meta = _metadata(assembly, sym)
    assert meta["vgpr_spill_count"] == "0" and meta["sgpr_spill_count"] == "0" and meta["private_segment_fixed_size"] == "0", meta
    ni = 8 if "256x128" in name else 4
    assert meta["agpr_count"] == str(16 * ni), meta
    lines = [l for l in lines if l]
    mfma = [i for i, l in enumerate(lines) if l.startswith("v_mfma_f32_16x16x32_bf16")]
    nop = next(i for i in range(mfma[-1], len(lines)) if lines[i].startswith("s_nop 7"))
    assert all(l.startswith("s_nop 7") for l in lines[nop:nop + 3])
    for falls_in, block in _blocks(lines[mfma[0]:nop]):
        for l in block:
            if AGPR.search(l) and not l.startswith("v_mfma_f32_16x16x32_bf16"):
                assert not falls_in and not any(b.startswith("v_mfma") for b in block) and l.startswith(("v_accvgpr_mov_b32", "v_accvgpr_write_b32")), l
    back = next(i for i in range(mfma[0], len(lines)) if lines[i].startswith("s_cbranch"))
    label = lines[back].split()[-1] + ":"
    head = max(i for i in range(mfma[0]) if lines[i].startswith(label))
    body = [l for l in lines[head + 1:back] if not l.endswith(":")]
    assert sum(l.startswith("v_mfma") for l in body) == 8 * ni and sum(l.startswith("s_barrier") for l in body) == 1
    assert sum(l.startswith("global_load_lds_dwordx4") for l in body) == ni + 4
    run, worst, seen = 0, 0, False
    for l in body:
        if l.startswith("v_mfma"):
            worst, seen, run = max(worst, run) if seen else 0, True, 0
        elif not l.startswith(("s_waitcnt", "s_barrier")):
            run += 1
    assert worst <= 5, worst        # two selects, an address add and a read


@pytest.mark.parametrize("M,N,K,name", [(1200, 1288, 632, "nk128_tail"), (1200, 1288, 648, "lines128"), (1200, 1288, 704, "nk128"), (2100, 2056, 1528, "nk256x128_tail"), (2100, 2056, 1544, "lines256x128")])
def test_bench_names_the_kernel_of_tiles_in_lines(assembly, M, N, K, name):
    import bench
    from paper_2602_20656_amd import binding as lg
    got = bench.gemm_kernel_name(lg.lagom_gemm_describe(M, N, K, lg.LAGOM_BF16), M, N, K)
    assert got == f"gemm_bf16_{name}_kernel" and re.search(r"^\S*\d%sI?\S*:" % got, assembly, re.M)


@pytest.mark.parametrize("name", SMALL + MEDIUM + LINES)
def test_no_load_into_lds_is_in_flight_when_results_are_staged_there(assembly, name):
    """Results pass through the LDS that the tiles lie in: behind the last step, on every path, all loads have landed and all wavefronts know."""
    _, lines = _body(assembly, name)
    lines = [l for l in lines if l]
    mfma = max(i for i, l in enumerate(lines) if l.startswith("v_mfma_f32_16x16x32_bf16"))
    write = next(i for i in range(mfma, len(lines)) if lines[i].startswith("ds_write"))
    nop = next(i for i in range(mfma, write) if lines[i].startswith("s_nop 7"))
    behind = lines[nop:write]              # one block: every path from the steps to the first write runs through all of it
    assert not any(l.endswith(":") or l.startswith(("s_cbranch", "s_branch")) for l in behind)
    wait = next((i for i, l in enumerate(behind) if l.startswith("s_waitcnt vmcnt(0)")), None)
    assert wait is not None and any(l.startswith("s_barrier") for l in behind[wait:])


def test_stores_through_the_l2_keep_their_registers_for_two_wait_states(assembly):
    """A vector instruction may write the registers of a store of more than 8 bytes two wait states behind it; the compiler does not look into inline asm."""
    lines = [l for l in (l.split(";")[0].strip() for l in assembly.splitlines()) if l]
    stores = [i for i, l in enumerate(lines) if re.match(r"global_store_dwordx4 .* sc1\b", l)]
    assert stores
    for i in stores:
        nop = re.match(r"s_nop (\d+)", lines[i + 1])
        assert nop and int(nop.group(1)) >= 1, lines[i:i + 3]


@pytest.mark.parametrize("tile,through", [((1, 2), ()), ((2, 2), ("x4",)), ((2, 4), ("x4",)), ((4, 2), ("x4",)), ((4, 4), ("x4",))])
def test_split_products_store_through_the_l2_by_a_rule_only(assembly, tile, through):
    """Vectors of four fp32 results leave tiles of 32 rows and more through the L2, or into it where rows of C lie off the 64-byte grid; all others go into it."""
    bodies = re.findall(r"^\S*gemm_bf16_split_kernelINS_9SplitTileILi%dELi%dE\S*:.*?^\.Lfunc_end" % tile, assembly, re.M | re.S)
    assert len(bodies) == 4          # both layouts of B, K a multiple of 64 or not
    for body in bodies:
        lines = [l.split(";")[0].strip() for l in body.splitlines()]
        for size in ("x4", "x2"):
            stores = [l for l in lines if l.startswith("global_store_dword%s " % size)]
            assert any("sc1" not in l for l in stores)
            assert any("sc1" in l for l in stores) == (size in through), (size, stores)


def test_no_other_product_stores_through_the_l2(assembly):
    """Parts of lines that go through the L2 are written to memory one by one: 1.05 - 1.5 of the time where the results are not in the last-level cache."""
    for sym, body in re.findall(r"^(\S*gemm_bf16\w*_kernel\S*):(.*?)^\.Lfunc_end", assembly, re.M | re.S):
        if "split" not in sym and "pieces" not in sym:
            assert not re.search(r"^\s*global_store\S* .* sc1\b", body, re.M), sym
