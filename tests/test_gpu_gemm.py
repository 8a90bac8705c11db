"""GPU parity: lagom_gemm through the C ABI against the fp64 oracle, rel-err <= 2e-2
(bf16 inputs, fp32 accumulation), both error measures."""
import numpy as np
import pytest
import torch

from oracle import collective as oc, gemm as og
from paper_2602_20656_amd import binding as lg, inputs
from gpu_util import dev, host

pytestmark = pytest.mark.gpu
GATE = 2e-2


def _gemm(a_bits, b_bits, b_is_nk, out):
    M, K = a_bits.shape
    N = b_bits.shape[0] if b_is_nk else b_bits.shape[1]
    dA, dB = dev(a_bits), dev(b_bits)
    pad = 256
    if out == "bf16":
        dC = dev(np.full(M * N + 2 * pad, 0x7B7B, np.uint16)); esz = 2
    else:
        dC = dev(np.full(M * N + 2 * pad, 123.0, np.float32)); esz = 4
    lg.lagom_gemm(dA, dB, dC.data_ptr() + pad * esz, M, N, K, b_is_nk,
                  lg.LAGOM_BF16 if out == "bf16" else lg.LAGOM_F32, torch.cuda.current_stream())
    torch.cuda.synchronize()
    h = host(dC, np.uint16 if out == "bf16" else np.float32)
    guard = h[:pad].tolist() + h[pad + M * N:].tolist()
    assert all(v == (0x7B7B if out == "bf16" else 123.0) for v in guard), "guard region clobbered"
    c = h[pad:pad + M * N].reshape(M, N)
    return oc.bf16_to_f32(c) if out == "bf16" else c


def _tile(M, N, K):
    """Tile of the kernel that a shape runs on."""
    g = lg.lagom_gemm_describe(M, N, K)
    return g.tile_m, g.tile_n


@pytest.mark.parametrize("M,N,K", [(512, 512, 512), (1, 1, 8), (300, 200, 136), (700, 520, 264), (256, 256, 64),
                                   (257, 255, 72), (33, 1000, 4096), (130, 77, 128), (513, 260, 192), (700, 300, 320), (1000, 520, 256), (300, 300, 64),
                                   # more than 256 tiles of 128 x 128 but not of 256 x 128: the 256 x 128 kernels, ragged, 1 to 4 K-steps
                                   (2100, 2200, 192), (2100, 2200, 64), (1800, 2440, 128), (2312, 1800, 256),
                                   # more than 256 tiles of 256 x 128, or a K tail: the 256 x 256 kernels, ragged in M and N
                                   (2100, 3720, 192), (2100, 3720, 64), (2100, 3720, 136),
                                   # K tails on the two smaller tilings
                                   (2312, 1800, 136), (1200, 1288, 328),
                                   (1000, 520, 328)])
@pytest.mark.parametrize("b_is_nk", [True, False])
@pytest.mark.parametrize("out", ["bf16", "f32"])
def test_gemm_small_shapes(M, N, K, b_is_nk, out):
    if not b_is_nk and N % 8:
        pytest.skip("[K,N] layout needs N % 8 == 0")
    a = inputs.normal_bf16(2, (M, K))
    b = inputs.normal_bf16(3, (N, K) if b_is_nk else (K, N))
    ref = og.gemm_f64(a, b, b_is_nk)
    got = _gemm(a, b, b_is_nk, out)
    e_max, e_fro = og.rel_errors(got, ref)
    assert e_max <= GATE and e_fro <= GATE, (e_max, e_fro)
    if out == "f32":   # fp32 accumulation alone is orders of magnitude inside the gate
        assert e_fro < 1e-5, e_fro


@pytest.mark.parametrize("K", [1 << 22, (1 << 22) + 64])
def test_gemm_longest_k_of_the_fast_kernel_and_the_first_beyond_it(K):
    """K = 2^22 is the last K the LDS-direct kernel takes (32-bit lane offsets); the next multiple of 64 goes to the general one."""
    a = inputs.normal_bf16(2, (2, K)); b = inputs.normal_bf16(3, (3, K), 0.02)
    ref = og.gemm_f64(a, b, True)
    for out in ("bf16", "f32"):
        e_max, e_fro = og.rel_errors(_gemm(a, b, True, out), ref)
        assert e_max <= GATE and e_fro <= GATE, (K, out, e_max, e_fro)


def test_gemm_b_kn_widest_n_of_the_fast_kernel_and_the_first_beyond_it():
    """B stored [K,N]: N = 2^23 is the widest row the LDS-direct kernel takes (its lane offsets reach two
    K-steps = 128 rows of B ahead in 32 bits); N + 8 goes to the general one.  Three K-steps, so that the
    look-ahead offsets are used.  Checked on the first, some middle and the last columns."""
    M, K, wide = 2, 192, (1 << 23) + 8
    a = inputs.normal_bf16(2, (M, K))
    b_wide = inputs.random_bits_bf16(3, (K, wide))
    for N in (wide, 1 << 23):
        b = b_wide if N == wide else np.ascontiguousarray(b_wide[:, :N])
        got = _gemm(a, b, False, "f32")
        rng = np.random.default_rng(N)
        cols = np.unique(np.concatenate([np.arange(0, 64), rng.integers(0, N, size=256), np.arange(N - 300, N)]))
        ref = og.gemm_f64(a, np.ascontiguousarray(b[:, cols]), False)
        e_max, e_fro = og.rel_errors(got[:, cols], ref)
        assert e_max <= GATE and e_fro <= GATE and e_fro < 1e-5, (N, e_max, e_fro)
        del b, got


def test_gemm_integer_inputs_are_exact():
    rng = np.random.default_rng(5)
    ai = rng.integers(-4, 5, size=(260, 320)); bi = rng.integers(-4, 5, size=(270, 320))
    a, b = inputs.to_bf16_bits(ai.astype(np.float32)), inputs.to_bf16_bits(bi.astype(np.float32))
    got = _gemm(a, b, True, "f32")
    assert np.array_equal(got.astype(np.int64), ai @ bi.T)


@pytest.mark.parametrize("M,N,K", [(260, 272, 320), (100, 8, 64), (256, 776, 128), (513, 264, 192), (64, 1032, 576),       # K split over wavefronts
                                   (1200, 1288, 64), (1030, 1032, 128), (1201, 1480, 192), (1200, 1288, 320), (1153, 1800, 576),  # 128 x 128
                                   (2100, 2056, 128), (2304, 2312, 320),                                                 # 256 x 128
                                   (2100, 3720, 128)])                                                                   # 256 x 256
@pytest.mark.parametrize("out", ["bf16", "f32"])
def test_gemm_b_kn_integer_inputs_are_exact(M, N, K, out):
    """B stored [K,N] with K a multiple of 64 takes the kernel whose LDS reads transpose B: any mix-up of
    rows, columns or k order shows as a wrong integer.  One to nine K-steps, ragged M and N tiles, N = 8."""
    assert (_tile(M, N, K)[0] < 128) == (M * N < 1000 * 1000)
    rng = np.random.default_rng(M + N + K)
    ai = rng.integers(-3, 4, size=(M, K)); bi = rng.integers(-3, 4, size=(K, N))
    a, b = inputs.to_bf16_bits(ai.astype(np.float32)), inputs.to_bf16_bits(bi.astype(np.float32))
    got = _gemm(a, b, False, out)
    want = ai @ bi
    if out == "bf16":   # |sums| < 9 * 576: not all representable in bf16; compare after the same rounding
        want = oc.bf16_to_f32(inputs.to_bf16_bits(want.astype(np.float32)))
    assert np.array_equal(got.astype(np.float64), want.astype(np.float64))


@pytest.mark.parametrize("K", [72, 96, 104, 120, 184, 4104])
@pytest.mark.parametrize("b_is_nk", [True, False])
@pytest.mark.parametrize("M,N,tile", [(260, 272, (16, 32)), (1200, 1288, (128, 128)), (2100, 2056, (256, 128)), (2100, 3720, (256, 256))])
def test_gemm_ragged_k_integer_inputs_are_exact(K, b_is_nk, M, N, tile):
    """K >= 64 that is no multiple of 64: the last step or slice of the LDS-direct kernels begins at column K - 64 and clears the
    columns that the one before it has multiplied (8 to 56 are left of it, in one or two 32-wide MFMA slices)."""
    assert _tile(M, N, K) == tile
    if K == 4104 and M > 2000:
        pytest.skip("one long K is enough")
    rng = np.random.default_rng(K)
    ai = rng.integers(-3, 4, size=(M, K)); bi = rng.integers(-3, 4, size=(K, N))
    a = inputs.to_bf16_bits(ai.astype(np.float32))
    b = inputs.to_bf16_bits((bi.T if b_is_nk else bi).astype(np.float32))
    got = _gemm(a, b, b_is_nk, "f32")
    assert np.array_equal(got.astype(np.int64), ai @ bi)


def _random_shapes(n, seed, rows, groups):
    rng = np.random.default_rng(seed)
    shapes = []
    for i in range(n):
        M = int(rng.integers(*rows)); N = 8 * int(rng.integers(*groups))
        K = 64 * int(rng.integers(1, 7)) if i % 3 else 8 * int(rng.integers(1, 40))   # two in three on the LDS-direct kernels
        shapes.append((M, N, K))
    return shapes


@pytest.mark.parametrize("n,rows,groups", [(24, (1, 700), (1, 90)),             # K split over wavefronts, and the general kernel
                                           (12, (1030, 1600), (129, 220))])     # 128 x 128 tiles
@pytest.mark.parametrize("b_is_nk", [True, False])
def test_gemm_seeded_random_shapes(b_is_nk, n, rows, groups):
    """Seeded shapes with ragged tiles in M and N and one to six K-steps."""
    for n, (M, N, K) in enumerate(_random_shapes(n, 77, rows, groups)):
        a = inputs.normal_bf16(100 + n, (M, K))
        b = inputs.normal_bf16(200 + n, (N, K) if b_is_nk else (K, N))
        ref = og.gemm_f64(a, b, b_is_nk)
        got = _gemm(a, b, b_is_nk, "f32" if n % 2 else "bf16")
        e_max, e_fro = og.rel_errors(got, ref)
        assert e_max <= GATE and e_fro <= GATE, (M, N, K, e_max, e_fro)


def test_gemm_b_kn_full_size_sampled_rows():
    M = N = K = 4096
    a = inputs.normal_bf16(2, (M, K))
    b = inputs.normal_bf16(3, (K, N), scale=0.02)
    got = _gemm(a, b, False, "bf16")
    rng = np.random.default_rng(11)
    rows = np.unique(np.concatenate([rng.integers(0, M, size=64), np.arange(0, 4), np.arange(M - 4, M)]))
    ref = og.gemm_f64(a, b, False, rows=rows)
    e_max, e_fro = og.rel_errors(got[rows], ref)
    assert e_max <= GATE and e_fro <= GATE, (e_max, e_fro)
    corners = ref[:, np.r_[0:32, N - 32:N]]
    e_max, e_fro = og.rel_errors(got[rows][:, np.r_[0:32, N - 32:N]], corners)
    assert e_max <= GATE and e_fro <= GATE


def test_b_kn_layout_rejects_unaligned_n():
    with pytest.raises(lg.LagomError):
        lg.lagom_gemm(4096, 8192, 16384, 64, 60, 64, False)


@pytest.mark.parametrize("M,N,K", [(4096, 4096, 4096), (4096, 3584, 8192), (8192, 4096, 4096), (8192, 8192, 8192)])
def test_gemm_full_size_sampled_rows(M, N, K):
    """Benchmark shapes: 64 seeded rows x all columns, plus the four corner tiles, against the oracle."""
    a = inputs.normal_bf16(2, (M, K))
    b = inputs.normal_bf16(3, (N, K), scale=0.02)
    got = _gemm(a, b, True, "bf16")
    rng = np.random.default_rng(M + N + K)
    rows = np.unique(np.concatenate([rng.integers(0, M, size=64), np.arange(0, 4), np.arange(M - 4, M)]))
    ref = og.gemm_f64(a, b, True, rows=rows)
    e_max, e_fro = og.rel_errors(got[rows], ref)
    assert e_max <= GATE and e_fro <= GATE, (e_max, e_fro)
    corners = ref[:, np.r_[0:32, N - 32:N]]
    e_max, e_fro = og.rel_errors(got[rows][:, np.r_[0:32, N - 32:N]], corners)
    assert e_max <= GATE and e_fro <= GATE


# More 256 x 256 tiles than compute units: several rounds of workgroups, ragged in M and N.
@pytest.mark.parametrize("M,N,K", [(4100, 4200, 128),      # 17 x 17 = 289 tiles, ragged in M and N: 33 tiles in a second round
                                   (4352, 7704, 64),       # 17 x 31 = 527 tiles: two to three rounds, one K-step
                                   (8192, 8200, 192)])     # 32 x 33 = 1056 tiles: four to five rounds
@pytest.mark.parametrize("b_is_nk", [True, False])
@pytest.mark.parametrize("out", ["bf16", "f32"])
def test_gemm_more_tiles_than_compute_units_integer_inputs_are_exact(M, N, K, b_is_nk, out):
    """Small integers in bf16: every product and every partial sum is exact in fp32, so any tile that is skipped, done
    twice, mixed with its neighbour's operands or written to the wrong place shows as a wrong integer."""
    rng = np.random.default_rng(M + N + K)
    a = rng.integers(-4, 5, size=(M, K)).astype(np.float32)
    b = rng.integers(-4, 5, size=(N, K) if b_is_nk else (K, N)).astype(np.float32)
    got = _gemm(oc.f32_to_bf16(a), oc.f32_to_bf16(b), b_is_nk, out)
    want = (a @ (b.T if b_is_nk else b)).astype(np.float32)       # exact: every partial sum is a small integer
    if out == "bf16":                                                # one rounding at the store, the oracle's
        want = oc.bf16_to_f32(oc.f32_to_bf16(want))
    bad = np.argwhere(got != want)
    assert bad.size == 0, f"{len(bad)} wrong elements, first at {bad[0]} (tile {bad[0][0] // 256}, {bad[0][1] // 256})"


@pytest.mark.parametrize("M,N,tile", [
    (20, 30, (16, 32)), (250, 250, (16, 32)), (1000, 100, (16, 32)),        # fewer tiles than XCDs; 16 x 8; 63 x 4
    (500, 500, (32, 32)), (2500, 80, (32, 32)),                             # 16 x 16; 79 x 3: whole tile-rows
    (5400, 90, (64, 32)), (650, 600, (64, 32)), (90, 5400, (32, 64)),       # 85 x 3; 11 x 19; 3 x 85
    (1000, 960, (64, 64)),                                                  # 16 x 15, a last group of another height
    (1200, 1288, (128, 128)), (2100, 2056, (256, 128)), (2100, 3720, (256, 256))])      # 110, 153 and 135 tiles: no multiples of 8
@pytest.mark.parametrize("b_is_nk", [True, False])
def test_gemm_blocks_of_tiles_integer_inputs_are_exact(M, N, tile, b_is_nk):
    """Above K = 512 the list of tiles runs through near-square blocks: every tile is taken once."""
    K = 520
    if not b_is_nk:
        N = (N + 7) // 8 * 8
    assert _tile(M, N, K) == tile
    rng = np.random.default_rng(M + N)
    a = rng.integers(-4, 5, size=(M, K)).astype(np.float32)
    b = rng.integers(-4, 5, size=(N, K) if b_is_nk else (K, N)).astype(np.float32)
    got = _gemm(oc.f32_to_bf16(a), oc.f32_to_bf16(b), b_is_nk, "f32")
    assert np.array_equal(got, a @ (b.T if b_is_nk else b))


@pytest.mark.parametrize("M,N", [(3970, 4456),     # 16 x 18 tiles, 255 inside: an edge tile among the large ones
                                 (4096, 6144),     # two rounds of quadrants, none empty
                                 (4096, 6400),     # more than two rounds: large tiles only
                                 (4224, 4232),     # edge tiles with one half in C exactly, and with 8 columns of the second
                                 (130, 66000)])    # one row of tiles, none inside
@pytest.mark.parametrize("K", [64, 200])
@pytest.mark.parametrize("b_is_nk", [True, False])
def test_gemm_last_round_in_quadrants_integer_inputs_are_exact(M, N, K, b_is_nk):
    rng = np.random.default_rng(M + N + K)
    a = rng.integers(-4, 5, size=(M, K)).astype(np.float32)
    b = rng.integers(-4, 5, size=(N, K) if b_is_nk else (K, N)).astype(np.float32)
    got = _gemm(oc.f32_to_bf16(a), oc.f32_to_bf16(b), b_is_nk, "f32")
    bad = np.argwhere(got != (a @ (b.T if b_is_nk else b)))
    assert bad.size == 0, f"{len(bad)} wrong elements, first at {bad[0]}"


@pytest.mark.parametrize("M,N,out", [(2304, 2312, "f32"),                         # 256 x 128 tiles, rows of C off the 128-byte grid
                                     (3400, 3400, "bf16"), (3400, 3400, "f32"),   # 256 x 256 tiles
                                     (3584, 3584, "f32"),                         # on the grid
                                     (8192, 4104, "bf16")])                       # off it, with quadrants behind the large tiles
@pytest.mark.parametrize("K", [64, 136])
@pytest.mark.parametrize("b_is_nk", [True, False])
def test_gemm_large_results_integer_inputs_are_exact(M, N, out, K, b_is_nk):
    if not b_is_nk:
        N = (N + 7) // 8 * 8
    rng = np.random.default_rng(M + N + K)
    a = rng.integers(-4, 5, size=(M, K)).astype(np.float32)
    b = rng.integers(-4, 5, size=(N, K) if b_is_nk else (K, N)).astype(np.float32)
    want = a @ (b.T if b_is_nk else b)
    if out == "bf16":
        want = oc.bf16_to_f32(oc.f32_to_bf16(want))
    assert np.array_equal(_gemm(oc.f32_to_bf16(a), oc.f32_to_bf16(b), b_is_nk, out), want)


@pytest.mark.parametrize("M,N", [(4100, 4200),     # 17 + 16 tiles at two edges left over: 194 pieces, most of the tiles' empty
                                 (4096, 4352),     # 16 whole tiles, 256 pieces
                                 (4352, 7704),     # 15 of the right edge's tiles behind two rounds, pieces 24 columns wide
                                 (130, 66000), (66000, 136),     # no tile inside C
                                 (4096, 4101),     # pieces 5 columns wide, rows off the 16-byte grid
                                 (4096, 4357)])    # as wide, 320 of them: quadrants
@pytest.mark.parametrize("K", [264, 320])
@pytest.mark.parametrize("b_is_nk", [True, False])
@pytest.mark.parametrize("out", ["f32", "bf16"])
def test_gemm_last_round_in_pieces_integer_inputs_are_exact(M, N, K, b_is_nk, out):
    if not b_is_nk and N % 8:
        pytest.skip("[K,N] layout needs N % 8 == 0")
    rng = np.random.default_rng(M + N + K)
    a = rng.integers(-4, 5, size=(M, K)).astype(np.float32)
    b = rng.integers(-4, 5, size=(N, K) if b_is_nk else (K, N)).astype(np.float32)
    want = a @ (b.T if b_is_nk else b)
    if out == "bf16":
        want = oc.bf16_to_f32(oc.f32_to_bf16(want))
    bad = np.argwhere(_gemm(oc.f32_to_bf16(a), oc.f32_to_bf16(b), b_is_nk, out) != want)
    assert bad.size == 0, f"{len(bad)} wrong elements, first at {bad[0]}"


@pytest.mark.parametrize("M,N,tile", [(130, 136, (16, 32)), (1200, 1288, (128, 128)), (2100, 2056, (256, 128)), (2100, 3720, (256, 256))])
@pytest.mark.parametrize("K", [72, 120, 136, 200, 264, 328, 392, 456])       # two to eight steps, each peeled form of the loop
@pytest.mark.parametrize("b_is_nk", [True, False])
def test_gemm_columns_in_two_k_steps_count_once(M, N, tile, K, b_is_nk):
    """The last K-step begins at column K - 64, so it loads columns that the step before it has multiplied: those must
    neither count twice (exact integers) nor carry an infinity of theirs into zero times infinity."""
    assert _tile(M, N, K) == tile
    rng = np.random.default_rng(M + K)
    a = rng.integers(-3, 4, size=(M, K)).astype(np.float32)
    b = rng.integers(-3, 4, size=(N, K) if b_is_nk else (K, N)).astype(np.float32)
    a[3, K // 64 * 64 - 1] = np.inf             # in the overlap: one row of C is infinite or NaN, and no other
    with np.errstate(invalid="ignore"):
        want = a @ (b.T if b_is_nk else b)
    got = _gemm(oc.f32_to_bf16(a), oc.f32_to_bf16(b), b_is_nk, "f32")
    assert np.array_equal(got, want, equal_nan=True)


@pytest.mark.parametrize("M,N,Ks", [
    (1, 8, (64, 4096)), (33, 1000, (72, 512, 1544)), (250, 500, (128,)),              # 16 x 32 tiles
    (500, 501, (64, 120, 1032)), (40, 4000, (576,)),                                  # 32 x 32
    (640, 640, (128, 264, 1544)), (65, 3000, (200,)), (700, 507, (320,)),             # 64 x 32
    (90, 5400, (128, 840)), (65, 5443, (136,)),                                       # 32 x 64
    (1000, 1000, (320, 328, 1544)), (1025, 963, (384,)),                              # 64 x 64
    (1000, 1000, (64, 256)), (1200, 1288, (64, 72, 136, 320, 1032))])                 # 128 x 128, K not split
@pytest.mark.parametrize("b_is_nk", [True, False])
@pytest.mark.parametrize("out", ["bf16", "f32"])
def test_gemm_few_tiles_integer_inputs_are_exact(M, N, Ks, b_is_nk, out):
    """K split over the wavefronts of a workgroup: fewer slices of K than wavefronts, one more than a multiple of them, a
    last slice that overlaps the one before it (an infinity in the overlap reaches one row only), ragged tiles."""
    if not b_is_nk:
        N = (N + 7) // 8 * 8
    for K in Ks:
        rng = np.random.default_rng(M + N + K)
        a = rng.integers(-3, 4, size=(M, K)).astype(np.float32)
        b = rng.integers(-3, 4, size=(N, K) if b_is_nk else (K, N)).astype(np.float32)
        if K % 64:
            a[M // 2, K // 64 * 64 - 1] = np.inf
        with np.errstate(invalid="ignore"):
            want = a @ (b.T if b_is_nk else b)
        if out == "bf16":        # one rounding at the store, the oracle's
            want = oc.bf16_to_f32(oc.f32_to_bf16(want.astype(np.float32)))
        got = _gemm(oc.f32_to_bf16(a), oc.f32_to_bf16(b), b_is_nk, out)
        assert np.array_equal(got, want, equal_nan=True), (K, np.argwhere(got != want)[:3])


@pytest.mark.parametrize("M,N,K", [(33, 1002, 136), (500, 500, 128), (500, 502, 128), (500, 504, 72), (64, 5404, 136), (90, 5402, 128), (640, 636, 136), (640, 634, 128),
                                   (1000, 956, 320), (1000, 958, 328), (4100, 4196, 328), (4100, 4198, 320)])      # 16 to 64 rows, and 64 x 64 pieces beside large tiles
@pytest.mark.parametrize("out", ["bf16", "f32"])
def test_gemm_split_rows_on_and_off_the_grids_of_four_and_eight(M, N, K, out):
    """Vectors of four results go through the L2 or into it by where rows of C begin; nothing beside C is written."""
    assert _tile(M, N, K)[0] in (16, 32, 64, 256)
    rng = np.random.default_rng(M + N + K)
    a = rng.integers(-4, 5, size=(M, K)).astype(np.float32)
    b = rng.integers(-4, 5, size=(N, K)).astype(np.float32)
    want = a @ b.T
    if out == "bf16":
        want = oc.bf16_to_f32(oc.f32_to_bf16(want))
    room = torch.full((M * N + 128,), 123.0, dtype=torch.bfloat16 if out == "bf16" else torch.float32, device="cuda")
    lg.lagom_gemm(torch.from_numpy(a).cuda().to(torch.bfloat16), torch.from_numpy(b).cuda().to(torch.bfloat16), room.data_ptr() + 64 * room.element_size(), M, N, K, True,
                  lg.LAGOM_BF16 if out == "bf16" else lg.LAGOM_F32, torch.cuda.current_stream())
    torch.cuda.synchronize()
    h = room.float().cpu().numpy()
    assert np.array_equal(h[64:64 + M * N].reshape(M, N), want)
    assert (h[:64] == 123.0).all() and (h[64 + M * N:] == 123.0).all()


@pytest.mark.parametrize("M,N", [(1201, 1203), (1202, 1285), (2100, 2201), (2065, 2308), (2100, 3725), (4100, 4198)])   # 128 x 128, 256 x 128, 256 x 256 tiles, and with quadrants
@pytest.mark.parametrize("K", [64, 136])
@pytest.mark.parametrize("out", ["bf16", "f32"])
def test_gemm_rows_off_the_16_byte_grid(M, N, K, out):
    """N no multiple of 8: rows of C start off the 16-byte grid and end inside a vector (1 to 7 elements of it)."""
    rng = np.random.default_rng(M + N + K)
    a = rng.integers(-4, 5, size=(M, K)).astype(np.float32)
    b = rng.integers(-4, 5, size=(N, K)).astype(np.float32)
    want = a @ b.T
    if out == "bf16":
        want = oc.bf16_to_f32(oc.f32_to_bf16(want))
    assert np.array_equal(_gemm(oc.f32_to_bf16(a), oc.f32_to_bf16(b), True, out), want)


@pytest.mark.parametrize("M,N,more", [(1025, 1032, 0), (1153, 1800, 0), (4001, 1000, 0),      # 81, 150 and 256 tiles of 128 x 128, one row or column in the last ones
                                      (2100, 2056, 960)])                                     # 256 x 128, from K = 1536 on
@pytest.mark.parametrize("K", [648, 1288, 1304, 1320, 1336, 1352, 1368, 1384, 1400])  # 8 to 56 columns behind the last whole step, rows 1 to 7 groups apart on the line
@pytest.mark.parametrize("b_is_nk", [True, False])
@pytest.mark.parametrize("shift", [0, 3])
def test_gemm_lines_of_rows_anywhere_integer_inputs_are_exact(M, N, more, K, b_is_nk, shift):
    """Tiles hold the lines that rows lie in, which begin `shift` groups of 16 bytes behind a line and K / 8 more from row to row.  The last columns
    of a row and the first of the next lie in one line: what is infinite there reaches its own row and column only."""
    K += more
    assert _tile(M, N, K) == ((256, 128) if more else (128, 128))
    rng = np.random.default_rng(M + K)
    a = rng.integers(-3, 4, size=(M, K)).astype(np.float32)
    b = rng.integers(-3, 4, size=(N, K) if b_is_nk else (K, N)).astype(np.float32)
    want = a @ (b.T if b_is_nk else b)
    bad_rows, bad_col = (1, M - 1), N - 2
    a[bad_rows[0], 0], a[bad_rows[1], K - 1] = np.inf, np.inf
    if b_is_nk: b[bad_col, K - 1] = np.inf
    else: b[K - 1, bad_col] = np.inf
    def placed(x):
        flat = torch.zeros(x.size + 64, dtype=torch.bfloat16, device="cuda")
        flat[8 * shift:8 * shift + x.size] = torch.from_numpy(x.reshape(-1)).to(torch.bfloat16).cuda()
        return flat, flat.data_ptr() + 16 * shift
    (fa, pa), (fb, pb), c = placed(a), placed(b), torch.zeros((M, N), dtype=torch.float32, device="cuda")
    lg.lagom_gemm(pa, pb, c, M, N, K, b_is_nk, lg.LAGOM_F32, torch.cuda.current_stream())
    torch.cuda.synchronize()
    got = c.cpu().numpy()
    clean = np.ones((M, N), bool)
    clean[list(bad_rows)] = False
    clean[:, bad_col] = False
    assert np.array_equal(got[clean], want[clean])
    assert not np.isfinite(got[list(bad_rows)]).any() and not np.isfinite(got[:, bad_col]).any()


@pytest.mark.parametrize("M,N,more", [(1025, 1032, 0), (2100, 2056, 960)])
@pytest.mark.parametrize("K", [1296, 1312, 1328])          # multiples of 16 and 32: some rows start at a line
@pytest.mark.parametrize("b_is_nk", [True, False])
@pytest.mark.parametrize("shift", [0, 3])
def test_gemm_lines_of_rows_that_start_alike_integer_inputs_are_exact(M, N, more, K, b_is_nk, shift):
    test_gemm_lines_of_rows_anywhere_integer_inputs_are_exact(M, N, more, K, b_is_nk, shift)


@pytest.mark.parametrize("M,N,K,tile", [(300, 192, 200, (16, 32)), (640, 640, 136, (64, 32)), (90, 5400, 128, (32, 64)), (1000, 960, 320, (64, 64)),
                                        (1200, 1280, 72, (128, 128)), (2100, 2112, 128, (256, 128)), (2100, 3712, 128, (256, 256)), (4100, 4224, 320, (256, 256))])
@pytest.mark.parametrize("out", ["bf16", "f32"])
@pytest.mark.parametrize("shift", [0, 1, 4])          # groups of 16 bytes that C begins behind a 128-byte line
def test_gemm_results_on_and_off_the_lines_integer_inputs_are_exact(M, N, K, tile, out, shift):
    """Rows of C on 128-byte lines, and off them by where C begins: stored past the L2, or through it; nothing beside C is written."""
    assert _tile(M, N, K) == tile
    rng = np.random.default_rng(M + K)
    a = rng.integers(-4, 5, size=(M, K)).astype(np.float32)
    b = rng.integers(-4, 5, size=(N, K)).astype(np.float32)
    want = a @ b.T
    if out == "bf16":
        want = oc.bf16_to_f32(oc.f32_to_bf16(want))
    dt, esz = (torch.bfloat16, 2) if out == "bf16" else (torch.float32, 4)
    room = torch.full((M * N + 512,), 123.0, dtype=dt, device="cuda")
    first = 128 // esz + 16 * shift // esz
    assert room.data_ptr() % 128 == 0
    lg.lagom_gemm(torch.from_numpy(a).cuda().to(torch.bfloat16), torch.from_numpy(b).cuda().to(torch.bfloat16), room.data_ptr() + first * esz, M, N, K, True,
                  lg.LAGOM_BF16 if out == "bf16" else lg.LAGOM_F32, torch.cuda.current_stream())
    torch.cuda.synchronize()
    h = room.float().cpu().numpy()
    assert np.array_equal(h[first:first + M * N].reshape(M, N), want)
    assert (h[:first] == 123.0).all() and (h[first + M * N:] == 123.0).all()
