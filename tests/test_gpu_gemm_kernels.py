"""The two tiled kernels of the MXFP4 product against the oracle's emulated product, each forced through the
diagnostics switch: the 256 x 256 tile kernel and the 256 x 128 tile kernel with two accumulator sets (C stores of a
tile issued during the next tile).  Shapes cover one tile, several tiles per workgroup (both accumulator sets, an odd
and an even count of tiles per workgroup), ragged edges, tile counts whose
split over the eight XCDs does and does not fall on whole bands of the tile order, and stage counts from the minimum of
the two-set kernel (8) up.  Every element is compared (1e-5 relative Frobenius and the per-element
accumulation allowance of test_gpu_parity)."""
import numpy as np
import pytest

from oracle import reference as orc
from paper_2604_02525_amd import inputs
from test_gpu_parity import ah, check_c, host, rel_fro, say, stored  # noqa: F401  (ah is a fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TILE256, DUAL = 1, 2


@pytest.fixture
def force(ah):
    yield lambda which: ah.adahop_debug_force_gemm_kernel(which)
    ah.adahop_debug_force_gemm_kernel(0)


def dequant_norms(codes, scales):
    table = np.array([0, .5, 1, 1.5, 2, 3, 4, 6, 0, .5, 1, 1.5, 2, 3, 4, 6], dtype=np.float64)   # magnitudes only
    mag2 = table[codes & 15] ** 2 + table[codes >> 4] ** 2                                        # per byte
    per_block = mag2.reshape(codes.shape[0], -1, 16).sum(axis=2)
    return np.sqrt((per_block * np.exp2(2.0 * (scales.astype(np.float64) - 127.0))).sum(axis=1))


@pytest.mark.parametrize("kernel", [TILE256, DUAL])
@pytest.mark.parametrize("shape", [(256, 128, 2048), (256, 256, 2048), (512, 384, 2304), (768, 1280, 4096),
                                   (300, 200, 2560), (1000, 650, 2048), (4352, 4096, 2048), (8448, 4224, 2048),
                                   (4096, 2176, 3072), (3584, 1024, 2048), (7168, 2048, 2048)])
def test_tiled_kernels_match_emulation(ah, force, kernel, shape):
    M, N, K = shape
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    a_codes = rng.integers(0, 256, size=(M, K // 2), dtype=np.uint8)
    b_codes = rng.integers(0, 256, size=(N, K // 2), dtype=np.uint8)
    a_scales = rng.integers(117, 137, size=(M, K // 32), dtype=np.uint8)
    b_scales = rng.integers(100, 120, size=(N, K // 32), dtype=np.uint8)
    say("tiled kernel", {TILE256: "256x256", DUAL: "256x128 two sets"}[kernel], shape)
    force(kernel)
    C = ah.adahop_gemm_mx(*(torch.from_numpy(t).cuda() for t in (a_codes, a_scales, b_codes, b_scales)))
    torch.cuda.synchronize()
    got = host(C).astype(np.float64)
    if M * N * K <= 4352 * 4096 * 2048:
        rows = cols = None
        ref = orc.mx_gemm(a_codes, a_scales, b_codes, b_scales)
    else:       # one row and one column in every 64-band: every tile, every wave's part of it
        rows = (np.arange(0, M, 64) + rng.integers(0, 64, (M + 63) // 64)).clip(max=M - 1).astype(np.int32)
        cols = (np.arange(0, N, 64) + rng.integers(0, 64, (N + 63) // 64)).clip(max=N - 1).astype(np.int32)
        ref = orc.mx_gemm(a_codes, a_scales, b_codes, b_scales, rows, cols)
        got = got[np.ix_(rows, cols)]
    err = rel_fro(got, ref)
    na, nb = dequant_norms(a_codes, a_scales), dequant_norms(b_codes, b_scales)
    bar = 2.0 ** -20 * np.outer(na if rows is None else na[rows], nb if cols is None else nb[cols])
    worst = float((np.abs(got - ref) / bar).max())
    say(f"  rel_fro {err:.2e}, worst element at {worst:.3f} of its allowance")
    assert err < 1e-5
    assert worst <= 1.0


@pytest.mark.parametrize("kernel", [TILE256, DUAL])
def test_tiled_kernels_single_nonzero_positions(ah, force, kernel):
    """One nonzero code per operand: the product lands in exactly one element of C with exactly the right value, for
    positions in different tiles, waves, accumulator tiles, pipeline stages and scale slots."""
    M, N, K = 768, 512, 2560
    force(kernel)
    rng = np.random.default_rng(kernel)
    for _ in range(12):
        m, n, ka = int(rng.integers(0, M)), int(rng.integers(0, N)), int(rng.integers(0, K))
        a_codes = np.zeros((M, K // 2), np.uint8)
        b_codes = np.zeros((N, K // 2), np.uint8)
        a_scales = np.full((M, K // 32), 127, np.uint8)
        b_scales = np.full((N, K // 32), 127, np.uint8)
        a_codes[m, ka // 2] = int(rng.integers(1, 16)) << (4 * (ka & 1))
        b_codes[n, ka // 2] = int(rng.integers(1, 16)) << (4 * (ka & 1))
        if (a_codes[m, ka // 2] >> (4 * (ka & 1))) & 7 == 0 or (b_codes[n, ka // 2] >> (4 * (ka & 1))) & 7 == 0:
            continue                                                       # a signed zero: nothing to find
        a_scales[m, ka // 32] = int(rng.integers(120, 135))
        b_scales[n, ka // 32] = int(rng.integers(120, 135))
        say("single nonzero", kernel, (m, n, ka))
        C = host(ah.adahop_gemm_mx(*(torch.from_numpy(t).cuda() for t in (a_codes, a_scales, b_codes, b_scales))))
        ref = orc.mx_gemm(a_codes, a_scales, b_codes, b_scales)
        assert np.count_nonzero(ref) == 1
        assert np.array_equal(C.astype(np.float64), ref)


RAGGED = [(257, 256, 544), (511, 383, 1056), (300, 130, 1824), (1000, 650, 2016), (769, 513, 2080), (2305, 1100, 2912)]


@pytest.mark.parametrize("kernel", [TILE256, DUAL])
@pytest.mark.parametrize("shape", RAGGED)
def test_ragged_shapes_in_whole_tiles(ah, force, kernel, shape):
    """Rows, columns and K one past, one short of and between whole tiles and stages: the last tile of a dimension and the
    last stage of K overlap the ones before them (scales re-ordered by the pre-pass).  The allowance is the one above."""
    M, N, K = shape
    rng = np.random.default_rng(5 * M + 3 * N + K)
    a_codes = rng.integers(0, 256, size=(M, K // 2), dtype=np.uint8)
    b_codes = rng.integers(0, 256, size=(N, K // 2), dtype=np.uint8)
    a_scales = rng.integers(117, 137, size=(M, K // 32), dtype=np.uint8)
    b_scales = rng.integers(100, 120, size=(N, K // 32), dtype=np.uint8)
    say("ragged", kernel, shape)
    force(kernel)
    got = host(ah.adahop_gemm_mx(*(torch.from_numpy(t).cuda() for t in (a_codes, a_scales, b_codes, b_scales)))).astype(np.float64)
    ref = orc.mx_gemm(a_codes, a_scales, b_codes, b_scales)
    bar = 2.0 ** -20 * np.outer(dequant_norms(a_codes, a_scales), dequant_norms(b_codes, b_scales))
    assert rel_fro(got, ref) < 1e-5
    assert float((np.abs(got - ref) / bar).max()) <= 1.0


@pytest.mark.parametrize("layouts", [(True, True), (True, False), (False, False)])
@pytest.mark.parametrize("M,N,K", [(301, 270, 1120), (520, 264, 800), (257, 512, 2272)])
@pytest.mark.parametrize("strategy,k", [(inputs.IHT, 0), (inputs.IHT_OE_K, 40), (inputs.IHT_OE_ROW, 5)])
def test_ragged_whole_path(ah, layouts, M, N, K, strategy, k):
    """The same with the stage-major scales written by the quantisers of both layouts, and gathered K-channels in front."""
    A = inputs.Operand(inputs.matrix(M, K, 1.0, 70, col_outliers=(5, 50.0, 50.0)), True)
    B = inputs.Operand(inputs.matrix(N, K, 0.02, 71), True)
    A, B = (op if kc else inputs.Operand(stored(op.bits, False)[0], False) for op, kc in zip((A, B), layouts))
    say("ragged whole path", (M, N, K), layouts, inputs.STRATEGY_NAMES[strategy])
    ta, tb = (torch.from_numpy(op.bits.view(np.int16)).cuda() for op in (A, B))
    opa = ah.Operand(ta if layouts[0] else ta[:, :M], layouts[0])
    opb = ah.Operand(tb if layouts[1] else tb[:, :N], layouts[1])
    out = ah.adahop_gemm(opa, opb, strategy, 32, k)
    torch.cuda.synchronize()
    bits_a = A.bits if layouts[0] else np.ascontiguousarray(A.bits[:, :M])
    bits_b = B.bits if layouts[1] else np.ascontiguousarray(B.bits[:, :N])
    ref = orc.adahop_gemm(bits_a, layouts[0], bits_b, layouts[1], strategy, 32, k)
    for name in ("a_codes", "a_scales", "b_codes", "b_scales"):
        assert np.array_equal(host(out[name]), ref[name]), name
    g = inputs.Gemm("ragged", inputs.Operand(bits_a, layouts[0]), inputs.Operand(bits_b, layouts[1]), strategy, 32, k)
    check_c(host(out["C"]), ref["C"], g, extracted=ref["idx"] if k else None, tol=1e-5)


def shifted(t, by):
    """The same bytes `by` bytes behind the start of an allocation, which ends with them."""
    room = torch.empty(t.numel() + by, dtype=torch.uint8, device="cuda")
    room[by:] = t.flatten()
    return room[by:].view(t.shape)


SMALL = (7, 8, 9, 10, 11)           # 128 x 128 shallow and deep, 64 x 64, 32 x 64, 32 x 32


@pytest.mark.parametrize("kernel", SMALL)
@pytest.mark.parametrize("shape", [(1, 1, 32), (31, 33, 64), (33, 65, 224), (64, 64, 256), (65, 127, 288), (129, 130, 512),
                                   (96, 1000, 1056), (300, 257, 2304), (130, 640, 4064), (17, 4100, 768), (300, 270, 96),
                                   (131, 261, 992)])
def test_small_tiles(ah, force, kernel, shape):
    """Rows and columns one past and one short of a tile, K from one block over less than a stage to more stages than
    rotate in LDS, an odd and an even count of them, canonical (K % 256 == 0, or up to 1024 at any address) and re-ordered scales, a C
    with a gap behind its rows that must stay as it was; both output types.  The allowance is the one above, plus half a bf16 step."""
    M, N, K = shape
    rng = np.random.default_rng(M + 5 * N + 11 * K)
    a_codes = rng.integers(0, 256, size=(M, K // 2), dtype=np.uint8)
    b_codes = rng.integers(0, 256, size=(N, K // 2), dtype=np.uint8)
    a_scales = rng.integers(117, 137, size=(M, K // 32), dtype=np.uint8)
    b_scales = rng.integers(100, 120, size=(N, K // 32), dtype=np.uint8)
    say("small tiles", kernel, shape)
    force(kernel)
    ref = orc.mx_gemm(a_codes, a_scales, b_codes, b_scales)
    bar = 2.0 ** -20 * np.outer(dequant_norms(a_codes, a_scales), dequant_norms(b_codes, b_scales))
    dev = [torch.from_numpy(t).cuda() for t in (a_codes, a_scales, b_codes, b_scales)]
    off = [dev[0], shifted(dev[1], 1), dev[2], shifted(dev[3], 3)]      # scales at odd addresses
    for dtype, ops in ((torch.float32, dev), (torch.bfloat16, dev), (torch.float32, off)):
        room = torch.full((M + 1, N + 3), 7.0, dtype=dtype, device="cuda")
        ah.adahop_gemm_mx(*ops, Cout=room[:M, :N])
        torch.cuda.synchronize()
        got = host(room.float()).astype(np.float64)
        assert (got[M] == 7.0).all() and (got[:, N:] == 7.0).all()
        step = 0.0 if dtype == torch.float32 else 2.0 ** -8
        assert float((np.abs(got[:M, :N] - ref) - step * np.abs(ref) - bar * (1.0 + step)).max()) <= 0.0


@pytest.mark.parametrize("M,N,K,k", [(1, 1, 32, 0), (95, 63, 224, 0), (97, 65, 288, 0), (96, 64, 768, 0), (193, 129, 2304, 0), (300, 257, 96, 0),
                                     (95, 129, 1120, 70), (97, 200, 2048, 200), (96, 11008, 4096, 0), (384, 4096, 1024, 9)])
def test_96_row_tiles(ah, force, M, N, K, k):
    """The 96 x 64 tiles at their edges, with fewer stages than rotate in LDS and more, with and without K-channels: the sums of the 128 x 128
    tiles in another order, against which the allowance is that of the oracle's tests on the same fp32 accumulation."""
    A = ah.Operand.from_bits(inputs.matrix(M, K, 1.0, 82, col_outliers=(5, 50.0, 50.0)), True)
    B = ah.Operand.from_bits(inputs.matrix(N, K, 0.02, 83), True)
    say("96 x 64 tiles", (M, N, K, k))
    got = {}
    for kernel in (7, 12):
        force(kernel)
        for dtype in (torch.float32, torch.bfloat16):
            room = torch.full((M + 1, N + 3), 7.0, dtype=dtype, device="cuda")
            ah.adahop_gemm(A, B, inputs.IHT_OE_K if k else inputs.IHT, 32, k, Cout=room[:M, :N])
            torch.cuda.synchronize()
            assert bool((room[M] == 7.0).all()) and bool((room[:, N:] == 7.0).all())
            got[kernel, dtype] = room[:M, :N]
    want = got[7, torch.float32].double()
    err = float((got[12, torch.float32].double() - want).norm() / want.norm())
    assert err < 1e-5
    assert torch.equal(got[12, torch.bfloat16], got[12, torch.float32].to(torch.bfloat16))


@pytest.mark.parametrize("M,N,K,chosen", [(610, 1971, 5376, True), (96, 16384, 4096, True), (261, 15506, 7168, False), (191, 23746, 9056, False)])
def test_96_row_tiles_only_one_per_compute_unit(ah, force, M, N, K, chosen):
    """Up to 256 of the 96 x 64 tiles, and above: the chosen kernel's bits are those of the 96 x 64 tiles, whose two waves per part add in an order of
    their own, or not (scaling blocks of very different sizes, so that the sums are rounded)."""
    gen = torch.Generator(device="cuda").manual_seed(M + N)

    def operand(rows):
        sizes = torch.exp2(torch.randint(-12, 13, (rows, K // 32, 1), generator=gen, device="cuda").float())
        return ah.Operand((torch.randn(rows, K // 32, 32, generator=gen, device="cuda") * sizes).view(rows, K).to(torch.bfloat16), True)
    A, B = operand(M), operand(N)
    say("choice of the 96 x 64 tiles", (M, N, K))
    got = {}
    for kernel in (0, 12):
        force(kernel)
        got[kernel] = ah.adahop_gemm(A, B, inputs.IHT, 32)["C"]
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[12]) == chosen
    force(7)
    assert not torch.equal(ah.adahop_gemm(A, B, inputs.IHT, 32)["C"], got[12])


@pytest.mark.parametrize("M,N,K,ld,dtype", [(4250, 8450, 96, 8452, torch.float32), (4250, 8450, 192, 8464, torch.float32),
                                            (8400, 8500, 64, 8501, torch.bfloat16), (6200, 8150, 288, 8192, torch.float32),
                                            (6200, 8150, 480, 8151, torch.float32), (4000, 3900, 32, 3901, torch.float32),
                                            (1930, 3300, 32, 3301, torch.float32), (1800, 3900, 64, 3900, torch.float32),
                                            (3400, 3750, 512, 3752, torch.bfloat16)])
def test_short_products_with_a_large_c(ah, M, N, K, ld, dtype):
    """The orders in which tiles are walked where C is larger than the Infinity Cache (rows of whole pages, of whole 64-byte pieces and of
    neither) and where it is larger than 24 MB, with the 128 x 128 tiles of a single stage of K and of more: rows at every tile's edges against the oracle, and the gap behind
    the rows as it was.  The allowance is the one above, plus half a bf16 step."""
    rng = np.random.default_rng(M + N + K)
    a_codes = rng.integers(0, 256, size=(M, K // 2), dtype=np.uint8)
    b_codes = rng.integers(0, 256, size=(N, K // 2), dtype=np.uint8)
    a_scales = rng.integers(117, 137, size=(M, K // 32), dtype=np.uint8)
    b_scales = rng.integers(100, 120, size=(N, K // 32), dtype=np.uint8)
    say("large C", (M, N, K, ld), dtype)
    room = torch.full((M, ld), 7.0, dtype=dtype, device="cuda")
    ah.adahop_gemm_mx(*(torch.from_numpy(t).cuda() for t in (a_codes, a_scales, b_codes, b_scales)), Cout=room[:, :N])
    torch.cuda.synchronize()
    assert bool((room[:, N:] == 7.0).all())
    rows = np.unique(np.concatenate([np.arange(0, M, 128), np.arange(127, M, 128), [M - 1]]))
    ref = orc.mx_gemm(a_codes[rows], a_scales[rows], b_codes, b_scales)
    bar = 2.0 ** -20 * np.outer(dequant_norms(a_codes[rows], a_scales[rows]), dequant_norms(b_codes, b_scales))
    got = host(room[torch.from_numpy(rows).cuda(), :N].float()).astype(np.float64)
    step = 0.0 if dtype == torch.float32 else 2.0 ** -8
    assert float((np.abs(got - ref) - step * np.abs(ref) - bar * (1.0 + step)).max()) <= 0.0


@pytest.mark.parametrize("M,N,K", [(5001, 4400, 64), (330, 65552, 192), (21000, 1040, 32), (2048, 10304, 128)])
def test_wide_tiles_of_one_stage(ah, force, M, N, K):
    """64 x 256 tiles (fp32, one stage of K, more than 80 MB on the 64-byte grid): the bits of the 128 x 128 ones, which add in the same
    order, with scales from the quantisers and from canonical arrays, remainders of both tile edges, and the gap behind the rows as it was."""
    gen = torch.Generator().manual_seed(M + K)
    A, B = (ah.Operand(torch.randn(n, K, generator=gen).to(torch.bfloat16).cuda(), True) for n in (M, N))
    say("wide tiles", (M, N, K))
    got = {}
    for which in (0, 8):
        force(which)
        room = torch.full((M, N + 16), 7.0, device="cuda")
        r = ah.adahop_gemm(A, B, inputs.IHT, 32, Cout=room[:, :N])
        packed = ah.adahop_gemm_mx(r["a_codes"], r["a_scales"], r["b_codes"], r["b_scales"])
        torch.cuda.synchronize()
        assert bool((room[:, N:] == 7.0).all())
        got[which] = room[:, :N].clone()
        assert torch.equal(packed, got[which])
    assert torch.equal(got[0], got[8])


@pytest.mark.parametrize("kernel", SMALL)
@pytest.mark.parametrize("M,N,K,k", [(40, 70, 96, 9), (96, 264, 1120, 70), (150, 129, 2048, 200)])
def test_small_tiles_with_k_channels(ah, force, kernel, M, N, K, k):
    """One, two and four gathered bf16 stages in front of one to nine FP4 stages, scales written by the quantisers."""
    A = inputs.Operand(inputs.matrix(M, K, 1.0, 80, col_outliers=(5, 50.0, 50.0)), True)
    B = inputs.Operand(inputs.matrix(N, K, 0.02, 81), True)
    say("small tiles with K-channels", kernel, (M, N, K, k))
    force(kernel)
    out = ah.adahop_gemm(*(ah.Operand.from_bits(op.bits, True) for op in (A, B)), inputs.IHT_OE_K, 32, k)
    torch.cuda.synchronize()
    ref = orc.adahop_gemm(A.bits, True, B.bits, True, inputs.IHT_OE_K, 32, k)
    assert np.array_equal(np.sort(host(out["idx"])), ref["idx"])
    check_c(host(out["C"]), ref["C"], inputs.Gemm("small", A, B, inputs.IHT_OE_K, 32, k), extracted=ref["idx"], tol=1e-5)


@pytest.mark.parametrize("kernel", [0, TILE256, DUAL])
@pytest.mark.parametrize("M,N,K,k,gap", [(2305, 1027, 4096, 0, 0), (2048, 2048, 2048, 0, 1), (1024, 1001, 1024, 20, 0),
                                         (300, 130, 2080, 0, 3), (520, 200, 2304, 100, 1)])
def test_bf16_output_of_any_alignment(ah, force, kernel, M, N, K, k, gap):
    """Widths and row strides that are no multiples of 16 bytes: the bits of the fp32 product rounded to nearest even.  Chosen by shape
    these products are taken by small tiles for either type; with the two-set kernel forced, which stores bf16 in pairs, the bf16 product with
    other rows goes to the 256 x 256 tiles, or with N < 256 to 128 x 128 tiles, and is compared with the fp32 product of the two-set kernel."""
    A = ah.Operand.from_bits(inputs.matrix(M, K, 1.0, 90, col_outliers=(5, 50.0, 50.0)), True)
    B = ah.Operand.from_bits(inputs.matrix(N, K, 0.02, 91), True)
    say("bf16 output of any alignment", kernel, (M, N, K, k, gap))
    force(kernel)
    strategy = inputs.IHT_OE_K if k else inputs.IHT
    full = ah.adahop_gemm(A, B, strategy, 32, k)["C"].to(torch.bfloat16)
    room = torch.full((M, N + gap), 7.0, dtype=torch.bfloat16, device="cuda")
    ah.adahop_gemm(A, B, strategy, 32, k, Cout=room[:, :N])
    torch.cuda.synchronize()
    assert torch.equal(room[:, :N].view(torch.int16), full.view(torch.int16))
    assert bool((room[:, N:] == 7.0).all())


@pytest.mark.parametrize("kernel", [TILE256, DUAL])
@pytest.mark.parametrize("M,N,K,k", [(520, 520, 2048, 0), (300, 264, 2080, 20)])
def test_rows_of_c_at_any_alignment(ah, force, kernel, M, N, K, k):
    """Rows of C that are whole 64-byte pieces (streamed) and that begin at 32, 16 and 4 (bf16: 2) bytes, or all of them behind
    such a first element: the bits of a C without gaps, and the gaps as they were."""
    A = ah.Operand.from_bits(inputs.matrix(M, K, 1.0, 92, col_outliers=(5, 50.0, 50.0)), True)
    B = ah.Operand.from_bits(inputs.matrix(N, K, 0.02, 93), True)
    strategy = inputs.IHT_OE_K if k else inputs.IHT
    force(kernel)
    for dtype in (torch.float32, torch.bfloat16):
        want = ah.adahop_gemm(A, B, strategy, 32, k, Cout=torch.empty((M, N), dtype=dtype, device="cuda"))["C"]
        for ld, first in ((576, 0), (584, 0), (580, 0), (577, 0), (576, 8), (576, 4), (576, 1)):
            say("rows of C", kernel, (M, N, K, k), dtype, ld, first)
            room = torch.full((M * ld + first,), 7.0, dtype=dtype, device="cuda")
            C = room[first:].view(M, ld)
            ah.adahop_gemm(A, B, strategy, 32, k, Cout=C[:, :N])
            torch.cuda.synchronize()
            assert torch.equal(C[:, :N], want), (dtype, ld, first)
            assert bool((C[:, N:] == 7.0).all()) and bool((room[:first] == 7.0).all())


@pytest.mark.parametrize("M,N,K,k", [(256, 128, 2048, 8), (520, 264, 2080, 100), (1000, 650, 2304, 128), (4352, 4100, 2048, 70)])
def test_two_set_kernel_with_k_channels(ah, force, M, N, K, k):
    """One and two gathered bf16 stages in front of eight and more FP4 stages, one tile and several (both accumulator sets)
    per workgroup: the bits of the 256 x 256 kernel, which adds in the same order (and is compared with the oracle elsewhere)."""
    A = ah.Operand.from_bits(inputs.matrix(M, K, 1.0, 95, col_outliers=(5, 50.0, 50.0)), True)
    B = ah.Operand.from_bits(inputs.matrix(N, K, 0.02, 96), True)
    say("two accumulator sets with K-channels", (M, N, K, k))
    force(DUAL)
    got = ah.adahop_gemm(A, B, inputs.IHT_OE_K, 32, k)["C"]
    force(TILE256 if N >= 256 else 8)
    want = ah.adahop_gemm(A, B, inputs.IHT_OE_K, 32, k)["C"]
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))


@pytest.mark.parametrize("M,N,K,k,gap", [(256, 128, 2048, 0, 0), (300, 130, 1824, 0, 2), (513, 386, 2080, 20, 6), (1000, 650, 2304, 128, 0),
                                         (4352, 4098, 2048, 70, 30), (2560, 7936, 2048, 0, 0)])
def test_two_set_kernel_with_bf16_output(ah, force, M, N, K, k, gap):
    """Pairs of columns from the accumulators of neighbouring lanes, with none, one and two bf16 stages, one tile and several (both
    accumulator sets) per workgroup, streamed rows and others: the kernel's own fp32 sums rounded to nearest even."""
    A = ah.Operand.from_bits(inputs.matrix(M, K, 1.0, 97, col_outliers=(5, 50.0, 50.0)), True)
    B = ah.Operand.from_bits(inputs.matrix(N, K, 0.02, 98), True)
    say("two accumulator sets, bf16", (M, N, K, k, gap))
    force(DUAL)
    strategy = inputs.IHT_OE_K if k else inputs.IHT
    want = ah.adahop_gemm(A, B, strategy, 32, k)["C"].to(torch.bfloat16)
    room = torch.full((M, N + gap), 7.0, dtype=torch.bfloat16, device="cuda")
    ah.adahop_gemm(A, B, strategy, 32, k, Cout=room[:, :N])
    torch.cuda.synchronize()
    assert torch.equal(room[:, :N].view(torch.int16), want.view(torch.int16))
    assert bool((room[:, N:] == 7.0).all())
