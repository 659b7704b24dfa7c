"""Edge cases of the GPU path against the oracle (run with -m gpu): smallest shapes, everything extracted,
all-zero and extreme-magnitude operands, and operands at the documented size limits."""
import numpy as np
import pytest

from oracle import reference as orc
from paper_2604_02525_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def say(*a):
    print("[case]", *a, flush=True)


@pytest.fixture(scope="module")
def ah():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_02525_amd import binding
    binding.lib()
    return binding


def host(t):
    return t.cpu().numpy()


def bf16(x):
    return torch.from_numpy(np.asarray(x, dtype=np.float32)).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)


def stored(logical, k_contig):
    """Device operand for logical [outer, K] bits; a K-strided array narrower than 8 is padded to ld = 8."""
    a = logical if k_contig else np.ascontiguousarray(logical.T)
    pad = (-a.shape[1]) % 8
    if pad:
        wide = np.zeros((a.shape[0], a.shape[1] + pad), dtype=np.uint16)
        wide[:, :a.shape[1]] = a
        return torch.from_numpy(wide.view(np.int16)).cuda()[:, :a.shape[1]], a
    return torch.from_numpy(a.view(np.int16)).cuda(), a


def whole(ah, A_log, B_log, a_kc, b_kc, strategy, b, k):
    ta, sa = stored(A_log, a_kc)
    tb, sb = stored(B_log, b_kc)
    out = ah.adahop_gemm(ah.Operand(ta, a_kc), ah.Operand(tb, b_kc), strategy, b, k)
    torch.cuda.synchronize()
    ref = orc.adahop_gemm(sa, a_kc, sb, b_kc, strategy, b, k)
    for name in ("a_scales", "b_scales", "a_codes", "b_codes"):
        assert np.array_equal(host(out[name]), ref[name]), name
    if k:
        assert np.array_equal(np.sort(host(out["idx"])), ref["idx"])
    got = host(out["C"]).astype(np.float64)
    den = max(np.linalg.norm(ref["C"]), 1e-300)
    assert np.linalg.norm(got - ref["C"]) / den < 1e-3 or np.array_equal(got, ref["C"])
    return got, ref


@pytest.mark.parametrize("layouts", [(True, True), (True, False), (False, False)])
def test_smallest_shapes(ah, layouts):
    rng = np.random.default_rng(1)
    for M, N, K, b in ((1, 1, 32, 32), (1, 9, 64, 32), (7, 1, 32, 0), (3, 5, 256, 256)):
        A = bf16(rng.standard_normal((M, K)))
        B = bf16(rng.standard_normal((N, K)) * 0.02)
        for strategy in ((inputs.NONE, inputs.IHT) if b else (inputs.NONE,)):
            say("smallest", (M, N, K), layouts, inputs.STRATEGY_NAMES[strategy])
            whole(ah, A, B, layouts[0], layouts[1], strategy, b, 0)


@pytest.mark.parametrize("layouts", [(True, True), (True, False), (False, True), (False, False)])
def test_smallest_shapes_with_extraction(ah, layouts):
    """One extracted row / column / K-channel (and all but one of them) on operands far smaller than any tile of the
    BF16 product kernels: a single workgroup whose loads past the last row repeat that row, a K of half a pipeline
    stage, a long side of one row."""
    rng = np.random.default_rng(4)
    for M, N, K in ((1, 1, 32), (1, 9, 64), (7, 1, 32), (3, 5, 256), (9, 17, 96), (260, 3, 160)):
        A = bf16(rng.standard_normal((M, K)) * np.where(rng.random((M, 1)) < 0.3, 50.0, 1.0))
        B = bf16(rng.standard_normal((N, K)) * 0.02)
        for strategy, dim in ((inputs.IHT_OE_ROW, M), (inputs.IHT_OE_COL, N), (inputs.IHT_OE_K, K)):
            for k in sorted({1, max(dim - 1, 1)}):
                say("smallest with extraction", (M, N, K), layouts, inputs.STRATEGY_NAMES[strategy], k)
                whole(ah, A, B, layouts[0], layouts[1], strategy, 32, k)


@pytest.mark.parametrize("layouts", [(True, True), (False, False)])
def test_everything_extracted_is_the_bf16_product(ah, layouts):
    """k equal to the whole extracted dimension: the residual is all zero (codes 0, scales 0) and C is the BF16 product
    of the original operands -- bf16 x bf16 with fp32 accumulation, compared with the exact product."""
    rng = np.random.default_rng(2)
    M, N, K = 40, 24, 96
    A = bf16(rng.standard_normal((M, K)))
    B = bf16(rng.standard_normal((N, K)))
    exact = orc.exact_gemm(A if layouts[0] else np.ascontiguousarray(A.T), layouts[0],
                           B if layouts[1] else np.ascontiguousarray(B.T), layouts[1])
    for strategy, k in ((inputs.IHT_OE_ROW, M), (inputs.IHT_OE_COL, N), (inputs.IHT_OE_K, K)):
        say("all extracted", inputs.STRATEGY_NAMES[strategy], layouts)
        got, ref = whole(ah, A, B, layouts[0], layouts[1], strategy, 32, k)
        masked = {inputs.IHT_OE_ROW: ("a",), inputs.IHT_OE_COL: ("b",), inputs.IHT_OE_K: ("a", "b")}[strategy]
        for side in masked:
            assert not ref[side + "_codes"].any() and not ref[side + "_scales"].any()
        assert np.linalg.norm(got - exact) / np.linalg.norm(exact) < 1e-5


def test_all_zero_and_signed_zero_operands(ah):
    M, N, K = 33, 17, 128
    Z = np.zeros((M, K), dtype=np.uint16)
    NZ = np.full((M, K), 0x8000, dtype=np.uint16)                        # -0.0 everywhere
    B = bf16(np.random.default_rng(3).standard_normal((N, K)))
    for name, A in (("zeros", Z), ("negative zeros", NZ)):
        for strategy, k in ((inputs.NONE, 0), (inputs.IHT, 0), (inputs.IHT_OE_ROW, 3), (inputs.IHT_OE_K, 5)):
            say(name, inputs.STRATEGY_NAMES[strategy])
            got, ref = whole(ah, A, B, True, True, strategy, 64, k)
            assert not got.any() and not ref["a_scales"].any()


@pytest.mark.parametrize("k_contig", [True, False])
@pytest.mark.parametrize("b", [0, 32, 256])
def test_extreme_magnitudes_quantise_bit_exact(ah, b, k_contig):
    """Blocks whose amax spans the whole bf16 range, from subnormals to the largest finite value: scale codes from 0
    to 252 (and the transform's sums stay finite: each 32-block holds one large value among tiny ones)."""
    rng = np.random.default_rng(4)
    outer, K = 96, 512
    x = rng.standard_normal((outer, K)).astype(np.float32) * 1e-3
    expo = rng.integers(-126, 120, size=(outer, K // 32))
    x[:, ::32] = np.ldexp(rng.uniform(1.0, 1.99, (outer, K // 32)).astype(np.float32), expo) * rng.choice([-1, 1], (outer, K // 32))
    x[0, :32] = np.float32(2.0 ** -133)                                  # a block of bf16 subnormals
    x[1, 0] = np.float32(3.38e38) if b == 0 else np.float32(1e30)        # near the largest finite bf16
    bits = bf16(x)
    t, s = stored(bits, k_contig)
    say("extreme magnitudes", b, k_contig)
    codes, scales = ah.adahop_iht_quantize(ah.Operand(t, k_contig), b)
    torch.cuda.synchronize()
    rc, rs = orc.iht_quantize(s, k_contig, b)
    assert np.array_equal(host(scales), rs) and np.array_equal(host(codes), rc)
    if b == 0:                                                            # (a transform spreads the large values over its block)
        assert rs.min() == 0 and rs.max() >= 240


def test_operands_at_the_size_limits(ah):
    """outer = 2^21 (the documented maximum) with the shortest K, and a long-K operand: every byte against the oracle;
    FOID over 2^21 indices."""
    rng = np.random.default_rng(5)
    outer = 1 << 21
    x = torch.randn((outer, 32), generator=torch.Generator().manual_seed(11)).to(torch.bfloat16)
    x[rng.integers(0, outer, 50)] *= 30.0
    bits = x.view(torch.int16).numpy().view(np.uint16)
    for kc, arr in ((True, bits), (False, np.ascontiguousarray(bits.T))):
        say("outer = 2^21", "K-contiguous" if kc else "K-strided")
        op = ah.Operand(torch.from_numpy(arr.view(np.int16)).cuda(), kc)
        codes, scales = ah.adahop_iht_quantize(op, 32)
        torch.cuda.synchronize()
        rc, rs = orc.iht_quantize(arr, kc, 32)
        assert np.array_equal(host(scales), rs) and np.array_equal(host(codes), rc)
        del codes, scales
        idx, mask, _ = ah.adahop_foid_topk(op, 0, 1000)
        torch.cuda.synchronize()
        ri, rm = orc.foid_topk(arr, kc, 0, 1000)
        assert np.array_equal(host(idx), ri) and np.array_equal(host(mask), rm)
        del op
    torch.cuda.empty_cache()
    K = 1 << 21
    y = torch.randn((24, K), generator=torch.Generator().manual_seed(12)).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
    for kc, arr in ((True, y), (False, np.ascontiguousarray(y.T))):
        say("K = 2^21", "K-contiguous" if kc else "K-strided")
        op = ah.Operand(torch.from_numpy(arr.view(np.int16)).cuda(), kc)
        codes, scales = ah.adahop_iht_quantize(op, 256)
        torch.cuda.synchronize()
        rc, rs = orc.iht_quantize(arr, kc, 256)
        assert np.array_equal(host(scales), rs) and np.array_equal(host(codes), rc)
        idx, mask, _ = ah.adahop_foid_topk(op, 1, 4096)                 # K-channels, scored over the first 24 rows
        torch.cuda.synchronize()
        ri, rm = orc.foid_topk(arr, kc, 1, 4096)
        assert np.array_equal(host(idx), ri) and np.array_equal(host(mask), rm)
    torch.cuda.empty_cache()


@pytest.mark.parametrize("rows", [1, 3, 17, 70])
@pytest.mark.parametrize("K", [224, 256, 1824, 2048, 3840, 3872, 4096, 4128, 4352, 8192, 8224, 12320])
def test_units_of_long_and_short_rows(ah, rows, K):
    """K-contiguous quantiser on both sides of rows that are one workgroup (16 units of 256), with rows that share one and rows that
    span several; masked rows and K-indices; rounded to nearest and stochastically."""
    x = inputs.matrix(rows, K, 1.0, 9600, row_outliers=(1, 40.0, 40.0))
    op = ah.Operand.from_bits(x, True)
    rng = np.random.default_rng(rows + K)
    zo, zk = (rng.random(rows) < 0.2).astype(np.uint8), (rng.random(K) < 0.1).astype(np.uint8)
    for b in (0, 32):
        for mo, mk in ((None, None), (zo, zk)):
            for seed in (None, 11):
                codes, scales = ah.adahop_iht_quantize(op, b, zero_outer=None if mo is None else torch.from_numpy(mo).cuda(),
                                                       zero_k=None if mk is None else torch.from_numpy(mk).cuda(), sr_seed=seed)
                rc, rs = orc.iht_quantize(x, True, b, mo, mk, sr_seed=seed)
                assert np.array_equal(host(scales), rs) and np.array_equal(host(codes), rc), (b, mo is not None, seed)


def test_units_counted_beyond_the_one_multiplication(ah):
    """Rows x units x units of 2^32 and more: numbered row by row; the same bits as in two halves, which are numbered consecutively."""
    rows, K = 300, 1 << 20
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(rows, K, generator=gen, device="cuda", dtype=torch.bfloat16)
    codes, scales = ah.adahop_iht_quantize(ah.Operand(x, True), 64)
    for at in (0, 150):
        c, s = ah.adahop_iht_quantize(ah.Operand(x[at:at + 150], True), 64)
        assert torch.equal(c, codes[at:at + 150]) and torch.equal(s, scales[at:at + 150])


@pytest.mark.parametrize("outer,K,pad", [(500, 4096, 0), (1023, 4096, 8), (1024, 4096, 0), (1030, 4096, 8), (1030, 4064, 0), (1030, 3840, 0)])
@pytest.mark.parametrize("block", [0, 32])
def test_rows_of_exactly_one_workgroup(ah, outer, K, pad, block):
    """K-contiguous rows of 16 units, of whole ones and with a shorter last one, and of 15, numbered row by row and over all rows: the bytes of the
    same matrix stored K-strided; rows and K-channels masked, rounded to nearest and stochastically."""
    gen = torch.Generator(device="cuda").manual_seed(outer * K + pad)
    x = torch.full((outer, K + pad), float("nan"), dtype=torch.bfloat16, device="cuda")
    x[:, :K] = torch.randn(outer, K, generator=gen, device="cuda")
    t = torch.zeros(K, (outer + 7) // 8 * 8, dtype=torch.bfloat16, device="cuda")
    t[:, :outer] = x[:, :K].t()
    zk, zo = torch.zeros(K, dtype=torch.uint8, device="cuda"), torch.zeros(outer, dtype=torch.uint8, device="cuda")
    zk[[0, K // 2, K - 1]] = 1
    zo[[0, outer // 2, outer - 1]] = 1
    say("rows of one workgroup", outer, K, pad, block)
    for kw in ({}, {"zero_k": zk}, {"zero_outer": zo}, {"sr_seed": 5}):
        got, want = (ah.adahop_iht_quantize(op, block, **kw) for op in (ah.Operand(x[:, :K], True), ah.Operand(t[:, :outer], False)))
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), list(kw)


@pytest.mark.parametrize("outer,K", [(40, 32), (72, 320), (1000, 2336), (1032, 2336), (4160, 8192), (8200, 4352), (29992, 512), (6976, 7712)])
@pytest.mark.parametrize("block", [0, 32])
def test_orders_of_the_workgroups_of_a_k_strided_operand(ah, outer, K, block):
    """Whole groups of 16 column tiles, a last group of one and of several, none at all, workgroups that are a multiple of eight and not, up to and
    beyond the count that keeps the plain order, rows on 128-byte lines and off them: the bytes of the same matrix stored K-contiguous, whose
    kernel numbers its work otherwise, with an extracted column and K-channels masked as well."""
    gen = torch.Generator(device="cuda").manual_seed(outer + K)
    x = torch.randn(outer, K, generator=gen, device="cuda").to(torch.bfloat16)
    t = x.t().contiguous()
    say("K-strided order", outer, K, block)
    idx = torch.tensor([0, K // 2, K - 1], dtype=torch.int32, device="cuda")
    for strategy, kw in ((inputs.IHT if block else inputs.NONE, {}), (inputs.IHT_OE_K, dict(k=3, idx=idx)) if block else (inputs.NONE, {})):
        want, got = (ah.adahop_pack_operand(op, True, strategy, block, **kw) for op in (ah.Operand(x, True), ah.Operand(t, False)))
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("outer,K,pad,block", [
    (outer, K, pad, block) for outer, K, pad in [(64, 256, 0), (63, 256, 1), (65, 288, 7), (128, 224, 8), (200, 768, 0), (192, 1056, 64), (328, 2048, 24)]
    for block in (0, 32, 128, 256) if not block or K % block == 0])
def test_tiles_of_a_k_strided_operand_at_and_off_its_edges(ah, outer, K, pad, block):
    """Tiles of 256 K x 64 columns that lie inside the operand as a whole and ones that do not, rows with and without a gap behind them, K-channels
    and columns masked, rounded to nearest and stochastically: the bytes of the same matrix stored K-contiguous."""
    gen = torch.Generator(device="cuda").manual_seed(outer * K + pad)
    x = torch.randn(outer, K, generator=gen, device="cuda").to(torch.bfloat16)
    wide = torch.full((K, (outer + pad + 7) // 8 * 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    wide[:, :outer] = x.t()
    ops = (ah.Operand(x, True), ah.Operand(wide[:, :outer], False))
    zk, zo = torch.zeros(K, dtype=torch.uint8, device="cuda"), torch.zeros(outer, dtype=torch.uint8, device="cuda")
    zk[[0, K // 2, K - 1]] = 1
    zo[[0, outer // 2, outer - 1]] = 1
    say("K-strided tiles", outer, K, pad, block)
    for kw in ({}, {"zero_k": zk}, {"zero_outer": zo}, {"sr_seed": 5}):
        want, got = (ah.adahop_iht_quantize(op, block, **kw) for op in ops)
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), list(kw)


@pytest.mark.parametrize("K,at,k", [(32, 0, 32), (64, 63, 1), (288, 4, 280), (512, 255, 2), (768, 250, 270), (4096, 512, 300), (8192, 0, 1), (8192, 8191, 1), (8192, 4090, 17),
                                    (3040, 300, 2500), (11008, 6000, 4096), (9000 // 32 * 32, 0, 257)])
def test_runs_of_k_channels_copied_by_the_quantisers(ah, K, at, k):
    """The extracted K-channels next to each other: units of 256 with none of them, a few, more than 16 and nothing else, before, between and behind the
    units with any, lists of one entry up to the longest that the quantisers take; several rows per workgroup and several passes.  Codes, scales, and C
    as with the same indices handed in, where the mask and the separate gather are used; and codes of zero where all of a block is extracted."""
    M, N, b = 37, 70, 32
    gen = torch.Generator(device="cuda").manual_seed(K + k)
    A = torch.randn(M, K, generator=gen, device="cuda")
    A[:, at:at + k] *= 100.0
    A, B = A.to(torch.bfloat16), torch.randn(N, K, generator=gen, device="cuda").to(torch.bfloat16)
    say("runs of K-channels", K, at, k)
    opa, opb = ah.Operand(A, True), ah.Operand(B, True)
    out = ah.adahop_gemm(opa, opb, inputs.IHT_OE_K, b, k)
    got = {n: out[n].clone() for n in ("C", "idx", "a_codes", "a_scales", "b_codes", "b_scales")}
    again = ah.adahop_gemm(opa, opb, inputs.IHT_OE_K, b, k, idx=got["idx"].clone())
    torch.cuda.synchronize()
    assert torch.equal(got["idx"], torch.arange(at, at + k, dtype=torch.int32, device="cuda"))
    for name, t in got.items():
        assert torch.equal(t, again[name]), name
    first, last = -(-at // b), (at + k) // b
    assert not got["a_codes"][:, first * b // 2:max(first, last) * b // 2].any() and not got["b_codes"][:, first * b // 2:max(first, last) * b // 2].any()


@pytest.mark.parametrize("outer,K,axis", [(1, 64, 1), (2, 288, 1), (45, 512, 1), (63, 320, 1), (65, 320, 1), (300, 32, 0), (72, 64, 0)])
@pytest.mark.parametrize("k_contig", [True, False])
def test_scores_of_few_samples(ah, outer, K, axis, k_contig):
    """Fewer than 64 samples per scored index (and 64), along the rows of the stored array and across them: the oracle's scores bit for bit."""
    rng = np.random.default_rng(outer + K)
    bits = bf16(rng.standard_normal((outer, K)) * np.exp(rng.standard_normal((outer, K))))
    t, a = stored(bits, k_contig)
    say("scores of few samples", outer, K, axis, k_contig)
    k = max((outer if axis == 0 else K) // 5, 1)
    idx, mask, scores = ah.adahop_foid_topk(ah.Operand(t, k_contig), axis, k)
    torch.cuda.synchronize()
    want = orc.foid_scores(a, k_contig, axis)
    assert np.array_equal(host(scores).view(np.uint32), want.view(np.uint32))
    assert np.array_equal(host(idx), np.flatnonzero(host(mask)))


@pytest.mark.parametrize("M,N,K,k", [(8, 63, 64, 3), (65, 200, 288, 64), (1000, 72, 1056, 65), (129, 4104, 2048, 200)])
@pytest.mark.parametrize("a_kc,b_kc", [(False, False), (True, False), (False, True)])
@pytest.mark.parametrize("given,sr", [(False, False), (True, False), (False, True)])
def test_k_channels_of_k_strided_operands_copied_beside_their_tiles(ah, M, N, K, k, a_kc, b_kc, given, sr):
    """The copies of K-strided operands (by workgroups ahead of their tiles) and of K-contiguous ones give the same product, indices selected and handed
    in, rounded to nearest and stochastically: ragged outer sizes, one to four groups of 64 channels."""
    gen = torch.Generator(device="cuda").manual_seed(M * N + k)
    A = torch.randn(M, K, generator=gen, device="cuda")
    A[:, torch.randperm(K, generator=gen, device="cuda")[:k]] *= 50.0
    A, B = A.to(torch.bfloat16), torch.randn(N, K, generator=gen, device="cuda").to(torch.bfloat16)
    say("K-channels beside the tiles", (M, N, K), k, a_kc, b_kc, given, sr)

    def strided(x):
        wide = torch.zeros((K, (x.shape[0] + 7) // 8 * 8), dtype=torch.bfloat16, device="cuda")
        wide[:, :x.shape[0]] = x.t()
        return ah.Operand(wide[:, :x.shape[0]], False)

    kw = {"sr_seed_a": 11} if sr else {}
    want = ah.adahop_gemm(ah.Operand(A, True), ah.Operand(B, True), inputs.IHT_OE_K, 32, k, **kw)
    keep = {n: want[n].clone() for n in ("C", "idx", "a_codes", "b_codes", "a_scales", "b_scales")}
    if given:
        kw["idx"] = keep["idx"].clone()
    got = ah.adahop_gemm(ah.Operand(A, True) if a_kc else strided(A), ah.Operand(B, True) if b_kc else strided(B), inputs.IHT_OE_K, 32, k, **kw)
    torch.cuda.synchronize()
    for n, t in keep.items():
        assert torch.equal(got[n], t), n
