"""Row / column extraction whose bf16 products are formed by the quantiser of the K-strided operand: against the oracle, and the
extracted rows / columns against fp64 products, at the edges of its tiles (64 columns, 256 K-elements, 16 extracted rows)."""
import numpy as np
import pytest

from oracle import reference as orc
from paper_2604_02525_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def bits(rng, outer, K, rows):
    """bf16 bits of an [outer, K] operand, some rows amplified."""
    x = rng.standard_normal((outer, K)).astype(np.float32)
    x[rng.permutation(outer)[:rows]] *= 30.0
    return torch.from_numpy(x).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)


def values(b):
    return (b.astype(np.uint32) << 16).view(np.float32).astype(np.float64)


def operand(ah, logical, k_contig, pad):
    """(device operand with `pad` elements more per stored row, all NaN; the stored array for the oracle)"""
    a = logical if k_contig else np.ascontiguousarray(logical.T)
    wide = np.full((a.shape[0], (a.shape[1] + 7) // 8 * 8 + pad), 0x7FC0, dtype=np.uint16)
    wide[:, :a.shape[1]] = a
    return ah.Operand(torch.from_numpy(wide.view(np.int16)).cuda()[:, :a.shape[1]], k_contig), a


# (extracted operand's rows, the other's, K, k, block, extracted operand K-contiguous)
CASES = [
    (40, 64, 32, 1, 32, True),          # one tile, an eighth of its K
    (64, 65, 256, 16, 256, True),       # a whole tile and one column of the next
    (97, 200, 288, 17, 32, True),       # second tile of 32 K-elements, second tile of rows with one row
    (130, 72, 544, 33, 32, True),
    (200, 136, 1024, 64, 128, True),
    (300, 1000, 1056, 96, 32, True),    # the most rows; columns that end inside a 16-byte piece
    (300, 256, 512, 97, 64, True),      # one more: the separate kernel
    (5000, 512, 4096, 48, 128, True),
    (64, 12808, 256, 5, 128, True),     # rows off the 128-byte lines: an order of the column tiles of their own
    (100, 12801, 512, 20, 256, False),
    (1030, 4100, 1312, 49, 32, False),
    (72, 20000, 32, 3, 32, False),
    (9000, 8192, 512, 90, 64, False),   # selection too wide to stand beside a K-strided operand
]


@pytest.mark.parametrize("short,long,K,k,block,short_kc", CASES)
@pytest.mark.parametrize("strategy", [inputs.IHT_OE_ROW, inputs.IHT_OE_COL])
def test_products_on_the_way(short, long, K, k, block, short_kc, strategy, long_kc=False):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_02525_amd import binding as ah
    print("[case]", short, long, K, k, block, short_kc, strategy, flush=True)
    rng = np.random.default_rng(short + long + K + k)
    row = strategy == inputs.IHT_OE_ROW
    S, L = bits(rng, short, K, k), bits(rng, long, K, 2)
    (s, s_st), (l, l_st) = operand(ah, S, short_kc, 8), operand(ah, L, long_kc, 16)
    A, B, a_st, b_st = (s, l, s_st, l_st) if row else (l, s, l_st, s_st)
    out = ah.adahop_gemm(A, B, strategy, block, k)
    torch.cuda.synchronize()
    small = short * long * K < 1 << 31
    idx = np.sort(out["idx"].cpu().numpy())
    mask = np.zeros(short, dtype=np.uint8)
    mask[idx] = 1
    assert len(set(idx.tolist())) == k and np.array_equal(out["mask"].cpu().numpy(), mask)
    ref = orc.adahop_gemm(a_st, A.k_contig, b_st, B.k_contig, strategy, block, k) if small else None
    if ref:
        assert np.array_equal(idx, ref["idx"])
        for name in ("a_codes", "b_codes", "a_scales", "b_scales"):
            assert np.array_equal(out[name].cpu().numpy(), ref[name]), name
    codes, scales = (out["a_codes"], out["a_scales"]) if row else (out["b_codes"], out["b_scales"])
    # the same bits with the indices handed in, and with the other operand packed beforehand
    other = {"b_packed" if row else "a_packed": ah.adahop_pack_operand(l, row, strategy, block)}
    for again in (ah.adahop_gemm(A, B, strategy, block, k, idx=out["idx"].clone()), ah.adahop_gemm(A, B, strategy, block, k, **other)):
        assert torch.equal(again["C"].view(torch.int32), out["C"].view(torch.int32))
    assert not codes.cpu().numpy()[idx].any() and not scales.cpu().numpy()[idx].any()
    C = out["C"].cpu().numpy().astype(np.float64)
    got = C[idx] if row else C[:, idx].T
    a, b = values(S[idx]), values(L)
    # products of bf16 values are exact in fp32; a sum of K of them in fp32, in any order, is off by at most K 2^-24 of the sum of magnitudes
    assert (np.abs(got - a @ b.T) <= K * 2.0 ** -24 * (np.abs(a) @ np.abs(b).T)).all()
    if ref:
        rest = np.delete(C - ref["C"], idx, axis=0 if row else 1)
        assert np.linalg.norm(rest) <= 1e-3 * np.linalg.norm(np.delete(ref["C"], idx, axis=0 if row else 1))


@pytest.mark.parametrize("short,long,K,k,block,short_kc", CASES + [
    (70, 127, 96, 33, 32, True), (70, 63, 2048, 9, 256, False), (600, 191, 4416, 70, 64, True),
    # an operand that is streamed past the caches, 16 .. 96 extracted rows
    (300, 20504, 4128, 5, 32, True), (300, 20504, 4352, 17, 64, True), (300, 20504, 4352, 33, 128, True), (300, 20504, 4352, 49, 256, True),
    (300, 20504, 4352, 90, 256, True), (300, 20488, 4352, 96, 64, False), (300, 20504, 4352, 16, 256, False), (300, 20504, 4352, 32, 128, False),
    (300, 20504, 4352, 48, 64, False), (300, 20504, 4352, 64, 32, False), (300, 20504, 4352, 65, 128, True),
])
@pytest.mark.parametrize("strategy", [inputs.IHT_OE_ROW, inputs.IHT_OE_COL])
def test_products_on_the_way_of_a_k_contiguous_operand(short, long, K, k, block, short_kc, strategy):
    """The same by the quantiser of a K-contiguous operand (tiles of 64 rows x 256 K-elements)."""
    test_products_on_the_way(short, long, K, k, block, short_kc, strategy, long_kc=True)


@pytest.mark.parametrize("sr", ["short", "long"])
def test_rounding_option(sr):
    """A stochastically rounded operand: extracted rows still count as zero, and the products of a rounded long operand are formed
    by themselves."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_02525_amd import binding as ah
    print("[case] rounding", sr, flush=True)
    rng = np.random.default_rng(7)
    S, L = bits(rng, 300, 544, 9), bits(rng, 264, 544, 0)
    (s, _), (l, _) = operand(ah, S, True, 0), operand(ah, L, False, 0)
    out = ah.adahop_gemm(s, l, inputs.IHT_OE_ROW, 32, 9, **{"sr_seed_a" if sr == "short" else "sr_seed_b": 77})
    idx = np.sort(out["idx"].cpu().numpy())
    zero = torch.zeros(300, dtype=torch.uint8)
    zero[torch.from_numpy(idx).long()] = 1
    for op, key, z, seed in ((s, "a", zero.cuda(), 77 if sr == "short" else None), (l, "b", None, 77 if sr == "long" else None)):
        codes, scales = ah.adahop_iht_quantize(op, 32, zero_outer=z, sr_seed=seed)
        assert torch.equal(codes, out[key + "_codes"]) and torch.equal(scales, out[key + "_scales"])
    a, b = values(S[idx]), values(L)
    assert (np.abs(out["C"].cpu().numpy()[idx] - a @ b.T) <= 544 * 2.0 ** -24 * (np.abs(a) @ np.abs(b).T)).all()


# More than 32 Mi elements, where the products of a packed or rounded operand are formed after the MXFP4 product: slices of two or three blocks
# (the quantiser's kernel without the quantisation), and longer ones (k_outlier_products: 32, 64 and 96 rows; 128 and 256 columns
# per workgroup; columns that end inside a workgroup's, and inside a 16-byte piece; K-elements that end inside a block).
@pytest.mark.parametrize("short,long,K,k,short_kc", [
    (96, 8200, 4128, 5, True), (330, 4160, 8224, 17, False), (300, 8251, 4128, 90, True), (64, 4096, 8224, 60, True), (90, 1088, 31008, 30, False),
    (64, 12801, 8224, 17, True), (64, 16384, 8192, 32, False), (80, 16377, 8032, 1, True),          # 32 rows: 128, 256 and 256 columns
    (200, 33000, 1056, 40, False), (96, 11000, 9248, 33, True), (96, 14337, 5152, 64, True), (96, 20008, 4320, 64, False),  # 64: 128, 128, 256, 256
    (120, 28681, 4128, 90, False), (100, 5000, 28704, 96, True), (96, 33100, 1184, 65, True)])      # 96
@pytest.mark.parametrize("strategy", [inputs.IHT_OE_ROW, inputs.IHT_OE_COL])
def test_same_bits_whoever_packs_the_other_operand(short, long, K, k, short_kc, strategy, long_kc=False):
    """Extracted rows / columns of a call that quantises both operands, of one with the other operand packed beforehand, of one that
    rounds it stochastically, and of the bf16 product by itself."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_02525_amd import binding as ah
    print("[case] packed", short, long, K, k, short_kc, strategy, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(short + long + K)

    def stored(outer, k_contig, rows):
        x = torch.randn(outer, K, generator=gen, device="cuda")
        x[torch.randperm(outer, generator=gen, device="cuda")[:rows]] *= 30.0
        x = x if k_contig else x.T
        wide = torch.full((x.shape[0], (x.shape[1] + 7) // 8 * 8 + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
        wide[:, :x.shape[1]] = x
        return ah.Operand(wide[:, :x.shape[1]], k_contig)
    s, l = stored(short, short_kc, k), stored(long, long_kc, 2)
    at = l.tensor.T if long_kc else l.tensor    # [K, long]
    assert long * K > 32 << 20
    row = strategy == inputs.IHT_OE_ROW
    A, B = (s, l) if row else (l, s)
    packed, seed = ("b_packed", "sr_seed_b") if row else ("a_packed", "sr_seed_a")
    want = ah.adahop_gemm(A, B, strategy, 32, k)
    idx = want["idx"].clone()
    given = {packed: ah.adahop_pack_operand(l, row, strategy, 32)}
    for again in (ah.adahop_gemm(A, B, strategy, 32, k, **given), ah.adahop_gemm(A, B, strategy, 32, k, idx=idx, **given)):
        assert torch.equal(again["idx"], idx) and torch.equal(again["C"].view(torch.int32), want["C"].view(torch.int32))

    def extracted(C):
        return (C[idx.long()] if row else C[:, idx.long()]).contiguous().view(torch.int32)
    rounded = ah.adahop_gemm(A, B, strategy, 32, k, **{seed: 5})
    assert torch.equal(extracted(rounded["C"]), extracted(want["C"]))
    alone = torch.full_like(want["C"], 3.0)
    ah.adahop_oe_gemm_bf16(A, B, strategy, idx, alone)
    assert torch.equal(extracted(alone), extracted(want["C"]))
    a, b = (A, B) if row else (B, A)
    take = a.tensor[idx.long()] if a.k_contig else a.tensor[:, idx.long()].T
    exact = take.double() @ at.double()
    bound = K * 2.0 ** -24 * (take.double().abs() @ at.double().abs())   # (see above)
    got = want["C"][idx.long()] if row else want["C"][:, idx.long()].T
    assert bool(((got.double() - exact).abs() <= bound).all())
    # infinities and NaN beside the end of K, where blocks are filled up with zeros
    at[K - 1, 3], at[K - 32, long - 1], at[K - 5, min(64, long - 2)] = float("inf"), -float("inf"), float("nan")
    want = ah.adahop_gemm(A, B, strategy, 32, k, idx=idx)
    again = ah.adahop_gemm(A, B, strategy, 32, k, idx=idx, **{packed: ah.adahop_pack_operand(l, row, strategy, 32)})
    # (the codes of a NaN have no defined sign: a K-contiguous operand's two quantisers subtract in different ways, and the rest of that row may differ)
    assert torch.equal(extracted(again["C"]), extracted(want["C"]))
    there = torch.arange(long, device="cuda") != (min(64, long - 2) if long_kc else -1)
    a, b = (C["C"][:, there] if row else C["C"][there] for C in (again, want))
    assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    assert bool(want["C"][idx.long()].isinf().any() if row else want["C"][:, idx.long()].isinf().any())


# K-contiguous, from 32 Mi elements on (k_outlier_products_kc): 16 .. 96 rows, each with every width that a workgroup may have; rows of the operand that end inside
# a workgroup's, a wave's and a load's 8; K-elements that end inside a block, at each quarter of it; one block, the shortest rows, and the longest
@pytest.mark.parametrize("short,long,K,k,short_kc", [
    (96, 8200, 4128, 5, True), (330, 4160, 8256, 17, False), (64, 1100, 31008, 40, True), (300, 8251, 4224, 60, True), (120, 28681, 1184, 90, False),
    (96, 8192, 4320, 96, True), (64, 131203, 256, 16, True), (40, 1048610, 32, 3, False), (24, 17, 2097120, 5, True),
    (64, 31452, 1184, 16, True), (64, 131203, 256, 20, True), (64, 64487, 544, 25, False), (96, 9423, 4128, 45, True), (64, 33199, 1184, 45, True),
    (96, 4293, 8224, 60, True), (64, 64370, 544, 49, True), (120, 68578, 544, 96, True), (80, 3486, 11040, 45, True)])
@pytest.mark.parametrize("strategy", [inputs.IHT_OE_ROW, inputs.IHT_OE_COL])
def test_same_bits_whoever_packs_a_k_contiguous_operand(short, long, K, k, short_kc, strategy):
    test_same_bits_whoever_packs_the_other_operand(short, long, K, k, short_kc, strategy, long_kc=True)


@pytest.mark.parametrize("long_kc", [False, True])
@pytest.mark.parametrize("long,K,k", [(20008, 4320, 64), (4100, 8224, 9)])
def test_products_by_themselves_under_capture(long, K, k, long_kc):
    """The products of a packed operand, long slices and short, from a graph: every replay, with new rows in place and eager calls between, has the
    eager call's bits."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_02525_amd import binding as ah
    print("[case] capture", long, K, k, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(long)
    rows = torch.randn(3, 96, K, generator=gen, device="cuda").to(torch.bfloat16)
    A = ah.Operand(rows[0].clone(), True)
    if long_kc:
        B = ah.Operand(torch.randn(long, K, generator=gen, device="cuda").to(torch.bfloat16), True)
    else:
        B = ah.Operand(torch.randn(K, (long + 7) // 8 * 8, generator=gen, device="cuda").to(torch.bfloat16)[:, :long], False)
    packed = ah.adahop_pack_operand(B, True, inputs.IHT_OE_ROW, 32)
    ws = torch.empty(ah.adahop_gemm_workspace_bytes(96, long, K, inputs.IHT_OE_ROW, k), dtype=torch.uint8, device="cuda")
    C, idx = torch.empty(96, long, device="cuda"), torch.randperm(96, generator=gen, device="cuda")[:k].to(torch.int32)

    def call(out):
        return ah.adahop_gemm(A, B, inputs.IHT_OE_ROW, 32, k, idx=idx, Cout=out, workspace=ws, b_packed=packed)
    ah.adahop_prepare_device()
    call(C)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(C)
    for i in (1, 2, 0):
        A.tensor.copy_(rows[i])
        graph.replay()
        got = C.clone()
        want = torch.full_like(C, 5.0)
        call(want)
        torch.cuda.synchronize()
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), i
