"""GPU parity of the stochastic-rounding option of the quantisers (run with -m gpu).

Both sides implement the same counter-based generator (Philox4x32-10 keyed by the seed, counted by the
element's position), so the bar is the usual one: codes and scales bit for bit, whatever the layout, the
transform block or the masks; the product within 1e-3 relative Frobenius of the oracle's.
"""
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


@pytest.mark.parametrize("k_contig", [True, False])
def test_sr_quantiser_at_the_edges_of_the_range(ah, k_contig):
    """No transform; every block has its largest magnitude at one exponent of the whole bf16 range (zero and subnormal
    blocks among them) and the other elements anywhere from there down to the smallest subnormal, magnitudes on and next
    to the E2M1 values, both zeros."""
    rng = np.random.default_rng(4)
    outer, K = 264, 512
    top = rng.integers(0, 255, size=(outer, K // 32, 1))
    exp = np.maximum(top - np.where(rng.random((outer, K // 32, 32)) < 0.8, rng.integers(0, 5, size=(outer, K // 32, 32)),
                                    rng.integers(0, 255, size=(outer, K // 32, 32))), 0)
    exp[:, :, 0] = top[:, :, 0]
    mant = np.where(rng.random(exp.shape) < 0.5, rng.choice([0, 1, 63, 64, 65, 127], size=exp.shape), rng.integers(0, 128, size=exp.shape))
    bits = (rng.integers(0, 2, size=exp.shape) << 15 | exp << 7 | mant).astype(np.uint16).reshape(outer, K)
    bits[5, :64] &= 0x8000
    stored = bits if k_contig else np.ascontiguousarray(bits.T)
    say("SR quantiser, edges of the range", "K-contiguous" if k_contig else "K-strided")
    codes, scales = ah.adahop_iht_quantize(ah.Operand(torch.from_numpy(stored.view(np.int16)).cuda(), k_contig), 0, sr_seed=77)
    torch.cuda.synchronize()
    rc, rs = orc.iht_quantize(stored, k_contig, 0, sr_seed=77)
    assert np.array_equal(host(scales), rs)
    assert np.array_equal(host(codes), rc)


@pytest.mark.parametrize("seed", [None, 78])
@pytest.mark.parametrize("K", [256, 288])
@pytest.mark.parametrize("k_contig", [True, False])
def test_elements_that_are_no_number(ah, k_contig, K, seed):
    """No transform: such an element does not count for its block's scale; rounded to nearest it takes the largest magnitude, rounded
    stochastically code 0, with its sign, as the oracle's comparisons have it.  Quiet ones, as arithmetic makes them: a signalling
    one (0x7f81) comes out of the hardware's maximum as a quiet one and does count, in every kernel."""
    rng = np.random.default_rng(6)
    bits = inputs.matrix(72, K, 1.0, 720)
    at = rng.random(bits.shape) < 0.02
    bits[at] = rng.choice(np.array([0x7fc0, 0xffc0, 0x7fe1, 0xffff], dtype=np.uint16), size=int(at.sum()))
    bits[3, :32] = 0xffc0
    stored = bits if k_contig else np.ascontiguousarray(bits.T)
    say("elements that are no number", "K-contiguous" if k_contig else "K-strided", K, seed)
    codes, scales = ah.adahop_iht_quantize(ah.Operand(torch.from_numpy(stored.view(np.int16)).cuda(), k_contig), 0, sr_seed=seed)
    torch.cuda.synchronize()
    rc, rs = orc.iht_quantize(stored, k_contig, 0, sr_seed=seed)
    assert np.array_equal(host(scales), rs)
    assert np.array_equal(host(codes), rc)


@pytest.mark.parametrize("k_contig", [True, False])
@pytest.mark.parametrize("b,outer,K", [(0, 70, 96), (32, 130, 160), (64, 67, 448), (128, 200, 512), (256, 131, 1024),
                                       (32, 300, 2048), (0, 9, 256)])
def test_sr_quantiser_bit_exact(ah, b, outer, K, k_contig):
    logical = inputs.matrix(outer, K, 1.0, 700 + b, row_outliers=(3, 60.0, 60.0), col_outliers=(4, 30.0, 30.0))
    stored = logical if k_contig else np.ascontiguousarray(logical.T)
    if stored.shape[1] % 8:
        wide = np.zeros((stored.shape[0], (stored.shape[1] + 7) // 8 * 8), dtype=np.uint16)
        wide[:, :stored.shape[1]] = stored
        t = torch.from_numpy(wide.view(np.int16)).cuda()[:, :stored.shape[1]]
    else:
        t = torch.from_numpy(stored.view(np.int16)).cuda()
    x = ah.Operand(t, k_contig)
    rng = np.random.default_rng(b + outer)
    zo = (rng.random(outer) < 0.05).astype(np.uint8)
    zk = (rng.random(K) < 0.05).astype(np.uint8)
    for seed, masks in ((1, False), (0xfedcba9876543210, True)):
        say("SR quantiser", b, outer, K, "K-contiguous" if k_contig else "K-strided", hex(seed), "masks" if masks else "")
        d_zo = torch.from_numpy(zo).cuda() if masks else None
        d_zk = torch.from_numpy(zk).cuda() if masks else None
        codes, scales = ah.adahop_iht_quantize(x, b, d_zo, d_zk, sr_seed=seed)
        torch.cuda.synchronize()
        rc, rs = orc.iht_quantize(stored, k_contig, b, zo if masks else None, zk if masks else None, sr_seed=seed)
        assert np.array_equal(host(scales), rs)
        assert np.array_equal(host(codes), rc)
    # a different seed changes codes but not scales; no seed is the deterministic quantiser
    c2, s2 = ah.adahop_iht_quantize(x, b, sr_seed=2)
    c0, s0 = ah.adahop_iht_quantize(x, b)
    c1, s1 = ah.adahop_iht_quantize(x, b, sr_seed=1)
    torch.cuda.synchronize()
    assert torch.equal(s2, s0) and torch.equal(s1, s0) and not torch.equal(c1, c2)
    r0, _ = orc.iht_quantize(stored, k_contig, b)
    assert np.array_equal(host(c0), r0)


@pytest.mark.parametrize("strategy,k", [(inputs.IHT, 0), (inputs.IHT_OE_ROW, 5), (inputs.IHT_OE_K, 9)])
def test_whole_path_with_stochastically_rounded_gradient_operand(ah, strategy, k):
    """dgrad-like product: the gradient (A) rounded stochastically, the weight (B, K-strided) to nearest."""
    T, d_out, d_in = 328, 512, 264
    G = inputs.Operand(inputs.matrix(T, d_out, 1e-3, 710, row_outliers=(4, 100.0, 100.0)), True)
    W = inputs.Operand(inputs.matrix(d_out, d_in, 0.02, 711), False)
    say("whole path, SR on A", inputs.STRATEGY_NAMES[strategy])
    dG, dW = ah.Operand.from_bits(G.bits, True), ah.Operand.from_bits(W.bits, False)
    out = ah.adahop_gemm(dG, dW, strategy, 128, k, sr_seed_a=77)
    torch.cuda.synchronize()
    ref = orc.adahop_gemm(G.bits, True, W.bits, False, strategy, 128, k, sr_seed_a=77)
    for name in ("a_scales", "b_scales", "a_codes", "b_codes"):
        assert np.array_equal(host(out[name]), ref[name]), name
    if k:
        assert np.array_equal(np.sort(host(out["idx"])), ref["idx"])
    err = np.linalg.norm(host(out["C"]).astype(np.float64) - ref["C"]) / np.linalg.norm(ref["C"])
    say(f"  vs oracle {err:.2e}")
    assert err < 1e-3
    det = ah.adahop_gemm(dG, dW, strategy, 128, k)
    torch.cuda.synchronize()
    assert torch.equal(det["b_codes"], out["b_codes"]) and not torch.equal(det["a_codes"], out["a_codes"])


@pytest.mark.parametrize("K,k,b", [(4096, 37, 128), (288, 9, 32), (4384, 70, 32)])
def test_stochastic_rounding_in_the_quantiser_that_copies_k_channels(ah, K, k, b):
    """OE-K on K-contiguous operands takes the quantiser that also copies the extracted channels out, one row per workgroup and several, K
    a whole number of 256-element units and not; its stochastic-rounding instance must draw as every other quantiser does."""
    M, N = 136, 72
    A = inputs.Operand(inputs.matrix(M, K, 1.0, 720, col_outliers=(12, 40.0, 80.0)), True)
    B = inputs.Operand(inputs.matrix(N, K, 0.02, 721), True)
    say("whole path, SR on both operands, channels copied by the quantiser")
    dA, dB = ah.Operand.from_bits(A.bits, True), ah.Operand.from_bits(B.bits, True)
    out = ah.adahop_gemm(dA, dB, inputs.IHT_OE_K, b, k, sr_seed_a=5, sr_seed_b=6)
    torch.cuda.synchronize()
    ref = orc.adahop_gemm(A.bits, True, B.bits, True, inputs.IHT_OE_K, b, k, sr_seed_a=5, sr_seed_b=6)
    for name in ("a_scales", "b_scales", "a_codes", "b_codes"):
        assert np.array_equal(host(out[name]), ref[name]), name
    assert np.array_equal(np.sort(host(out["idx"])), ref["idx"])
    err = np.linalg.norm(host(out["C"]).astype(np.float64) - ref["C"]) / np.linalg.norm(ref["C"])
    say(f"  vs oracle {err:.2e}")
    assert err < 1e-3


@pytest.mark.parametrize("K,b", [(512, 256), (544, 32), (96, 32)])
@pytest.mark.parametrize("layouts", [(True, False), (False, True), (False, False)])
@pytest.mark.parametrize("strategy", [inputs.IHT_OE_ROW, inputs.IHT_OE_COL])
def test_stochastic_rounding_in_the_quantiser_that_copies_rows(ah, strategy, layouts, K, b):
    """The rounded operand is the one that rows / columns are extracted from, and its quantiser copies them out: K-contiguous and K-strided, K
    a whole number of 256-element units and not.  With the indices handed in, so that a kernel of its own gathers them, C has the same bits."""
    M, N, k = 131, 72, 5
    A = inputs.matrix(M, K, 1e-3, 730, row_outliers=(4, 100.0, 100.0))
    B = inputs.matrix(N, K, 0.02, 731, row_outliers=(4, 50.0, 50.0))
    say("SR, rows copied by the quantiser", inputs.STRATEGY_NAMES[strategy], layouts, K, b)
    ops, host_ops = [], []
    for bits, kc in ((A, layouts[0]), (B, layouts[1])):
        arr = bits if kc else np.ascontiguousarray(bits.T)
        wide = np.zeros((arr.shape[0], (arr.shape[1] + 7) // 8 * 8), dtype=np.uint16)
        wide[:, :arr.shape[1]] = arr
        ops.append(ah.Operand(torch.from_numpy(wide.view(np.int16)).cuda()[:, :arr.shape[1]], kc))
        host_ops += [arr, kc]
    seeds = dict(sr_seed_a=77) if strategy == inputs.IHT_OE_ROW else dict(sr_seed_b=78)
    out = ah.adahop_gemm(*ops, strategy, b, k, **seeds)
    again = ah.adahop_gemm(*ops, strategy, b, k, idx=out["idx"].clone(), **seeds)
    torch.cuda.synchronize()
    ref = orc.adahop_gemm(*host_ops, strategy, b, k, **seeds)
    for name in ("a_scales", "b_scales", "a_codes", "b_codes"):
        assert np.array_equal(host(out[name]), ref[name]), name
    assert np.array_equal(np.sort(host(out["idx"])), ref["idx"])
    assert torch.equal(out["C"].view(torch.int32), again["C"].view(torch.int32))
    assert np.linalg.norm(host(out["C"]).astype(np.float64) - ref["C"]) / np.linalg.norm(ref["C"]) < 1e-3


@pytest.mark.parametrize("layouts", [(True, False), (False, True), (False, False)])
@pytest.mark.parametrize("rounded", ["a", "b"])
@pytest.mark.parametrize("M,N,K,b", [(3, 1, 32, 32), (70, 65, 288, 32), (130, 200, 512, 256), (64, 13001, 544, 32), (13001, 70, 320, 64)])
def test_one_operand_rounded_beside_the_other(ah, layouts, rounded, M, N, K, b):
    """Both operands quantised in one launch where the other one is K-strided: one workgroup of either, shorter last tiles, rows
    off the 128-byte lines (an order of their own).  Codes and scales are the bits of the quantisers by themselves."""
    say("rounded beside", layouts, rounded, (M, N, K, b))
    ops = {}
    for key, outer, kc in (("a", M, layouts[0]), ("b", N, layouts[1])):
        x = inputs.matrix(outer, K, 1e-3 if key == rounded else 0.02, 9700 + outer)
        wide = np.zeros(((outer, K) if kc else (K, (outer + 7) // 8 * 8)), dtype=np.uint16)
        wide[:, :(K if kc else outer)] = x if kc else x.T
        ops[key] = ah.Operand(torch.from_numpy(wide.view(np.int16)).cuda()[:, :(K if kc else outer)], kc)
    out = ah.adahop_gemm(ops["a"], ops["b"], inputs.IHT, b, 0, **{"sr_seed_" + rounded: 4711})
    for key in ("a", "b"):
        codes, scales = ah.adahop_iht_quantize(ops[key], b, sr_seed=4711 if key == rounded else None)
        torch.cuda.synchronize()
        assert torch.equal(out[key + "_codes"], codes) and torch.equal(out[key + "_scales"], scales), key
