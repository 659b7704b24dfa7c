"""GPU-vs-oracle parity through the C ABI (run with -m gpu on an MI355X).

Bars: packed E2M1 codes, E8M0 scales, FOID indices and masks bit-exact.  GEMM outputs: within 1e-3
relative Frobenius error of the oracle's emulated-MXFP4 result, taken separately over the extracted
rows / columns (BF16 path, ~100x larger values) and over the rest, so that the large entries cannot
hide an error in the ordinary ones; and every compared element within
    |C_gpu[i, j] - C_oracle[i, j]| <= 2^-20 |A[i, :]|_2 |B[j, :]|_2.
Both sides sum the same exact products (E2M1 values times powers of two, or bf16 x bf16, are exact in
fp32); only the fp32 accumulation order of the GPU differs from the oracle's double sum.  A length-K
fp32 accumulation errs by about sqrt(K) 2^-24 |C| and |C| is about |A_i| |B_j| / sqrt(K) for these
inputs, so the allowance is some tens of times the expected error and, relative to a typical |C|,
sqrt(K) 2^-20 <= 1e-4: a wrong operand byte, scale or tile lands orders of magnitude above it.
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


def dev_op(ah, op):
    return ah.Operand.from_bits(op.bits, op.k_contig)


def host(t):
    return t.cpu().numpy()


def rel_fro(got, ref):
    return float(np.linalg.norm(got.astype(np.float64) - ref) / max(np.linalg.norm(ref), 1e-300))


def row_norms(op, sel=None):
    """2-norms of the logical rows (all of them, or those in sel) of an inputs.Operand, in float64."""
    bits = op.bits if op.k_contig else op.bits.T
    if sel is not None:
        bits = bits[np.asarray(sel, dtype=np.int64)]
    out = np.empty(bits.shape[0])
    for r0 in range(0, bits.shape[0], 1024):          # in slabs: a whole config operand in float64 is gigabytes
        v = (np.ascontiguousarray(bits[r0:r0 + 1024]).astype(np.uint32) << 16).view(np.float32).astype(np.float64)
        out[r0:r0 + 1024] = np.sqrt((v * v).sum(axis=1))
    return out


def check_c(got, ref, g, rows=None, cols=None, extracted=None, tol=1e-3):
    """The bars of the module docstring on C (got: what the GPU wrote, ref: the oracle's, both on rows x cols).
    extracted: the indices the strategy routed to BF16 (rows for OE-row, columns for OE-col)."""
    got = got.astype(np.float64)
    bar = 2.0 ** -20 * np.outer(row_norms(g.A, rows), row_norms(g.B, cols))
    excess = np.abs(got - ref) - bar
    worst = np.unravel_index(np.argmax(excess), excess.shape)
    assert excess[worst] <= 0.0, (f"element {worst} of the compared block: |{got[worst]} - {ref[worst]}| exceeds the "
                                  f"accumulation allowance {bar[worst]:.3e}")
    err = rel_fro(got, ref)
    assert err < tol
    parts = {}
    if extracted is not None and len(extracted):
        R = np.arange(ref.shape[0]) if rows is None else np.asarray(rows)
        Cc = np.arange(ref.shape[1]) if cols is None else np.asarray(cols)
        if g.strategy == inputs.IHT_OE_ROW:
            m = np.isin(R, extracted)
            split = ((got[m], ref[m]), (got[~m], ref[~m]))
        elif g.strategy == inputs.IHT_OE_COL:
            m = np.isin(Cc, extracted)
            split = ((got[:, m], ref[:, m]), (got[:, ~m], ref[:, ~m]))
        else:
            split = ()
        for name, (a, b) in zip(("extracted", "residual"), split):
            if a.size:
                parts[name] = rel_fro(a, b)
                assert parts[name] < tol, name
    return err, parts, float((np.abs(got - ref) / bar).max())


def rand_bits(rng, shape, scale=1.0):
    x = torch.from_numpy((rng.standard_normal(shape) * scale).astype(np.float32))
    return x.to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)


def stored(bits_ok, k_contig, pad=0):
    """bits_ok is logical [outer, K]; return the array as stored (optionally with ld > width)."""
    a = bits_ok if k_contig else np.ascontiguousarray(bits_ok.T)
    pad += (-(a.shape[1] + pad)) % 8          # the ABI wants ld to be a multiple of 8 elements
    if pad:
        wide = np.zeros((a.shape[0], a.shape[1] + pad), dtype=a.dtype)
        wide[:, :a.shape[1]] = a
        return wide, a.shape[1]
    return a, a.shape[1]


# ----------------------------------------------------------------------------- quantisers

@pytest.mark.parametrize("k_contig", [True, False])
@pytest.mark.parametrize("b", [0, 32, 64, 128, 256])
def test_iht_quantize_bit_exact(ah, b, k_contig):
    rng = np.random.default_rng(100 + b + int(k_contig))
    for outer, K, pad, masks in ((77, 3 * max(b, 32), 0, False), (300, 4 * max(b, 32), 8, True),
                                 (130, 1280 if b != 256 else 1280, 0, True), (1, max(b, 32), 0, False)):
        if b and K % b:
            K = (K // b + 1) * b
        say("iht_quantize", dict(b=b, k_contig=k_contig, outer=outer, K=K, pad=pad, masks=masks))
        logical = rand_bits(rng, (outer, K))
        logical[rng.integers(0, outer), :] = 0                      # an all-zero row
        logical[:, 5] = rand_bits(rng, (outer,), 60.0)              # an outlier channel
        arr, width = stored(logical, k_contig, pad)
        t = torch.from_numpy(arr.view(np.int16)).cuda()
        x = ah.Operand(t[:, :width], k_contig)
        zo = zk = zo_d = zk_d = None
        if masks:
            zo = (rng.random(outer) < 0.1).astype(np.uint8)
            zk = (rng.random(K) < 0.05).astype(np.uint8)
            zo_d, zk_d = torch.from_numpy(zo).cuda(), torch.from_numpy(zk).cuda()
        codes, scales = ah.adahop_iht_quantize(x, b, zo_d, zk_d)
        torch.cuda.synchronize()
        rc, rs = orc.iht_quantize(arr[:, :width], k_contig, b, zo, zk)
        assert np.array_equal(host(scales), rs)
        assert np.array_equal(host(codes), rc)


@pytest.mark.parametrize("b", [256, 32])
def test_iht_quantize_k_strided_long_rows_bit_exact(ah, b):
    """K-strided operand with 278 tiles of 64 columns, rows off the 128-byte lines (the quantiser then starts its workgroups in groups of
    16 column tiles that walk the K-blocks together): a whole number of groups plus a narrower last one with a ragged
    last tile, three K-blocks, with both masks."""
    outer, K = (8 * 32 + 21) * 64 + 40, 768
    rng = np.random.default_rng(300 + b)
    logical = rand_bits(rng, (outer, K))
    logical[:, 700] = rand_bits(rng, (outer,), 60.0)
    arr, width = stored(logical, False)
    x = ah.Operand(torch.from_numpy(arr.view(np.int16)).cuda()[:, :width], False)
    zo = (rng.random(outer) < 0.05).astype(np.uint8)
    zk = (rng.random(K) < 0.05).astype(np.uint8)
    say("iht_quantize, K-strided, long rows", dict(b=b, outer=outer, K=K))
    for masks in (False, True):
        codes, scales = ah.adahop_iht_quantize(x, b, torch.from_numpy(zo).cuda() if masks else None,
                                               torch.from_numpy(zk).cuda() if masks else None)
        torch.cuda.synchronize()
        rc, rs = orc.iht_quantize(arr[:, :width], False, b, zo if masks else None, zk if masks else None)
        assert np.array_equal(host(scales), rs)
        assert np.array_equal(host(codes), rc)


def test_quantize_mx_every_bf16_pattern_bit_exact(ah):
    """Every finite bf16 value, placed so that it lands in each E2M1 binade (and in the saturating
    range) relative to the block scale set by an anchor element."""
    allbits = np.arange(65536, dtype=np.uint32)
    vals = (allbits << 16).view(np.float32)
    keep = np.isfinite(vals) & (np.abs(vals) > 2.0 ** -100) & (np.abs(vals) < 2.0 ** 100)
    pats = allbits[keep].astype(np.uint16)
    v = vals[keep]
    e = np.floor(np.log2(np.abs(v))).astype(np.int64)
    blocks = []
    for shift in (-4, -3, -2, -1, 0, 1, 2):      # anchor = 2^(e - shift + 2): value/X falls in binade `shift`
        anchor = np.exp2((e - shift + 2).astype(np.float64)).astype(np.float32)
        anchor_bits = (anchor.view(np.uint32) >> 16).astype(np.uint16)
        blk = np.zeros((len(pats), 32), dtype=np.uint16)
        blk[:, 0] = anchor_bits
        blk[:, 7] = pats
        blk[:, 30] = pats ^ 0x8000
        blocks.append(blk)
    # value itself is the block maximum (exercises saturation: value / X in [4, 8))
    blk = np.zeros((len(pats), 32), dtype=np.uint16)
    blk[:, 3] = pats
    blocks.append(blk)
    logical = np.concatenate(blocks, axis=0)
    say("quantize_mx all bf16 patterns", logical.shape)
    for k_contig in (True, False):
        arr, width = stored(logical, k_contig)
        x = ah.Operand(torch.from_numpy(arr.view(np.int16)).cuda()[:, :width], k_contig)
        codes, scales = ah.adahop_quantize_mx(x)
        torch.cuda.synchronize()
        rc, rs = orc.quantize_mx(arr[:, :width], k_contig)
        assert np.array_equal(host(scales), rs)
        assert np.array_equal(host(codes), rc)


# ----------------------------------------------------------------------------- FOID

@pytest.mark.parametrize("k_contig", [True, False])
@pytest.mark.parametrize("axis", [0, 1])
def test_foid_topk_bit_exact(ah, axis, k_contig):
    rng = np.random.default_rng(7 + axis * 2 + int(k_contig))
    for outer, K, ks in ((200, 96, (0, 1, 7, 96)), (4100, 160, (41, 160)), (40, 2080, (13,)), (28672, 64, (574, 72))):
        logical = rand_bits(rng, (outer, K))
        dim = outer if axis == 0 else K
        hot = rng.permutation(dim)[:5]
        if axis == 0:
            logical[hot, :] = rand_bits(rng, (5, K), 30.0)
        else:
            logical[:, hot] = rand_bits(rng, (outer, 5), 30.0)
        dup = rng.permutation(dim)[:6]              # exact score ties: identical sample windows
        if axis == 0:
            logical[dup[1::2], :64] = logical[dup[0::2], :64]
        else:
            logical[:64, dup[1::2]] = logical[:64, dup[0::2]]
        arr, width = stored(logical, k_contig)
        x = ah.Operand(torch.from_numpy(arr.view(np.int16)).cuda()[:, :width], k_contig)
        ref_scores = orc.foid_scores(arr[:, :width], k_contig, axis)
        for k in ks:
            k = min(k, dim)
            say("foid_topk", dict(axis=axis, k_contig=k_contig, outer=outer, K=K, k=k))
            idx, mask, scores = ah.adahop_foid_topk(x, axis, k)
            torch.cuda.synchronize()
            assert np.array_equal(host(scores).view(np.uint32), ref_scores.view(np.uint32))
            ridx, rmask = orc.topk(ref_scores, k)
            assert np.array_equal(host(idx), ridx)
            assert np.array_equal(host(mask), rmask)


def test_topk_selection_paths_bit_exact(ah):
    """The exact top-k on score vectors chosen to take each way through the selection kernel: a short candidate list
    behind the threshold from the thread maxima; more candidates than the list holds (all scores equal, or equal in
    their upper 16 bits); k above the number of threads; fewer key-owning threads than k; k = dim; dims just above
    and below the list size; well separated outliers, with k at, below and above their number (the select stops
    early, also with a threshold below that of the candidate list).  Scores come from rows that are constant except for two entries, so that their fp32
    variance scores can be steered: x = (a, -a, 0, ...) scores 2 a^2 exactly."""
    rng = np.random.default_rng(77)
    cases = []
    for dim, ks, kind in ((28672, (287, 574, 1, 1024, 1025, 3000, 28672), "random"), (28672, (287, 5000), "equal"),
                          (28672, (300,), "two-level"), (4097, (41, 4097), "random"), (4096, (41, 1500), "random"),
                          (9000, (90, 1100), "few-big"), (32768, (328, 640), "random"), (1090, (1089, 1024, 70), "random"),
                          (16384, (164, 100, 165, 200), "separated"), (3000, (30, 29, 31), "separated"),
                          (4100, (1000, 820, 41), "random"), (8191, (81, 1024), "random"), (32767, (327,), "separated")):
        if kind == "random":
            a = np.abs(rng.standard_normal(dim)).astype(np.float32) + 0.5
        elif kind == "equal":
            a = np.full(dim, 1.5, dtype=np.float32)
        elif kind == "separated":            # 1 % of the scores far above the rest and spread over several leading
            a = rng.uniform(0.5, 1.5, dim).astype(np.float32)  # digits: the select stops at its first or second digit
            big = rng.permutation(dim)[:ks[0]]
            a[big] = rng.uniform(8.0, 64.0, ks[0]).astype(np.float32)
        elif kind == "two-level":            # upper 16 bits of every score equal; they differ further down
            a = (1.0 + rng.integers(0, 60, dim) * 2.0 ** -9).astype(np.float32)
        else:                                # a handful of large scores among many equal small ones
            a = np.full(dim, 0.25, dtype=np.float32)
            a[rng.permutation(dim)[:50]] = rng.uniform(8.0, 16.0, 50).astype(np.float32)
        cases.append((dim, ks, kind, a))
    for dim, ks, kind, a in cases:
        x = np.zeros((dim, 64), dtype=np.float32)
        x[:, 0], x[:, 1] = a, -a
        bits = torch.from_numpy(x).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
        op = ah.Operand.from_bits(bits, True)
        ref_scores = orc.foid_scores(bits, True, 0)
        for k in ks:
            say("top-k paths", dict(dim=dim, k=k, kind=kind))
            idx, mask, scores = ah.adahop_foid_topk(op, 0, k)
            torch.cuda.synchronize()
            assert np.array_equal(host(scores).view(np.uint32), ref_scores.view(np.uint32))
            ridx, rmask = orc.topk(ref_scores, k)
            assert np.array_equal(host(idx), ridx)
            assert np.array_equal(host(mask), rmask)


def test_topk_score_scratch_at_odd_addresses(ah):
    """Score scratch that is only 4-byte aligned, which is all the interface asks for (the selection kernel then
    loads and clears element by element), on sizes with a ragged last wave."""
    import ctypes as C
    rng = np.random.default_rng(78)
    for dim, k in ((5000, 50), (28671, 287), (130, 7)):
        bits = rand_bits(rng, (dim, 64))
        bits[rng.permutation(dim)[:k // 2], :] = rand_bits(rng, (k // 2, 64), 30.0)
        op = ah.Operand.from_bits(bits, True)
        ref_scores = orc.foid_scores(bits, True, 0)
        ridx, rmask = orc.topk(ref_scores, k)
        for s_off, m_off in ((1, 0), (3, 8), (2, 0)):
            say("top-k, scratch at odd addresses", dict(dim=dim, k=k, scores_offset=4 * s_off, mask_offset=m_off))
            scores = torch.zeros(dim + 8, dtype=torch.float32, device="cuda")
            mask = torch.full((dim + 16,), 7, dtype=torch.uint8, device="cuda")
            idx = torch.zeros(k, dtype=torch.int32, device="cuda")
            rc = ah.lib().adahop_foid_topk(C.byref(op.c()), 0, k, idx.data_ptr(), mask.data_ptr() + m_off,
                                           scores.data_ptr() + 4 * s_off, torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            assert rc == 0
            assert np.array_equal(host(scores)[s_off:s_off + dim].view(np.uint32), ref_scores.view(np.uint32))
            assert np.array_equal(host(idx), ridx)
            m = host(mask)
            assert np.array_equal(m[m_off:m_off + dim], rmask)
            assert (m[:m_off] == 7).all() and (m[m_off + dim:] == 7).all()      # nothing written around the mask


# ----------------------------------------------------------------------------- MXFP4 product

@pytest.mark.parametrize("shape", [(32, 32, 64), (128, 128, 256), (200, 136, 96), (257, 129, 32), (64, 384, 1056),
                                   (256, 256, 256), (512, 512, 512), (768, 1280, 2304), (2304, 512, 256),
                                   (300, 520, 512), (700, 256, 768), (256, 333, 1024)])
def test_gemm_mx_matches_emulation(ah, shape):
    M, N, K = shape
    rng = np.random.default_rng(M + N + K)
    a_codes = rng.integers(0, 256, size=(M, K // 2), dtype=np.uint8)
    b_codes = rng.integers(0, 256, size=(N, K // 2), dtype=np.uint8)
    a_scales = rng.integers(117, 137, size=(M, K // 32), dtype=np.uint8)
    b_scales = rng.integers(100, 120, size=(N, K // 32), dtype=np.uint8)
    say("gemm_mx", shape)
    C = ah.adahop_gemm_mx(*(torch.from_numpy(t).cuda() for t in (a_codes, a_scales, b_codes, b_scales)))
    torch.cuda.synchronize()
    ref = orc.mx_gemm(a_codes, a_scales, b_codes, b_scales)
    err = rel_fro(host(C), ref)
    say("  rel_fro", err)
    assert err < 1e-3
    assert err < 1e-5        # what the arithmetic predicts; a layout mistake gives O(1)


def test_gemm_mx_single_nonzero_probes_operand_layout(ah):
    """One nonzero code per operand at a time: the product must land in exactly one output element
    with exactly the right value, for positions covering every lane group, nibble and scale slot."""
    M = N = 64
    K = 128
    for (m, ka, code_a, sa), (n, code_b, sb) in [((0, 0, 7, 127), (0, 2, 127)), ((33, 37, 3, 130), (5, 6, 120)),
                                                 ((63, 127, 15, 125), (63, 9, 129)), ((17, 64, 5, 127), (40, 12, 127)),
                                                 ((8, 95, 1, 127), (31, 1, 126))]:
        a_codes = np.zeros((M, K // 2), np.uint8)
        b_codes = np.zeros((N, K // 2), np.uint8)
        a_scales = np.full((M, K // 32), 127, np.uint8)
        b_scales = np.full((N, K // 32), 127, np.uint8)
        a_codes[m, ka // 2] = code_a << (4 * (ka & 1))
        b_codes[n, ka // 2] = code_b << (4 * (ka & 1))
        a_scales[m, ka // 32] = sa
        b_scales[n, ka // 32] = sb
        say("gemm_mx probe", (m, n, ka))
        C = host(ah.adahop_gemm_mx(*(torch.from_numpy(t).cuda() for t in (a_codes, a_scales, b_codes, b_scales))))
        ref = orc.mx_gemm(a_codes, a_scales, b_codes, b_scales)
        assert np.count_nonzero(ref) == 1
        assert np.array_equal(C.astype(np.float64), ref)


# ----------------------------------------------------------------------------- whole path

def run_whole(ah, g, rows=None, cols=None, given_idx=None, tol=1e-3):
    A, B = dev_op(ah, g.A), dev_op(ah, g.B)
    idx_d = None if given_idx is None else torch.from_numpy(np.asarray(given_idx, dtype=np.int32)).cuda()
    out = ah.adahop_gemm(A, B, g.strategy, g.iht_block, g.k, idx=idx_d)
    torch.cuda.synchronize()
    ref = orc.adahop_gemm(g.A.bits, g.A.k_contig, g.B.bits, g.B.k_contig, g.strategy, g.iht_block, g.k,
                          idx=given_idx, rows=rows, cols=cols)
    if g.strategy >= inputs.IHT_OE_ROW and g.k > 0:
        got_idx = np.sort(host(out["idx"]))
        assert np.array_equal(got_idx, ref["idx"]), "extraction indices differ"
        mask = np.zeros(out["mask"].numel(), np.uint8)
        mask[ref["idx"]] = 1
        assert np.array_equal(host(out["mask"]), mask)
    for name in ("a_scales", "b_scales", "a_codes", "b_codes"):
        assert np.array_equal(host(out[name]), ref[name]), name
    C = out["C"]
    if rows is not None:
        C = C[torch.from_numpy(np.asarray(rows, dtype=np.int64)).cuda()]
    if cols is not None:
        C = C[:, torch.from_numpy(np.asarray(cols, dtype=np.int64)).cuda()]
    got = host(C)
    err, parts, used = check_c(got, ref["C"], g, rows, cols, ref["idx"] if g.k > 0 else None, tol)
    exact = orc.exact_gemm(g.A.bits, g.A.k_contig, g.B.bits, g.B.k_contig, rows=rows, cols=cols)
    q = rel_fro(got, exact)
    say(f"  {g.name} {inputs.STRATEGY_NAMES[g.strategy]} b={g.iht_block} k={g.k} shape={g.shape}: "
        f"vs oracle {err:.3e} " + " ".join(f"{n} {v:.3e}" for n, v in parts.items()) +
        f", worst element at {used:.3f} of its allowance, vs exact product {q:.3e} "
        f"({got.shape[0]} x {got.shape[1]} elements compared)")
    return err, q


def test_config0_iht_and_none(ah):
    g = inputs.config0()[0]
    say("config0 IHT")
    _, q_iht = run_whole(ah, g)
    g.strategy = inputs.NONE
    say("config0 none")
    _, q_none = run_whole(ah, g)
    assert q_iht < q_none                      # CN pair: the transform must help (paper Sec. 3.2)


LAYOUTS = {"fwd": (True, True), "dgrad": (True, False), "wgrad": (False, False)}


@pytest.mark.parametrize("kind", ["fwd", "dgrad", "wgrad"])
@pytest.mark.parametrize("strategy", [inputs.IHT, inputs.IHT_OE_ROW, inputs.IHT_OE_COL, inputs.IHT_OE_K])
def test_whole_path_small_all_layouts(ah, strategy, kind):
    """Ragged M and N spanning several workgroup tiles; K spans several transform blocks."""
    M, N, K, b = 328, 200, 512, 128
    a_kc, b_kc = LAYOUTS[kind]
    A_log = inputs.matrix(M, K, 1.0, 50, row_outliers=(5, 100.0, 100.0), col_outliers=(6, 50.0, 50.0))
    B_log = inputs.matrix(N, K, 0.02, 51, row_outliers=(4, 30.0, 30.0))
    A = inputs.Operand(A_log if a_kc else np.ascontiguousarray(A_log.T), a_kc)
    B = inputs.Operand(B_log if b_kc else np.ascontiguousarray(B_log.T), b_kc)
    k = {inputs.IHT: 0, inputs.IHT_OE_ROW: 9, inputs.IHT_OE_COL: 7, inputs.IHT_OE_K: 21}[strategy]
    g = inputs.Gemm(f"small.{kind}", A, B, strategy, b, k)
    say("whole path", kind, inputs.STRATEGY_NAMES[strategy])
    run_whole(ah, g)
    if k:
        given = np.random.default_rng(5).permutation({inputs.IHT_OE_ROW: M, inputs.IHT_OE_COL: N,
                                                      inputs.IHT_OE_K: K}[strategy])[:k].astype(np.int32)
        say("whole path, caller-chosen indices", kind, inputs.STRATEGY_NAMES[strategy])
        run_whole(ah, g, given_idx=given)


@pytest.mark.parametrize("strategy,k", [(inputs.IHT, 0), (inputs.IHT_OE_K, 5), (inputs.IHT_OE_K, 70),
                                        (inputs.IHT_OE_ROW, 6), (inputs.IHT_OE_COL, 3)])
@pytest.mark.parametrize("M,N", [(768, 512), (840, 600)])
def test_whole_path_tile_aligned_shape(ah, strategy, k, M, N):
    """K a multiple of 256, whole tiles and (second shape) ragged edges, K-channel part fused."""
    K = 1024
    A = inputs.Operand(inputs.matrix(M, K, 1.0, 60, row_outliers=(4, 100.0, 100.0), col_outliers=(5, 50.0, 50.0)), True)
    B = inputs.Operand(np.ascontiguousarray(inputs.matrix(N, K, 0.02, 61).T), False)
    g = inputs.Gemm("tiled", A, B, strategy, 256, k)
    say("tile-aligned whole path", inputs.STRATEGY_NAMES[strategy], k)
    run_whole(ah, g)


@pytest.mark.parametrize("strategy,k", [(inputs.IHT, 0), (inputs.IHT_OE_K, 5), (inputs.IHT_OE_K, 70), (inputs.IHT_OE_K, 150),
                                        (inputs.IHT_OE_ROW, 9)])
@pytest.mark.parametrize("M,N", [(4352, 4096), (4608, 3840)])
def test_more_tiles_than_compute_units(ah, strategy, k, M, N):
    """272 and 270 tiles of 256x256: some workgroups of the persistent kernel walk two tiles, with the stage pipeline
    running from one into the next (one, two and three gathered-bf16 stages per tile for the three OE-K ranks; an odd
    and an even number of stages per tile; a tile count that is and is not a multiple of 8).  C on a seeded sample of
    rows and columns that covers every tile row and tile column."""
    K = 768
    A = inputs.Operand(inputs.matrix(M, K, 1.0, 62, row_outliers=(6, 100.0, 100.0), col_outliers=(5, 50.0, 50.0)), True)
    B = inputs.Operand(inputs.matrix(N, K, 0.02, 63), True)
    g = inputs.Gemm("manytiles", A, B, strategy, 256, k)
    rng = np.random.default_rng(M + k)
    rows = np.unique(np.concatenate([np.arange(0, M, 256) + rng.integers(0, 256, M // 256), rng.integers(0, M, 16)]))
    cols = np.unique(np.concatenate([np.arange(0, N, 256) + rng.integers(0, 256, N // 256), rng.integers(0, N, 48)]))
    if strategy == inputs.IHT_OE_ROW:
        sel, _ = orc.foid_topk(A.bits, True, 0, k)
        rows = np.unique(np.concatenate([rows, sel[:4]]))
    say("more tiles than compute units", inputs.STRATEGY_NAMES[strategy], k, (M, N, K))
    run_whole(ah, g, rows=rows.astype(np.int32), cols=cols.astype(np.int32))


@pytest.mark.parametrize("M,N,K", [(4096, 8192, 768), (2048, 16384, 1024), (16384, 4096, 768), (8192, 8192, 768),
                                   (2304, 8192, 768)])
def test_every_order_of_the_tile_walk_gives_the_same_bits(ah, M, N, K):
    """The persistent 256 x 256 kernel walks its tiles in bands of A or of B, in XCD-contiguous runs or swept over the
    other operand (chosen by shape: the sweep only for operands larger than the Infinity Cache).  Forced each way on
    512 and 1024 tiles (two and four rounds of the 256 workgroups; two bands; two groups of 32 minor tiles; a shape
    whose sweep along B cannot run and falls back), every tile must be computed exactly once, with the same bits, and
    agree with the oracle on a sample that touches every tile."""
    rng = np.random.default_rng(M + N + K)
    a_codes = rng.integers(0, 256, size=(M, K // 2), dtype=np.uint8)
    b_codes = rng.integers(0, 256, size=(N, K // 2), dtype=np.uint8)
    a_scales = rng.integers(117, 137, size=(M, K // 32), dtype=np.uint8)
    b_scales = rng.integers(100, 120, size=(N, K // 32), dtype=np.uint8)
    dev = [torch.from_numpy(t).cuda() for t in (a_codes, a_scales, b_codes, b_scales)]
    say("tile walk orders", (M, N, K))
    out = {}
    try:
        for which in (0, 3, 4, 5, 6):
            ah.adahop_debug_force_gemm_kernel(which)
            C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
            ah.adahop_gemm_mx(*dev, Cout=C)
            torch.cuda.synchronize()
            out[which] = host(C)
    finally:
        ah.adahop_debug_force_gemm_kernel(0)
    for which in (0, 4, 5, 6):
        assert np.array_equal(out[3].view(np.uint32), out[which].view(np.uint32)), which
    rows = np.arange(0, M, 256) + rng.integers(0, 256, M // 256)
    cols = np.arange(0, N, 256) + rng.integers(0, 256, N // 256)
    ref = orc.mx_gemm(a_codes[rows], a_scales[rows], b_codes[cols], b_scales[cols])
    err = rel_fro(out[4][np.ix_(rows, cols)], ref)
    say("  rel_fro", err)
    assert err < 1e-5


@pytest.mark.parametrize("a_kc,b_kc", [(True, True), (True, False), (False, True)])
@pytest.mark.parametrize("K,k", [(4096, 41), (8192, 5), (8192, 200)])
def test_oe_k_channels_copied_by_the_quantiser(ah, a_kc, b_kc, K, k):
    """K-contiguous operands whose K is a whole number of 4096-element passes: the quantiser that the whole path runs
    also copies the extracted channels out, where otherwise a gather kernel does.  With the indices handed back in,
    the path takes the gather kernels: both must give the same C bit for bit (same copy, same summation order), and
    the oracle's on a sample of rows.  (Operands with one K-strided side mix the two routes in one product.)"""
    M, N, b = 304, 264, 128
    A_log = inputs.matrix(M, K, 1.0, 70 + k, col_outliers=(max(k // 2, 3), 40.0, 80.0))
    B_log = inputs.matrix(N, K, 0.02, 71 + k)
    A = inputs.Operand(A_log if a_kc else np.ascontiguousarray(A_log.T), a_kc)
    B = inputs.Operand(B_log if b_kc else np.ascontiguousarray(B_log.T), b_kc)
    g = inputs.Gemm("kcopy", A, B, inputs.IHT_OE_K, b, k)
    say("K-channels copied by the quantiser", (M, N, K), k, a_kc, b_kc)
    rows = np.arange(0, M, 7, dtype=np.int32)
    run_whole(ah, g, rows=rows)
    dA, dB = dev_op(ah, A), dev_op(ah, B)
    first = ah.adahop_gemm(dA, dB, inputs.IHT_OE_K, b, k)
    c_first, idx = host(first["C"]), first["idx"].clone()
    second = ah.adahop_gemm(dA, dB, inputs.IHT_OE_K, b, k, idx=idx)
    assert np.array_equal(c_first, host(second["C"]))


def test_oe_k_zero_equals_iht(ah):
    g = inputs.config0()[0]
    A, B = dev_op(ah, g.A), dev_op(ah, g.B)
    say("k=0 equals IHT")
    c_iht = host(ah.adahop_gemm(A, B, inputs.IHT, 32)["C"])
    for s in (inputs.IHT_OE_ROW, inputs.IHT_OE_COL, inputs.IHT_OE_K):
        assert np.array_equal(host(ah.adahop_gemm(A, B, s, 32, 0)["C"]), c_iht)


@pytest.mark.parametrize("M,N,K,k_row,k_col,k_k", [(152, 88, 160, 37, 5, 19), (520, 264, 1088, 300, 70, 33)])
def test_oe_gemm_bf16_standalone(ah, M, N, K, k_row, k_col, k_k):
    """Second term of Eq. 7 / Eq. 8 / the K-channel form alone; the larger case needs several row-tile groups
    and several K slices of the row / column kernel."""
    rng = np.random.default_rng(3)
    for a_kc, b_kc in LAYOUTS.values():
        A_log, B_log = rand_bits(rng, (M, K)), rand_bits(rng, (N, K), 0.05)
        A = inputs.Operand(A_log if a_kc else np.ascontiguousarray(A_log.T), a_kc)
        B = inputs.Operand(B_log if b_kc else np.ascontiguousarray(B_log.T), b_kc)
        dA, dB = dev_op(ah, A), dev_op(ah, B)
        for kind, dim, k in ((inputs.IHT_OE_ROW, M, k_row), (inputs.IHT_OE_COL, N, k_col), (inputs.IHT_OE_K, K, k_k)):
            sel = np.sort(rng.permutation(dim)[:k]).astype(np.int32)
            base = rng.standard_normal((M, N)).astype(np.float32)
            C = torch.from_numpy(base.copy()).cuda()
            say("oe_gemm_bf16", dict(a_kc=a_kc, b_kc=b_kc, kind=kind, k=k))
            ah.adahop_oe_gemm_bf16(dA, dB, kind, torch.from_numpy(sel).cuda(), C)
            torch.cuda.synchronize()
            want = base.astype(np.float64)
            if kind == inputs.IHT_OE_ROW:
                want[sel, :] = orc.bf16_gemm(A.bits, a_kc, B.bits, b_kc, rows=sel)
            elif kind == inputs.IHT_OE_COL:
                want[:, sel] = orc.bf16_gemm(A.bits, a_kc, B.bits, b_kc, cols=sel)
            else:
                want += orc.bf16_gemm(A.bits, a_kc, B.bits, b_kc, ksel=sel)
            assert rel_fro(host(C), want) < 1e-5


# ----------------------------------------------------------------------------- pattern detection (App. A)

@pytest.mark.parametrize("shape", [(2, 32), (37, 544), (9, 4128), (289, 1024), (2500, 4096), (2060, 6176), (4102, 8224)])
@pytest.mark.parametrize("k_contig", [True, False])
def test_detect_pattern_at_block_edges(ah, shape, k_contig):
    """Fewer rows than a workgroup has waves, rows one past a block, a chunk of one column, the most blocks of the kernel with
    small pieces, both workgroup sizes of the other; what lies
    behind the rows of the stored matrix is not a number.  The bounds of the test below."""
    outer, K = shape
    logical = inputs.matrix(outer, K, 1.0, 9100, col_outliers=(2, 50.0, 50.0))
    arr, width = stored(logical, k_contig)
    wide = np.full((arr.shape[0], (width + 7) // 8 * 8 + 8), 0x7fc0, dtype=np.uint16)
    wide[:, :width] = arr[:, :width]
    say("detect_pattern, block edges", shape, k_contig)
    p, st = ah.adahop_detect_pattern(ah.Operand(torch.from_numpy(wide.view(np.int16)).cuda()[:, :width], k_contig))
    torch.cuda.synchronize()
    want_p, want_st = orc.detect_pattern(logical, True)
    assert int(host(p)[0]) == want_p
    assert np.allclose(host(st), want_st, rtol=1e-9, atol=1e-12), (host(st), want_st)


@pytest.mark.parametrize("shape", [(600, 1056), (256, 512), (1030, 288)])
@pytest.mark.parametrize("k_contig", [True, False])
def test_detect_pattern_matches_oracle(ah, shape, k_contig):
    """CV figures to 1e-9 relative and the class exactly, for plain, row-outlier and channel-outlier tensors in both
    storage orders; sizes span several 256 x 512 blocks with ragged tails."""
    outer, K = shape
    for seed, kw in ((1, {}), (2, dict(row_outliers=(5, 100.0, 100.0))), (3, dict(col_outliers=(6, 50.0, 50.0)))):
        logical = inputs.matrix(outer, K, 1.0, 9000 + seed, **kw)
        arr, width = stored(logical, k_contig)
        say("detect_pattern", shape, k_contig, kw)
        x = ah.Operand(torch.from_numpy(arr.view(np.int16)).cuda()[:, :width], k_contig)
        p, st = ah.adahop_detect_pattern(x)
        torch.cuda.synchronize()
        want_p, want_st = orc.detect_pattern(logical, True)
        assert int(host(p)[0]) == want_p
        assert np.allclose(host(st), want_st, rtol=1e-9, atol=1e-12), (host(st), want_st)


@pytest.mark.parametrize("shape", [(3, 256), (521, 1056), (513, 288), (1031, 32)])
def test_detect_pattern_where_the_memory_ends_with_the_matrix(ah, shape):
    """Rows of no whole number of 16-byte pieces, the last of which ends with the memory: the last rows' workgroups read their
    last pieces by halves, the others do not.  The bounds of the test above."""
    outer, K = shape
    logical = inputs.matrix(outer, K, 1.0, 9110, row_outliers=(1, 50.0, 50.0))
    ld = (outer + 7) // 8 * 8
    flat = np.full((K - 1) * ld + outer, 0x7fc0, dtype=np.uint16)
    np.lib.stride_tricks.as_strided(flat, (K, outer), (2 * ld, 2))[:] = logical.T
    x = torch.from_numpy(flat.view(np.int16)).cuda().as_strided((K, outer), (ld, 1))
    say("detect_pattern, end of memory", shape)
    p, st = ah.adahop_detect_pattern(ah.Operand(x, False))
    torch.cuda.synchronize()
    want_p, want_st = orc.detect_pattern(logical, True)
    assert int(host(p)[0]) == want_p
    assert np.allclose(host(st), want_st, rtol=1e-9, atol=1e-12), (host(st), want_st)


def ending_with_its_last_element(ah, bits):
    """K-strided operand of logical [outer, K] bits with nothing of its own behind the last element: NaNs follow there."""
    outer, K = bits.shape
    ld = (outer + 7) // 8 * 8
    flat = np.full(K * ld + 8, 0x7fc0, dtype=np.uint16)
    np.lib.stride_tricks.as_strided(flat, (K, outer), (2 * ld, 2))[:] = bits.T
    return ah.Operand(torch.from_numpy(flat.view(np.int16)).cuda().as_strided((K, outer), (ld, 1)), False)


@pytest.mark.parametrize("outer", [1, 7, 65, 130, 187])
@pytest.mark.parametrize("K,b", [(32, 32), (96, 0), (256, 256), (544, 32)])
def test_quantiser_where_the_memory_ends_with_the_matrix(ah, outer, K, b):
    """K-strided rows of no whole number of 16-byte pieces: the last one's last piece is read element by element, with one, some and
    seven of them in it, in a tile of its own and beside whole pieces, and with K-rows behind the last one in its tile."""
    bits = inputs.matrix(outer, K, 1.0, 9600)
    x = ending_with_its_last_element(ah, bits)
    say("quantiser, end of memory", outer, K, b)
    for seed in (None, 31):
        codes, scales = ah.adahop_iht_quantize(x, b, sr_seed=seed)
        torch.cuda.synchronize()
        rc, rs = orc.iht_quantize(bits, True, b, sr_seed=seed)
        assert np.array_equal(host(scales), rs) and np.array_equal(host(codes), rc), seed


@pytest.mark.parametrize("N,K,k", [(41, 32, 3), (263, 96, 70), (129, 1600, 130), (4097, 576, 20), (8190, 512, 180)])
@pytest.mark.parametrize("col", [False, True])
def test_row_and_column_product_where_the_memory_ends_with_the_matrix(ah, N, K, k, col):
    """The same for the long operand of the BF16 product, of which a workgroup takes 128 rows (short L) or 256, in stages of 64 K-rows,
    the last of 32 or 64.  The allowance of the module docstring."""
    S = inputs.matrix(200, K, 1.0, 9610, row_outliers=(3, 40.0, 40.0))
    L = inputs.matrix(N, K, 0.02, 9611)
    idx = np.sort(np.random.default_rng(N + K).permutation(200)[:k]).astype(np.int32)
    s, l = ah.Operand.from_bits(S, True), ending_with_its_last_element(ah, L)
    say("row / column product, end of memory", N, K, k, col)
    C = torch.zeros((N, 200) if col else (200, N), dtype=torch.float32, device="cuda")
    a, b = (l, s) if col else (s, l)
    ah.adahop_oe_gemm_bf16(a, b, inputs.IHT_OE_COL if col else inputs.IHT_OE_ROW, torch.from_numpy(idx).cuda(), C)
    torch.cuda.synchronize()
    got = host(C).astype(np.float64)
    got = (got.T if col else got)[idx]
    sf, lf = (orc.bf16_to_double(x) for x in (S[idx], L))
    ref = sf @ lf.T
    bar = 2.0 ** -20 * np.outer(np.linalg.norm(sf, axis=1), np.linalg.norm(lf, axis=1))
    assert float((np.abs(got - ref) - bar).max()) <= 0.0


# ----------------------------------------------------- extracted parts copied out by the quantisers

@pytest.mark.parametrize("layouts", [(True, True), (True, False), (False, False), (False, True)])
@pytest.mark.parametrize("M,N,K,b", [(70, 40, 256, 256), (300, 130, 288, 32), (64, 520, 1056, 32), (130, 72, 2304, 128),
                                     (33, 41, 8480, 32), (2100, 6000, 4224, 64)])
@pytest.mark.parametrize("strategy", [inputs.IHT, inputs.IHT_OE_ROW, inputs.IHT_OE_COL, inputs.IHT_OE_K])
def test_quantisers_of_both_operands(ah, layouts, M, N, K, b, strategy):
    """Rows of one unit, of a shorter last unit, of several rows per workgroup and of more than one pass; both operands in
    one launch (test_quantisers_of_a_large_and_a_small_operand: in two).  Codes and scales are the oracle's bits; with the
    indices handed in, so that the extracted parts are gathered by kernels of their own, C has the same bits."""
    k = {inputs.IHT: 0, inputs.IHT_OE_ROW: max(1, M // 50), inputs.IHT_OE_COL: max(1, N // 50), inputs.IHT_OE_K: max(1, K // 50)}[strategy]
    A = inputs.matrix(M, K, 1.0, 9200, row_outliers=(2, 60.0, 60.0), col_outliers=(3, 30.0, 30.0))
    B = inputs.matrix(N, K, 0.02, 9201, row_outliers=(2, 50.0, 50.0))
    say("quantisers of both operands", layouts, (M, N, K, b), inputs.STRATEGY_NAMES[strategy], k)
    ops = []
    for bits, kc in ((A, layouts[0]), (B, layouts[1])):
        arr, width = stored(bits, kc)
        ops.append(ah.Operand(torch.from_numpy(arr.view(np.int16)).cuda()[:, :width], kc))
    out = ah.adahop_gemm(*ops, strategy, b, k)
    again = ah.adahop_gemm(*ops, strategy, b, k, idx=out["idx"].clone()) if k else out
    torch.cuda.synchronize()
    assert torch.equal(out["C"].view(torch.int32), again["C"].view(torch.int32))
    idx = np.sort(host(out["idx"])) if k else None
    mask_a = mask_b = mask_k = None
    if strategy == inputs.IHT_OE_ROW:
        mask_a = np.zeros(M, np.uint8); mask_a[idx] = 1
    if strategy == inputs.IHT_OE_COL:
        mask_b = np.zeros(N, np.uint8); mask_b[idx] = 1
    if strategy == inputs.IHT_OE_K:
        mask_k = np.zeros(K, np.uint8); mask_k[idx] = 1
    for name, bits, zo in (("a", A, mask_a), ("b", B, mask_b)):
        rc, rs = orc.iht_quantize(bits, True, b, zo, mask_k)
        assert np.array_equal(host(out[name + "_scales"]), rs), name
        assert np.array_equal(host(out[name + "_codes"]), rc), name


@pytest.mark.parametrize("M,N,K", [(24576, 40, 2048), (24577, 40, 2048), (24600, 12400, 2048), (900, 24601, 2080)])
@pytest.mark.parametrize("layouts", [(True, False), (False, True)])
def test_quantisers_of_a_large_and_a_small_operand(ah, layouts, M, N, K):
    """A K-contiguous operand beside a K-strided one, on both sides of 48 Mi elements and of twice as many as the other's: the bits of each by itself,
    also where one of them is rounded stochastically."""
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    say("quantisers of a large and a small operand", layouts, (M, N, K))
    ops = []
    for rows, kc in ((M, layouts[0]), (N, layouts[1])):
        ld = K if kc else (rows + 7) // 8 * 8
        t = torch.randn(*((rows, ld) if kc else (K, ld)), generator=gen, device="cuda").to(torch.bfloat16)
        ops.append(ah.Operand(t if kc else t[:, :rows], kc))
    for seeds in ((None, None), (5, None), (None, 6)):
        out = ah.adahop_gemm(*ops, inputs.IHT, 32, sr_seed_a=seeds[0], sr_seed_b=seeds[1])
        for name, op, seed in (("a", ops[0], seeds[0]), ("b", ops[1], seeds[1])):
            codes, scales = ah.adahop_iht_quantize(op, 32, sr_seed=seed)
            assert torch.equal(codes, out[name + "_codes"]) and torch.equal(scales, out[name + "_scales"]), (name, seeds)


@pytest.mark.parametrize("dim,k,free_kc", [(40, 40, True), (257, 3, True), (1024, 200, True), (1025, 256, True), (2048, 30, True), (2049, 30, True),
                                           (4099, 257, True), (8192, 82, True), (8192, 5000, True), (8193, 82, True), (16383, 164, True),
                                           (16384, 164, True), (16384, 9000, True), (16385, 164, True),
                                           (300, 100, False), (1024, 100, False), (1025, 100, False), (8192, 100, False), (8193, 100, False)])
@pytest.mark.parametrize("strategy", [inputs.IHT_OE_ROW, inputs.IHT_OE_COL])
@pytest.mark.parametrize("ties", [False, True])
def test_selection_beside_a_quantiser(ah, dim, k, free_kc, strategy, ties):
    """Fewer and more keys than threads, k up to and past what the threads' maxima can bound, the largest counts that the joint
    launches take (of 256 threads 8192, beside a K-strided operand, of 512 threads 16384) and one more; equal
    scores.  Indices and mask are those of the selection by itself, codes the oracle's.  (Beside a K-strided operand more than 96 rows: fewer
    are multiplied on the way of its quantiser, which then waits for the selection.)"""
    K, other = 96, 200
    bits = inputs.matrix(dim, K, 1.0, 9300, row_outliers=(3, 60.0, 60.0))
    if ties:
        bits[:] = bits[np.arange(dim) % 7]
    free = inputs.matrix(other, K, 0.02, 9301)
    say("selection beside a quantiser", dim, k, free_kc, inputs.STRATEGY_NAMES[strategy], "ties" if ties else "")
    x, y = ah.Operand.from_bits(bits, True), ah.Operand.from_bits(free if free_kc else np.ascontiguousarray(free.T), free_kc)
    want_idx, want_mask, _ = ah.adahop_foid_topk(x, 0, k)
    row = strategy == inputs.IHT_OE_ROW
    out = ah.adahop_gemm(*((x, y) if row else (y, x)), strategy, 32, k)
    torch.cuda.synchronize()
    assert torch.equal(out["idx"], want_idx) and torch.equal(out["mask"], want_mask)
    for name, b, zo in (("a" if row else "b", bits, host(want_mask)), ("b" if row else "a", free, None)):
        rc, rs = orc.iht_quantize(b, True, 32, zo, None)
        assert np.array_equal(host(out[name + "_scales"]), rs) and np.array_equal(host(out[name + "_codes"]), rc), name


@pytest.mark.parametrize("dim,other,K", [(2048, 4096, 4096), (2048, 4104, 4096), (2049, 4104, 4096), (1500, 8200, 2080), (8193, 8192, 4096), (8193, 4200, 8192), (8193, 8193, 8192)])
def test_selection_beside_a_large_quantiser(ah, dim, other, K):
    """Beside K-contiguous operands on both sides of 16 Mi elements, where workgroups of 256 threads take up to 2048 keys, and of 32 and 64 Mi,
    above which more than 8192 keys are selected first: the bits of each step by itself."""
    gen = torch.Generator(device="cuda").manual_seed(dim + K)
    x, y = (ah.Operand(torch.randn(n, K, generator=gen, device="cuda").to(torch.bfloat16), True) for n in (dim, other))
    say("selection beside a large quantiser", dim, other, K)
    want_idx, want_mask, _ = ah.adahop_foid_topk(x, 0, 20)
    out = ah.adahop_gemm(x, y, inputs.IHT_OE_ROW, 32, 20)
    torch.cuda.synchronize()
    assert torch.equal(out["idx"], want_idx) and torch.equal(out["mask"], want_mask)
    for name, op, zo in (("a", x, want_mask), ("b", y, None)):
        codes, scales = ah.adahop_iht_quantize(op, 32, zero_outer=zo)
        assert torch.equal(out[name + "_codes"], codes) and torch.equal(out[name + "_scales"], scales), name


@pytest.mark.parametrize("strategy", [inputs.IHT_OE_ROW, inputs.IHT_OE_COL])
@pytest.mark.parametrize("dim,other,k", [(40, 200, 3), (8192, 256, 82), (8192, 40, 82), (8193, 264, 20), (8200, 40, 9), (16385, 264, 20), (16392, 40, 9)])
def test_scores_left_in_the_workspace(ah, strategy, dim, other, k):
    """Row and column extraction leave the scores of all rows in the workspace, as the header says: selected beside the other
    operand's quantiser (up to 16384 rows) and not, with and without room for the table of positions beside the partial sums of the outlier product."""
    K = 96
    x = ah.Operand.from_bits(inputs.matrix(dim, K, 1.0, 9400, row_outliers=(3, 60.0, 60.0)), True)
    y = ah.Operand.from_bits(inputs.matrix(other, K, 0.02, 9401), True)
    say("scores in the workspace", inputs.STRATEGY_NAMES[strategy], dim, other, k)
    out = ah.adahop_gemm(*((x, y) if strategy == inputs.IHT_OE_ROW else (y, x)), strategy, 32, k)
    idx, mask, scores = ah.adahop_foid_topk(x, 0, k)
    again = ah.adahop_gemm(*((x, y) if strategy == inputs.IHT_OE_ROW else (y, x)), strategy, 32, k, idx=idx.clone())
    torch.cuda.synchronize()
    at = out["layout"].scores
    assert torch.equal(out["workspace"][at:at + 4 * dim].view(torch.int32), scores.view(torch.int32))
    assert torch.equal(out["idx"], idx) and torch.equal(out["mask"], mask)
    assert torch.equal(out["C"].view(torch.int32), again["C"].view(torch.int32))


def test_k_channels_copied_by_the_quantisers_of_many_channels(ah):
    """More K-channels than the selection that writes the table of their positions takes: the copies are those of the separate gather
    (indices handed in), K-contiguous beside K-contiguous and beside K-strided."""
    M, N, K, k = 70, 40, 33024, 330
    A = inputs.matrix(M, K, 1.0, 9500, col_outliers=(9, 30.0, 30.0))
    B = inputs.matrix(N, K, 0.02, 9501)
    say("K-channels copied by the quantisers", M, N, K, k)
    opa = ah.Operand.from_bits(A, True)
    for opb in (ah.Operand.from_bits(B, True), ah.Operand.from_bits(np.ascontiguousarray(B.T), False)):
        out = ah.adahop_gemm(opa, opb, inputs.IHT_OE_K, 128, k)
        got = {n: out[n].clone() for n in ("C", "idx", "a_codes", "a_scales", "b_codes", "b_scales")}
        want_idx, _, _ = ah.adahop_foid_topk(opa, 1, k)
        again = ah.adahop_gemm(opa, opb, inputs.IHT_OE_K, 128, k, idx=got["idx"].clone())
        torch.cuda.synchronize()
        assert torch.equal(got["idx"], want_idx)
        for name, t in got.items():
            assert torch.equal(t, again[name]), name
