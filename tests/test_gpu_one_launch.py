"""Small products of two K-contiguous operands, which are quantised and multiplied in one launch, against the two launches that
the same call takes with the 32 x 32 kernel forced, and against the product of the same operands packed beforehand: the same codes, scales
and bits of C, on both sides of the line and at the edges of tiles, stages and scaling blocks."""
import pytest
import torch

from paper_2604_02525_amd import binding as ah

pytestmark = pytest.mark.gpu

SHAPES = [  # M, N, K, transform block (0: none), columns that the rows of the operands have beyond K, one launch or two
    (1, 1, 32, 32, 0, True), (7, 40, 96, 32, 0, True), (32, 32, 256, 256, 0, True), (33, 65, 352, 32, 8, True), (31, 64, 224, 0, 0, True),
    (256, 256, 256, 128, 0, True), (100, 200, 320, 64, 16, True), (65, 33, 512, 256, 0, True), (513, 31, 736, 32, 0, True),
    (256, 1024, 768, 256, 0, True),         # 256 tiles, three stages: the last of the line
    (257, 1024, 256, 32, 0, True), (512, 1024, 256, 64, 0, True),   # up to 512 tiles, one stage
    (512, 1024, 288, 32, 0, False), (513, 1024, 256, 32, 0, False), (8, 8200, 768, 128, 0, False), (64, 64, 800, 32, 0, False),  # beyond it
]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("M,N,K,block,pad,one", SHAPES)
def test_same_bits_as_in_two_launches(M, N, K, block, pad, one, bf16):
    gen = torch.Generator(device="cuda").manual_seed(M * 7 + N * 3 + K)

    def operand(rows, std):
        x = torch.randn(rows, K + pad, generator=gen, device="cuda").mul_(std)
        x[0, :32] = 0.0                         # a block of zeros, and one far above the others
        x[rows - 1, K - 32:K] *= 3000.0
        return ah.Operand(x.to(torch.bfloat16)[:, :K], True)
    A, B = operand(M, 1.0), operand(N, 0.02)
    strategy = ah.ADAHOP_IHT if block else ah.ADAHOP_NONE
    names = ("C", "a_codes", "a_scales", "b_codes", "b_scales")

    def call(**packed):
        C = torch.full((M, N + 3), 7.0, dtype=torch.bfloat16 if bf16 else torch.float32, device="cuda")
        ws = torch.full((ah.adahop_gemm_workspace_bytes(M, N, K, strategy, 0),), 0xA5, dtype=torch.uint8, device="cuda")
        r = ah.adahop_gemm(A, B, strategy, block, 0, Cout=C[:, :N], workspace=ws, **packed)
        torch.cuda.synchronize()
        assert bool((C[:, N:] == 7.0).all())    # nothing is written beside the rows of C
        at = r["layout"].gemm
        scratch = ws[at:at + ah.adahop_gemm_mx_workspace_bytes(M, N, K)]
        return {n: r[n] for n in names}, bool((scratch == 0xA5).all())
    got, untouched = call()
    assert untouched == one                     # the quantisers of two launches write the second copy of the scales there
    try:
        ah.adahop_debug_force_gemm_kernel(11)
        want, untouched = call()
    finally:
        ah.adahop_debug_force_gemm_kernel(0)
    assert not untouched
    for n in names:
        assert torch.equal(got[n], want[n]), n
    packed, _ = call(a_packed=(got["a_codes"], got["a_scales"]), b_packed=(got["b_codes"], got["b_scales"]))
    assert torch.equal(packed["C"], got["C"])
