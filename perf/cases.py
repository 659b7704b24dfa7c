"""The work that a user of this library has it do, as timed cases.

Every case is one pass through the public entry points of paper_2604_02525_amd.binding on operands that are already on
the GPU, with the output, the workspace and (where a program would keep one) the packed weight allocated beforehand.
Three kinds of work:

  product  one product of a linear layer (adahop_gemm): forward Y = X W^T, input gradient G_X = G_Y W, or weight gradient
           G_W = G_Y^T X, each with the operand layouts that these have in a training step (X [tokens, d_in], W [d_out,
           d_in], G_Y [tokens, d_out], row-major).  "layer" runs all three, one after the other;
  pack     one operand quantised by itself (adahop_pack_operand), as for a weight that is packed once per step;
  detect   the outlier pattern of one tensor (adahop_detect_pattern), what a calibration step does per tensor.

Operands follow the library's synthetic tensors: activations N(0, 1) with 16 channels x 50, weights N(0, 0.02), output
gradients N(0, 0.001) with 0.5 % of the token rows x 100.
"""
import math

import torch

from paper_2604_02525_amd import binding as ah

STRATEGIES = {"none": ah.ADAHOP_NONE, "iht": ah.ADAHOP_IHT, "oe_row": ah.ADAHOP_IHT_OE_ROW, "oe_col": ah.ADAHOP_IHT_OE_COL,
              "oe_k": ah.ADAHOP_IHT_OE_K}
BLOCKS = (32, 64, 128, 256)
# Layer widths of the library's configurations and benchmark workloads.
WIDTHS = (2048, 4096, 8192, 11008, 12288, 14336, 28672)
MAX_FLOPS = 2.0 * 16384 * 28672 * 8192
MAX_BYTES = 2.0 * (16384 + 28672) * 8192 + 4.0 * 16384 * 28672


def _product(direction, tokens, d_in, d_out, strategy, k, block, name=None, bf16_out=False, packed_w=False, sr=False):
    case = {"kind": "product", "direction": direction, "tokens": tokens, "d_in": d_in, "d_out": d_out, "strategy": strategy,
            "k": k, "block": block, "bf16_out": bf16_out, "packed_w": packed_w, "sr": sr}
    return dict(case, name=name) if name else case


def _layer(tokens, d_in, d_out, strategies, pct, block, name=None):
    case = {"kind": "layer", "tokens": tokens, "d_in": d_in, "d_out": d_out, "fwd": strategies[0], "dgrad": strategies[1],
            "wgrad": strategies[2], "pct": pct, "block": block}
    return dict(case, name=name) if name else case


def _tensor(kind, outer, K, k_contig, block=0, name=None):
    case = {"kind": kind, "outer": outer, "K": K, "k_contig": k_contig, "block": block}
    return dict(case, name=name) if name else case


def listed():
    return [
        # The smallest product of the library's configurations: launches and host work count.
        _product("fwd", 256, 256, 256, "iht", 0, 32, name="fwd_256"),
        # A micro-batch of few tokens against a weight that was packed once, bf16 activations out.
        _product("fwd", 96, 4096, 11008, "iht", 0, 128, name="fwd_96_packed_bf16", bf16_out=True, packed_w=True),
        # A packed batch of odd length through a layer whose widths are no multiples of the tiles.
        _product("fwd", 1000, 3040, 5000, "oe_k", 31, 32, name="fwd_ragged"),
        # Forward up-projection of a small model, channel outliers extracted.
        _product("fwd", 8192, 2048, 8192, "oe_k", 8, 128, name="fwd_8192_oe_k"),
        # Input gradient where whole token rows stand out: row extraction, 1 %.
        _product("dgrad", 8192, 4096, 4096, "oe_row", 82, 128, name="dgrad_8192_oe_row"),
        # A training step's three products of an attention projection.
        _layer(8192, 4096, 4096, ("oe_k", "oe_row", "oe_col"), 1.0, 128, name="layer_8192"),
        # The same for a feed-forward projection and a token count that is no multiple of the tiles (63 x 32).
        _layer(2016, 4096, 11008, ("oe_k", "oe_row", "oe_col"), 1.0, 32, name="layer_2016"),
        # Input gradient with stochastically rounded gradients and bf16 output.
        _product("dgrad", 8192, 4096, 11008, "iht", 0, 128, name="dgrad_8192_sr_bf16", bf16_out=True, sr=True),
        # Weight gradient over many tokens, column extraction: both operands K-strided.
        _product("wgrad", 32768, 4096, 4096, "oe_col", 64, 32, name="wgrad_32768_oe_col"),
        # The largest products of the library's benchmark.
        _product("fwd", 16384, 8192, 28672, "oe_k", 82, 256, name="fwd_16384_oe_k"),
        # A large weight packed by itself.
        _tensor("pack", 28672, 8192, True, 256, name="pack_28672"),
        # A calibration step's look at one large activation.
        _tensor("detect", 16384, 8192, True, name="detect_16384"),
    ]


def _shape(direction, tokens, d_in, d_out):
    """(M, N, K) of a product."""
    return {"fwd": (tokens, d_out, d_in), "dgrad": (tokens, d_in, d_out), "wgrad": (d_out, d_in, tokens)}[direction]


def _extracted_dim(strategy, M, N, K):
    return {"oe_row": M, "oe_col": N, "oe_k": K}.get(strategy, 0)


def _k(strategy, pct, M, N, K):
    """ceil(pct % of the extracted dimension)."""
    return int(math.ceil(pct * _extracted_dim(strategy, M, N, K) / 100.0 - 1e-9))


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng):
    """A layer width: one of the usual ones or any multiple of 32 from 256 to 28672."""
    return rng.choice(WIDTHS) if rng.random() < 0.4 else max(256, _log_int(rng, 256, 28672) // 32 * 32)


def _block(rng, *Ks):
    return rng.choice([b for b in BLOCKS if all(K % b == 0 for K in Ks)])


def draw(rng):
    while True:
        case = _draw(rng)
        w = work(case)
        if w["flops"] <= MAX_FLOPS and w["bytes"] <= MAX_BYTES:
            return case


def _draw(rng):
    what = rng.random()
    if what < 0.6:
        direction = rng.choice(("fwd", "dgrad", "wgrad"))
        tokens, d_in, d_out = _log_int(rng, 16, 32768), _width(rng), _width(rng)
        if direction == "wgrad":
            tokens = max(32, tokens // 32 * 32)     # the contraction: whole scaling blocks
        elif direction == "fwd" and rng.random() < 0.25:
            d_out += rng.randrange(32)              # a vocabulary-like width
        M, N, K = _shape(direction, tokens, d_in, d_out)
        strategy = rng.choice(("none", "iht", "iht", "oe_row", "oe_col", "oe_k"))
        packed = direction != "wgrad" and strategy in ("none", "iht", "oe_row") and rng.random() < 0.3
        sr = direction != "fwd" and rng.random() < 0.2
        return _product(direction, tokens, d_in, d_out, strategy, _k(strategy, rng.choice((0.25, 1.0, 2.0)), M, N, K),
                        _block(rng, K), bf16_out=rng.random() < 0.3, packed_w=packed, sr=sr)
    if what < 0.8:
        tokens, d_in, d_out = max(32, _log_int(rng, 64, 16384) // 32 * 32), _width(rng), _width(rng)
        strategies = (rng.choice(("iht", "oe_k")), rng.choice(("iht", "oe_row")), rng.choice(("iht", "oe_col", "oe_k")))
        return _layer(tokens, d_in, d_out, strategies, rng.choice((0.25, 1.0, 2.0)), _block(rng, tokens, d_in, d_out))
    outer, K = _log_int(rng, 64, 32768), _width(rng)
    k_contig = rng.random() < 0.5
    if not k_contig:
        outer = max(64, outer // 8 * 8)             # rows of the stored array are 16-byte pieces
    if what < 0.9:
        return _tensor("pack", outer, K, k_contig, _block(rng, K))
    return _tensor("detect", outer, K, k_contig)


def _normal(gen, rows, cols, std, rows_x=None, cols_x=None):
    """bf16 N(0, std^2) on the GPU; rows_x / cols_x = (count, factor): that many rows / columns amplified."""
    x = torch.randn(rows, cols, generator=gen, device="cuda", dtype=torch.float32).mul_(std)
    if rows_x:
        x[torch.randperm(rows, generator=gen, device="cuda")[:rows_x[0]]] *= rows_x[1]
    if cols_x:
        x[:, torch.randperm(cols, generator=gen, device="cuda")[:cols_x[0]]] *= cols_x[1]
    return x.to(torch.bfloat16)


def _activation(gen, tokens, d):
    return _normal(gen, tokens, d, 1.0, cols_x=(16, 50.0))


def _weight(gen, d_out, d_in):
    return _normal(gen, d_out, d_in, 0.02)


def _gradient(gen, tokens, d):
    return _normal(gen, tokens, d, 1e-3, rows_x=(int(math.ceil(0.005 * tokens)), 100.0))


def _operands(direction, X, W, G):
    if direction == "fwd":
        return ah.Operand(X, True), ah.Operand(W, True)
    if direction == "dgrad":
        return ah.Operand(G, True), ah.Operand(W, False)
    return ah.Operand(G, False), ah.Operand(X, False)


def _state_of_product(gen, case, workspace=None, X=None, W=None, G=None):
    """What a program keeps for one product: operands, output, workspace, the packed weight, the rounding seed."""
    direction, strategy, k = case["direction"], STRATEGIES[case["strategy"]], case["k"]
    tokens, d_in, d_out = case["tokens"], case["d_in"], case["d_out"]
    if X is None and direction != "dgrad":
        X = _activation(gen, tokens, d_in)
    if W is None and direction != "wgrad":
        W = _weight(gen, d_out, d_in)
    if G is None and direction != "fwd":
        G = _gradient(gen, tokens, d_out)
    A, B = _operands(direction, X, W, G)
    out = torch.empty((A.outer, B.outer), dtype=torch.bfloat16 if case["bf16_out"] else torch.float32, device="cuda")
    if workspace is None:
        workspace = torch.empty(ah.adahop_gemm_workspace_bytes(A.outer, B.outer, A.K, strategy, k), dtype=torch.uint8,
                                device="cuda")
    packed = ah.adahop_pack_operand(B, True, strategy, case["block"]) if case["packed_w"] else None
    return {"A": A, "B": B, "C": out, "workspace": workspace, "strategy": strategy, "block": case["block"], "k": k,
            "packed": packed, "sr_seed": gen.initial_seed() if case["sr"] else None}


def _layer_products(case):
    for direction in ("fwd", "dgrad", "wgrad"):
        strategy = case[direction]
        M, N, K = _shape(direction, case["tokens"], case["d_in"], case["d_out"])
        yield _product(direction, case["tokens"], case["d_in"], case["d_out"], strategy, _k(strategy, case["pct"], M, N, K),
                       case["block"])


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    if case["kind"] == "product":
        return {"products": [_state_of_product(gen, case)]}
    if case["kind"] == "layer":
        tokens, d_in, d_out = case["tokens"], case["d_in"], case["d_out"]
        X, W, G = _activation(gen, tokens, d_in), _weight(gen, d_out, d_in), _gradient(gen, tokens, d_out)
        products = list(_layer_products(case))
        need = max(ah.adahop_gemm_workspace_bytes(*_shape(p["direction"], tokens, d_in, d_out), STRATEGIES[p["strategy"]], p["k"])
                   for p in products)
        workspace = torch.empty(need, dtype=torch.uint8, device="cuda")     # the products run one after the other
        return {"products": [_state_of_product(gen, p, workspace, X, W, G) for p in products]}
    outer, K, k_contig = case["outer"], case["K"], case["k_contig"]
    x = _weight(gen, *((outer, K) if k_contig else (K, outer))) if case["kind"] == "pack" else None
    if case["kind"] == "pack":
        return {"pack": ah.Operand(x, k_contig), "block": case["block"],
                "codes": torch.empty((outer, K // 2), dtype=torch.uint8, device="cuda"),
                "scales": torch.empty((outer, K // 32), dtype=torch.uint8, device="cuda")}
    x = _activation(gen, *((outer, K) if k_contig else (K, outer)))
    op = ah.Operand(x, k_contig)
    need = int(ah.lib().adahop_detect_pattern_workspace_bytes(op.c()))
    return {"detect": op, "workspace": torch.empty(need, dtype=torch.uint8, device="cuda")}


def run(state):
    if "products" in state:
        got = []
        for p in state["products"]:
            r = ah.adahop_gemm(p["A"], p["B"], p["strategy"], p["block"], p["k"], Cout=p["C"], workspace=p["workspace"],
                               b_packed=p["packed"], sr_seed_a=p["sr_seed"])
            got.append({"C": r["C"], "idx": r["idx"]} if p["k"] else {"C": r["C"]})
        return got
    if "pack" in state:
        return ah.adahop_pack_operand(state["pack"], True, ah.ADAHOP_IHT, state["block"], codes=state["codes"],
                                      scales=state["scales"])
    return ah.adahop_detect_pattern(state["detect"], workspace=state["workspace"])


def _product_work(case):
    M, N, K = _shape(case["direction"], case["tokens"], case["d_in"], case["d_out"])
    extra = {"oe_row": case["k"] * N * K, "oe_col": M * case["k"] * K, "oe_k": M * N * case["k"]}.get(case["strategy"], 0)
    weight = (1 / 2 + 1 / 32) if case["packed_w"] else 2.0
    return {"bytes": 2.0 * M * K + weight * N * K + (2.0 if case["bf16_out"] else 4.0) * M * N,
            "flops": 2.0 * (M * N * K + extra)}


def work(case):
    if case["kind"] == "product":
        return _product_work(case)
    if case["kind"] == "layer":
        # X, W and G_Y are each an operand of two of the three products, which a program calls one by one.
        parts = [_product_work(p) for p in _layer_products(case)]
        return {"bytes": sum(p["bytes"] for p in parts), "flops": sum(p["flops"] for p in parts)}
    n = float(case["outer"]) * case["K"]
    if case["kind"] == "pack":
        # read bf16, write E2M1 codes and E8M0 scales; log2(block) butterfly additions per element
        return {"bytes": (2 + 1 / 2 + 1 / 32) * n, "flops": math.log2(case["block"]) * n}
    return {"bytes": 2.0 * n, "flops": 0.0}


def tolerance(case):
    """Largest differences between two correct implementations, from the products compared with the same sums in fp64."""
    if case["kind"] == "pack":
        return "exact"                              # codes and scales are defined bit for bit
    if case["kind"] == "detect":
        return {"rel": 1e-10, "max": 1e-9}          # fp64 sums over up to 2^28 values; the class is a whole number
    if case["kind"] == "product" and case["bf16_out"]:
        # one rounding of fp32 sums that differ in their last bits: about 1 value in 10^4 lands one bf16 step (up to
        # 2^-7 of the value) away
        return {"rel": 2e-4, "max": 8e-3}
    # fp32 sums over the same codes, scales and bf16 values: 2e-8 (K = 2048) .. 3e-7 (K = 32768, bf16 outlier columns)
    # from the fp64 sums, single values up to 1.8e-5 of the root mean square
    return {"rel": 1.2e-6, "max": 8e-5}
