"""What a user of this library has it do, as timed cases: quantized layers from one token to a long prefill in every
weight format, the linear layers of a decoder block, and the offline calibration of a layer.

`listed()` names the cases, `draw()` gives more of the same ranges; `prepare()` makes what a user's program holds before
the call, `run()` is one pass through the public entry points of `paper_2505_14638_amd`, `work()` states what the pass
cannot do without and `tolerance()` how far another correct implementation at the same precision may be off.
"""
import torch

from paper_2505_14638_amd import binding as B
from paper_2505_14638_amd.block import DecoderBlockLinears

GROUP = 128
FORMATS = ("code_exact", "two_level", "asym", "pow2", "asym_two_level")


def _layer(name, m, k, n, fmt="code_exact", group=GROUP, x="bf16", y="bf16", one_call=False):
    """A quantized layer: activations [m, k] of type `x` are quantized and multiplied with packed weights [n, k] of format
    `fmt`, output of type `y`.  group 0: one scale per output channel.  one_call: the entry point that quantizes its own
    input (up to 16 tokens, m * k <= 65536), otherwise w4a8_quantize_act and the layer."""
    return {"name": name, "kind": "layer", "m": m, "k": k, "n": n, "fmt": fmt, "group": group, "x": x, "y": y, "one_call": one_call}


def _block(name, m, hidden=4096, ffn=14336, qkv=6144):
    """The linear layers of a decoder block (QKV, O, gate|up with SiLU*mul, down) with the quantizations folded in."""
    return {"name": name, "kind": "block", "m": m, "hidden": hidden, "ffn": ffn, "qkv": qkv}


def _hessian(name, t, k, x="bf16"):
    """Offline calibration, first half: the Hessian of a layer of k features on t tokens and the factor of its inverse."""
    return {"name": name, "kind": "hessian", "t": t, "k": k, "x": x}


def _dpq(name, k, n, mse_grid=0):
    """Offline calibration, second half: the weights [n, k] quantized with error compensation, then packed.  mse_grid:
    candidates of the search over scales (0: none)."""
    return {"name": name, "kind": "dpq", "k": k, "n": n, "mse_grid": mse_grid}


def listed():
    return [
        # the smallest call: a toy-sized layer with per-channel scales in float32 throughout, where launches count
        _layer("single_8", 8, 1024, 1024, group=0, x="f32", y="f32"),
        # one token of one user through a whole 8B decoder block
        _block("block_1", 1),
        # a decode step of a batch of users
        _block("block_32", 32),
        # a large decode batch, or one chunk of a chunked prefill
        _block("block_128", 128),
        # a prompt
        _block("block_1024", 1024),
        # a decode step of a batch of users on the deepest layer of a 70B model
        _layer("decode_16_down_70b", 16, 28672, 8192),
        # sizes that no tile divides: a short prompt on a model of other widths, float32 in and out
        _layer("ragged_333", 333, 2944, 5003, x="f32", y="f32"),
        # a long prefill through the largest layer of an 8B block
        _layer("prefill_8192_gate_up", 8192, 4096, 28672),
        # the format that calibration produces (unsigned codes, zero-points, two levels of scales), in prefill
        _layer("prefill_2048_asym_two_level", 2048, 4096, 28672, fmt="asym_two_level"),
        # power-of-two group scales, in prefill on the deepest layer of an 8B block
        _layer("prefill_2048_pow2_down", 2048, 14336, 4096, fmt="pow2"),
        # offline: one square layer of an 8B block calibrated on 8192 tokens, in its two halves
        _hessian("hessian_4096", 8192, 4096),
        _dpq("dpq_4096", 4096, 4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(("layer",) * 6 + ("block",) * 3 + ("hessian", "dpq"))
    if kind == "block":
        hidden, ffn = 128 * _log_int(rng, 16, 32), 128 * _log_int(rng, 40, 112)
        return dict(_block("", _log_int(rng, 1, 1024), hidden, ffn, hidden + 256 * rng.randint(1, hidden // 256)), name=None)
    if kind == "hessian":
        return dict(_hessian("", _log_int(rng, 512, 8192), 128 * rng.randint(8, 32), rng.choice(("bf16", "f32"))), name=None)
    if kind == "dpq":
        return dict(_dpq("", 128 * rng.randint(8, 32), rng.randint(256, 4096), rng.choice((0, 20))), name=None)
    k, n = 128 * _log_int(rng, 8, 112), _log_int(rng, 512, 28672)
    if rng.random() < 0.5:                                      # half of the widths are round, as a model's usually are
        n = max(512, n // 128 * 128)
    m = _log_int(rng, 1, 8192)
    while m * n * k > 8192 * 4096 * 28672:
        m = max(1, m // 2)
    fmt = rng.choice(("code_exact",) * 4 + FORMATS[1:])
    one_call = fmt == "code_exact" and m <= 4 and m * k <= 65536 and rng.random() < 0.5
    return dict(_layer("", m, k, n, fmt, rng.choice((GROUP, GROUP, GROUP, 0)), rng.choice(("bf16", "f32")),
                       rng.choice(("bf16", "bf16", "f32")), one_call), name=None)


def _dtype(name):
    return torch.float32 if name == "f32" else torch.bfloat16


def _activations(gen, m, k, dtype):
    """N(0, 1) with 1 % of the channels twenty times as large: the outlier channels that force a large static scale."""
    x = torch.randn((m, k), generator=gen, device="cuda")
    cols = torch.randperm(k, generator=gen, device="cuda")[: max(1, round(0.01 * k))]
    x[:, cols] *= 20.0
    return x.to(dtype)


def _calibration_activations(gen, t, k, dtype):
    """Correlated features of unequal magnitude with outlier channels: what error compensation works on."""
    x = torch.randn((t, k), generator=gen, device="cuda")
    rank = 64
    x += 0.3 * torch.randn((t, rank), generator=gen, device="cuda") @ torch.randn((rank, k), generator=gen, device="cuda")
    x *= torch.exp(2.0 * torch.rand(k, generator=gen, device="cuda") - 1.0)
    cols = torch.randperm(k, generator=gen, device="cuda")[: max(1, round(0.01 * k))]
    x[:, cols] *= 20.0
    return x.to(dtype)


def _weights(gen, n, k):
    return torch.randn((n, k), generator=gen, device="cuda") * 0.02


def _prepare_layer(case, gen):
    m, k, n, fmt = case["m"], case["k"], case["n"], case["fmt"]
    group = case["group"] or k
    x = _activations(gen, m, k, _dtype(case["x"]))
    st = {"case": case, "group": group, "x": x, "s_x": B.calibrate_act_scale([x]),
          "x8": torch.empty((m, k), dtype=torch.uint8, device="cuda"),
          "y": torch.empty((m, n), dtype=_dtype(case["y"]), device="cuda"), "ws": None}
    if fmt in ("two_level", "asym_two_level"):
        # both levels: weights / w_out lie in the FP8 domain (|w8| <= 448), the group scales are those of that domain
        w = _weights(gen, n, k)
        w_out = w.abs().amax(dim=1) / 448.0
        w8 = (w / w_out[:, None]).reshape(n, k // group, group)
        if fmt == "two_level":
            s8 = w8.abs().amax(dim=2) / 7.0
            codes = torch.clamp(torch.round(w8 / s8[..., None]), -8, 7).to(torch.int8).reshape(n, k)
            st["packed"], st["scales"] = B.pack_weights(codes, group, B.LAYOUT_TILED, s8.contiguous())
        else:
            lo, hi = w8.amin(dim=2).clamp(max=0), w8.amax(dim=2).clamp(min=0)
            s8 = (hi - lo) / 15.0
            zero = torch.clamp(torch.round(-lo / s8), 0, 15)
            codes = torch.clamp(torch.round(w8 / s8[..., None] + zero[..., None]), 0, 15).to(torch.uint8).reshape(n, k)
            st["packed"], st["scales"] = B.pack_weights_asym(codes, group, s8.contiguous(), zero.to(torch.uint8).contiguous())
        st["w_out"] = w_out
    elif fmt == "asym":
        st["packed"], st["scales"] = B.pack_weights_asym(_weights(gen, n, k), group)
    else:
        st["packed"], st["scales"] = B.pack_weights(_weights(gen, n, k), group, B.LAYOUT_TILED, pow2=fmt == "pow2")
    if fmt == "code_exact" and not case["one_call"]:
        need = B.linear_workspace_bytes(m, k, n, group)
        st["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    return st


def _run_layer(st):
    case, n, group, fmt, y = st["case"], st["case"]["n"], st["group"], st["case"]["fmt"], st["y"]
    if case["one_call"]:
        return B.linear_quantize_in(st["x"], st["s_x"], st["packed"], st["scales"], n, group, out=y)
    x8 = B.quantize_act(st["x"], st["s_x"], out=st["x8"])
    if fmt == "code_exact":
        B.linear(x8, st["s_x"], st["packed"], st["scales"], n, group, B.LAYOUT_TILED, out=y, workspace=st["ws"])
    elif fmt == "two_level":
        B.linear_two_level(x8, st["s_x"], st["packed"], st["scales"], st["w_out"], n, group, out=y)
    elif fmt == "asym_two_level":
        B.linear_asym_two_level(x8, st["s_x"], st["packed"], st["scales"], st["w_out"], n, group, out=y)
    elif fmt == "asym":
        B.linear_asym(x8, st["s_x"], st["packed"], st["scales"], n, group, out=y)
    else:
        B.linear_pow2(x8, st["s_x"], st["packed"], st["scales"], n, group, out=y)
    return x8, y


def _prepare_block(case, gen):
    m, hidden, ffn = case["m"], case["hidden"], case["ffn"]
    blk = DecoderBlockLinears(hidden, ffn, case["qkv"], GROUP, "cuda", fused=True)
    x = _activations(gen, m, hidden, torch.bfloat16)
    h = x
    for name, (k, n) in blk.dims.items():                       # static scales from one unquantized-width pass, as in calibration
        blk.load_layer(name, _weights(gen, n, k))
        scale = B.calibrate_act_scale([h])
        blk.set_act_scale(name, float(scale))
        h = B.linear(B.quantize_act(h, scale), scale, *blk.weights[name], n, GROUP, B.LAYOUT_TILED)
        h = h[:, :hidden] if name == "qkv" else B.silu_mul(h) if name == "gate_up" else h
    return {"case": case, "block": blk, "x": x}


def _prepare_hessian(case, gen):
    x = _calibration_activations(gen, case["t"], case["k"], _dtype(case["x"]))
    # the visiting order is an input here: orders from sums that differ in the last bit could swap equal columns
    return {"case": case, "x": x, "perm": B.gar_permutation(x.double().square().sum(dim=0).float(), GROUP)}


def _run_hessian(st):
    h = B.hessian_accumulate(st["x"])
    u, info = B.hessian_inverse_factor(h, 0.01, st["perm"])
    return h, u, info


def _prepare_dpq(case, gen):
    n, k = case["n"], case["k"]
    x = _calibration_activations(gen, 2 * k, k, torch.float32).double()
    h = x.t().contiguous() @ x
    diag = h.diagonal().float().contiguous()
    perm = B.gar_permutation(diag, GROUP).long()
    h = h[perm][:, perm] + 0.01 * h.diagonal().mean() * torch.eye(k, dtype=torch.float64, device="cuda")
    # H^-1 = U^T U with U upper triangular: U = J L^-1 J, L the lower factor of J H J (J reverses the order)
    lower = torch.linalg.cholesky(h.flip(0, 1))
    eye = torch.eye(k, dtype=torch.float64, device="cuda")
    u = torch.linalg.solve_triangular(lower, eye, upper=False).flip(0, 1).float().contiguous()
    w = _weights(gen, n, k)
    return {"case": case, "w": w, "u": u, "diag": diag, "w_scale": w.abs().amax(dim=1) / 448.0}


def _run_dpq(st):
    perm = B.gar_permutation(st["diag"], GROUP)
    codes, scales, zeros = B.dpq_calibrate(st["w"], st["u"], st["w_scale"], GROUP, perm, st["case"]["mse_grid"])
    packed, params = B.pack_weights_asym(codes, GROUP, scales, zeros)
    return codes, scales, zeros, packed, params


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    return {"layer": _prepare_layer, "block": _prepare_block, "hessian": _prepare_hessian, "dpq": _prepare_dpq}[case["kind"]](case, gen)


def run(state):
    kind = state["case"]["kind"]
    if kind == "block":
        return state["block"].forward(state["x"])
    return {"layer": _run_layer, "hessian": _run_hessian, "dpq": _run_dpq}[kind](state)


def _weight_bytes(n, k, group, fmt="code_exact"):
    return n * k // 2 + n * (k // group) * (5 if fmt.startswith("asym") else 4)


def work(case):
    size = {"f32": 4, "bf16": 2}
    if case["kind"] == "block":
        m, h, f, q = case["m"], case["hidden"], case["ffn"], case["qkv"]
        dims = ((h, q), (h, h), (h, 2 * f), (f, h))
        return {"bytes": sum(_weight_bytes(n, k, GROUP) for k, n in dims) + 4 * m * h, "flops": sum(2 * m * k * n for k, n in dims)}
    if case["kind"] == "hessian":
        # symmetric and triangular results: t k^2 for X^T X, 2 k^3 / 3 for the factorization and the inverse of its factor
        t, k = case["t"], case["k"]
        return {"bytes": size[case["x"]] * t * k + 8 * k * k, "flops": t * k * k + 2 * k ** 3 // 3}
    if case["kind"] == "dpq":
        # a multiplication and a subtraction for every pair of columns q < v of every row
        k, n = case["k"], case["n"]
        return {"bytes": 4 * n * k + 2 * k * k + n * k + n * k // 2 + 10 * n * (k // GROUP), "flops": n * k * k}
    m, k, n = case["m"], case["k"], case["n"]
    return {"bytes": _weight_bytes(n, k, case["group"] or k, case["fmt"]) + size[case["x"]] * m * k + size[case["y"]] * m * n
            + (0 if case["one_call"] else m * k), "flops": 2 * m * k * n}


def tolerance(case):
    """Measured: the path against itself in 64 bits on the same quantized inputs (layers, blocks), or with its tokens in
    another order (Hessian); stated four times larger."""
    if case["kind"] == "dpq":
        return "exact"                                          # every step is one float32 operation in a fixed order
    if case["kind"] == "hessian":
        return {"rel": 1.5e-4, "max": 4e-3}                     # 3.8e-5 and 9e-4 on U, which carries the condition of H
    if case["kind"] == "block":
        # a last-bit difference in a bf16 intermediate moves some E4M3 codes of the next layer by a step: 2.1e-2, 0.22
        return {"rel": 3e-2, "max": 0.9}
    if case["y"] == "f32":
        return {"rel": 7e-5, "max": 2e-3}                       # 1.8e-5 and 4.4e-4: the matrix unit's own alignment of products
    return {"rel": 1.4e-3, "max": 1.6e-2}                       # 3.5e-4: single roundings to bf16 that fall the other way, one step each
