"""The work a training or serving program has libgws do, as measurable cases.

Four kinds of case, all through the public entry points of ``paper_2505_11170_amd``:

 ``sample``  the sampling passes over a list of weights, once per training step: forward (w_hat and scale, or
             microscaling codes) and, with ``bwd``, backward (dL/db_t or dL/db_i, and dL/dw copied or aliased).
 ``linear``  one sampled-weight linear: Y = X w_hat (``form`` says where w_hat is kept) and, with ``grad``, its
             input gradient ("x") or input and weight gradient ("xw").
 ``gemm``    the product on a weight that was sampled before (evaluation and serving: w_hat is kept).
 ``layer``   the five products of a decoder layer, several layers in a row, with the sampling of the coming weights
             riding in the products' launches.

Inputs are synthetic with the distributions that the passes meet: W ~ N(0, 0.02), b_t ~ U[4, 9] per block,
gradients ~ N(0, 1e-3), activations ~ N(0, 1), all from the seed.  ``exact`` computes the same outputs with torch in
64 bits and shares no code with the library.
"""
import math

import torch

import paper_2505_11170_amd as gws

DEV = "cuda:0"
FMT = {"bf16": gws.FMT_BF16, "fp8": gws.FMT_FP8_E4M3, "fp6": gws.FMT_FP6_E3M2}
BASIS = {"bits": gws.BASIS_BITS, "uniform": gws.BASIS_UNIFORM_BF16, "box_muller": gws.BASIS_BOX_MULLER}
STEP = 17          # index of the gradient update that the pass belongs to
B_INIT, B_TARGET, LAMBDA = 6.0, 4.0, 1e-4   # parametrised bitwidth (Eq. 11, Eq. 12)


# ---------------------------------------------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------------------------------------------
def _sample(blocks, hidden, qkv, mlp, gated, *, fmt="fp8", bwd=True, copy=False, bi=False, mx=False, basis="bits"):
    """The weights of `blocks` transformer blocks.  Plain: hidden x qkv, hidden x hidden, hidden x mlp, mlp x hidden.
    Gated: q hidden x hidden, k and v qkv x hidden, o, gate and up mlp x hidden, down hidden x mlp.
    mlp = 0: one hidden x qkv weight per block."""
    return {"kind": "sample", "blocks": blocks, "hidden": hidden, "qkv": qkv, "mlp": mlp, "gated": gated, "fmt": fmt,
            "bwd": bwd, "copy": copy, "bi": bi, "mx": mx, "basis": basis}


def _linear(M, K, N, *, nk=False, fmt="fp8", form="hat", grad=""):
    return {"kind": "linear", "M": M, "K": K, "N": N, "nk": nk, "fmt": fmt, "form": form, "grad": grad}


def _gemm(M, K, N, *, nk=False, fmt="fp8"):
    return {"kind": "gemm", "M": M, "K": K, "N": N, "nk": nk, "fmt": fmt}


def _layer(tokens, hidden, qkv, mlp, layers, fmt="fp8"):
    return {"kind": "layer", "M": tokens, "hidden": hidden, "qkv": qkv, "mlp": mlp, "layers": layers, "fmt": fmt}


def listed():
    return [
        # the smallest call: one attention output weight of the 124M model, forward; the launch is what it costs
        dict(_sample(1, 768, 768, 0, False, bwd=False), name="sample_one_768x768"),
        # one training step's sampling of the 124M model: 48 weights, forward and backward, gradients passed through
        dict(_sample(12, 768, 2304, 3072, False), name="sample_step_124m"),
        # the same for the 1B decoder: 154 weights of 22 layers, far beyond every cache
        dict(_sample(22, 2048, 256, 5632, True), name="sample_step_1b"),
        # a model whose widths are multiples of nothing the kernels are tiled for, parametrised bitwidth, FP6 target,
        # dL/dw wanted in a buffer of its own
        dict(_sample(8, 1000, 3000, 2700, False, fmt="fp6", copy=True, bi=True), name="sample_ragged_bi_fp6"),
        # deployment: the sampled weights of eight decoder layers as microscaling FP6 codes
        dict(_sample(8, 2048, 256, 5632, True, fmt="fp6", bwd=False, mx=True), name="export_mx_fp6"),
        # the comparison system of the paper's unit benchmark: rounded normal from a Box-Muller transform
        dict(_sample(1, 2048, 8192, 0, False, fmt="bf16", basis="box_muller"), name="box_muller_2048x8192"),
        # a few tokens through a sampled linear by a caller with no place for w_hat
        dict(_linear(16, 2048, 5632, form="bare"), name="linear_16_tokens"),
        # serving: a few tokens through a weight sampled before, stored [N x K]
        dict(_gemm(4, 5632, 2048, nk=True), name="gemm_4_tokens"),
        # a short, uneven batch: forward and input gradient of the 124M model's q/k/v weight, w_hat in a workspace
        dict(_linear(1000, 768, 2304, form="ws", grad="x"), name="linear_ragged_tokens"),
        # a training micro-batch of the 124M model's MLP: forward, input gradient, weight gradient with dL/db_t
        dict(_linear(4096, 768, 3072, grad="xw"), name="linear_step_124m_mlp"),
        # the same for the 1B model's gate weight over 8192 tokens
        dict(_linear(8192, 2048, 5632, grad="xw"), name="linear_step_1b_gate"),
        # the forward pass of two decoder layers over 8192 tokens, sampling riding in the products' launches
        dict(_layer(8192, 2048, 2560, 5632, 2), name="layers_1b_riding"),
    ]


def _log_int(rng, lo, hi, mult=1):
    return max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))) // mult * mult))


def draw(rng):
    kind = rng.choice(("sample", "sample", "linear", "linear", "gemm", "layer"))
    fmt = rng.choice(("fp8", "fp8", "fp6", "bf16"))
    if kind == "sample":
        # widths: half the time multiples of 64, as models have them, half the time whatever comes
        unit = rng.choice((64, 1))
        hidden = _log_int(rng, 256, 4096, unit)
        gated = rng.random() < 0.5
        mlp = int(hidden * rng.uniform(2.5, 4)) // unit * unit
        qkv = max(unit, hidden // rng.choice((1, 4, 8)) // unit * unit) if gated else 3 * hidden
        per_block = hidden * (2 * hidden + 2 * qkv + 3 * mlp) if gated else hidden * (qkv + hidden + 2 * mlp)
        blocks = _log_int(rng, 1, max(1, min(48, int(5e8 // per_block))))
        option = rng.choice(("", "", "copy", "bi", "mx", "box_muller", "uniform"))
        if option == "mx":
            return _sample(blocks, hidden, qkv, mlp, gated, fmt=rng.choice(("fp8", "fp6")), bwd=False, mx=True)
        if option in ("box_muller", "uniform"):
            return _sample(blocks, hidden, qkv, mlp, gated, fmt=fmt, basis=option)
        return _sample(blocks, hidden, qkv, mlp, gated, fmt=fmt, bwd=rng.random() < 0.8, copy=option == "copy", bi=option == "bi")
    nk = rng.random() < 0.5
    if kind == "layer":
        hidden = 256 * rng.randint(2, 8)
        return _layer(256 * _log_int(rng, 2, 32), hidden, hidden + 256 * rng.randint(1, 2), 256 * rng.randint(2, 22), rng.randint(1, 2), fmt)
    if kind == "gemm":
        return _gemm(_log_int(rng, 1, 4096), 32 * _log_int(rng, 16, 176), 32 * _log_int(rng, 16, 176), nk=nk, fmt=fmt)
    if rng.random() < 0.5:
        # training: tokens a multiple of 64, weights of whole 256 x 256 tiles
        return _linear(64 * _log_int(rng, 8, 128), 256 * _log_int(rng, 2, 16), 256 * _log_int(rng, 2, 16), nk=nk, fmt=fmt, grad="xw")
    return _linear(_log_int(rng, 1, 8192), 32 * _log_int(rng, 16, 96), 32 * _log_int(rng, 16, 128), nk=nk, fmt=fmt,
                   form=rng.choice(("hat", "ws", "static", "bare")), grad=rng.choice(("", "x")))


# ---------------------------------------------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------------------------------------------
def _shapes(case):
    h, q, f = case["hidden"], case["qkv"], case["mlp"]
    if not f:
        block = [(h, q)]
    elif case["gated"]:
        block = [(h, h), (q, h), (q, h), (h, h), (f, h), (h, f), (f, h)]
    else:
        block = [(h, q), (h, h), (h, f), (f, h)]
    return block * case["blocks"]


def _nb(n):
    return (n + 31) // 32


def _up8(n):
    return (n + 7) // 8 * 8


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _normal(gen, n, std):
    """n BF16 values of N(0, std), drawn a part at a time (the fp32 draws of a whole model would be twice the model)."""
    out = torch.empty(n, dtype=torch.bfloat16, device=DEV)
    part = 1 << 27
    for i in range(0, n, part):
        out[i:i + part] = torch.randn(min(part, n - i), generator=gen, device=DEV) * std
    return out


class _Arena:
    """Weights of a model behind one another in one buffer, as an optimizer keeps them: views by tensor."""

    def __init__(self, sizes, dtype, data=None, align=128):
        self.off, n = [], 0
        for s in sizes:
            self.off.append(n)
            n += (s + align - 1) // align * align
        self.flat = torch.zeros(n, dtype=dtype, device=DEV) if data is None else data(n)
        self.sizes = sizes

    def __getitem__(self, i):
        return self.flat[self.off[i]:self.off[i] + self.sizes[i]]


def _weight_seed(seed, i):
    return gws.gws_derive_seed(int(seed), i)


def prepare(case, seed):
    return {"sample": _prepare_sample, "linear": _prepare_linear, "gemm": _prepare_gemm, "layer": _prepare_layer}[case["kind"]](case, seed)


def _prepare_sample(case, seed):
    gen, shapes = _gen(seed), _shapes(case)
    elems = [r * _up8(c) for r, c in shapes]
    blocks = [_nb(r) * _nb(c) for r, c in shapes]
    w = _Arena(elems, torch.bfloat16, lambda n: _normal(gen, n, 0.02))
    # b_t ~ U[4, 9], or the parameter b_i ~ U[0, 2] that Eq. 11 maps into the same range
    bt = _Arena(blocks, torch.float32, lambda n: torch.rand(n, generator=gen, device=DEV) * 2 if case["bi"] else 4 + 5 * torch.rand(n, generator=gen, device=DEV))
    scale = _Arena(blocks, torch.float32)
    s = {"case": case, "seed": seed, "shapes": shapes, "w": w, "bt": bt, "scale": scale, "fmt": FMT[case["fmt"]], "basis": BASIS[case["basis"]]}
    descs, outs = [], []
    if case["mx"]:
        s["ldc"] = [_up8(c) if case["fmt"] == "fp8" else ((c * 6 + 7) // 8 + 1) // 2 * 2 for _, c in shapes]
        s["codes"] = _Arena([r * l for (r, _), l in zip(shapes, s["ldc"])], torch.uint8, align=256)
        s["xscale"] = _Arena(blocks, torch.uint8)
    else:
        s["w_hat"] = _Arena(elems, torch.bfloat16)
    if case["bwd"]:
        s["g"] = _Arena(elems, torch.bfloat16, lambda n: _normal(gen, n, 1e-3))
        s["dbt"] = _Arena(blocks, torch.float32)
        s["dw"] = _Arena(elems, torch.bfloat16) if case["copy"] else s["g"]
    for i, (r, c) in enumerate(shapes):
        d = gws.TensorDesc(rows=r, cols=c, ld=_up8(c), seed=_weight_seed(seed, i), w=w[i], bt=bt[i], scale=scale[i])
        if case["mx"]:
            outs.append(gws.MxOut(s["codes"][i], s["xscale"][i], s["ldc"][i]))
        else:
            d.w_hat = s["w_hat"][i]
        if case["bwd"]:
            d.g, d.dw, d.dbt = s["g"][i], s["dw"][i], s["dbt"][i]
        descs.append(d)
    s["pack"] = gws.pack(descs)
    if case["mx"]:
        s["mx"] = gws.pack_mx(outs)
    if case["bi"]:
        s["bw"] = gws.pack_bitwidth([gws.Bitwidth(B_INIT, B_TARGET, LAMBDA)] * len(shapes))
    return s


def _weight(gen, K, N, nk, seed, i):
    r, c = (N, K) if nk else (K, N)
    return gws.TensorDesc(rows=r, cols=c, seed=_weight_seed(seed, i), w=_normal(gen, r * c, 0.02).view(r, c),
                          bt=4 + 5 * torch.rand(_nb(r), _nb(c), generator=gen, device=DEV))


def _hat(d):
    d.w_hat = torch.zeros_like(d.w)
    d.scale = torch.zeros(_nb(d.rows), _nb(d.cols), device=DEV)
    return d


def _prepare_linear(case, seed):
    gen = _gen(seed)
    M, K, N = case["M"], case["K"], case["N"]
    s = {"case": case, "seed": seed, "x": _normal(gen, M * K, 1.0).view(M, K), "y": torch.zeros(M, N, dtype=torch.bfloat16, device=DEV)}
    d = s["d"] = _weight(gen, K, N, case["nk"], seed, 0)
    if case["form"] == "hat":
        _hat(d)
    if case["form"] == "ws":
        s["ws"] = torch.empty(gws.gws_linear_fwd_workspace_bytes(d), dtype=torch.uint8, device=DEV)
    if case["grad"]:
        s["dy"] = _normal(gen, M * N, 1e-3).view(M, N)
        s["dx"] = torch.zeros(M, K, dtype=torch.bfloat16, device=DEV)
        if case["form"] != "hat":      # the input gradient needs the w_hat of the step: kept from an earlier call
            s["kept"] = gws.TensorDesc(rows=d.rows, cols=d.cols, seed=d.seed, w=d.w, bt=d.bt)
            _hat(s["kept"])
            gws.gws_sample_fwd([s["kept"]], FMT[case["fmt"]], STEP)
    if case["grad"] == "xw":
        d.dw = torch.zeros_like(d.w)
        d.dbt = torch.zeros_like(d.scale)
        n = gws.gws_linear_bwd_w_workspace_bytes(d, M)
        s["bws"] = torch.empty(n, dtype=torch.uint8, device=DEV) if n else None
    return s


def _prepare_gemm(case, seed):
    gen = _gen(seed)
    M, K, N = case["M"], case["K"], case["N"]
    d = _hat(_weight(gen, K, N, case["nk"], seed, 0))
    gws.gws_sample_fwd([d], FMT[case["fmt"]], STEP)
    return {"case": case, "seed": seed, "d": d, "x": _normal(gen, M * K, 1.0).view(M, K), "y": torch.zeros(M, N, dtype=torch.bfloat16, device=DEV)}


def _layer_weights(case):
    h, q, f = case["hidden"], case["qkv"], case["mlp"]
    return (("qkv", h, q), ("o", h, h), ("gate", h, f), ("up", h, f), ("down", f, h))


def _prepare_layer(case, seed):
    gen = _gen(seed)
    s = {"case": case, "seed": seed, "x": {}, "layers": [], "y": []}
    for n, k, _ in _layer_weights(case):
        s["x"][n] = _normal(gen, case["M"] * k, 1.0).view(case["M"], k)
    for l in range(case["layers"]):
        s["layers"].append({n: _hat(_weight(gen, k, m, False, seed, 5 * l + i)) for i, (n, k, m) in enumerate(_layer_weights(case))})
        s["y"].append({n: torch.zeros(case["M"], m, dtype=torch.bfloat16, device=DEV) for n, _, m in _layer_weights(case)})
    return s


# ---------------------------------------------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------------------------------------------
def run(s):
    return {"sample": _run_sample, "linear": _run_linear, "gemm": _run_gemm, "layer": _run_layer}[s["case"]["kind"]](s)


def _run_sample(s):
    case = s["case"]
    if case["mx"]:
        gws.gws_sample_fwd_mx(s["pack"], s["mx"], s["fmt"], STEP)
        return {"codes": s["codes"].flat, "xscale": s["xscale"].flat, "scale": s["scale"].flat}
    if case["bi"]:
        gws.gws_sample_fwd_bi(s["pack"], s["bw"], s["fmt"], STEP)
    elif case["basis"] != "bits":
        gws.gws_sample_fwd_basis(s["pack"], s["basis"], s["fmt"], STEP)
    else:
        gws.gws_sample_fwd(s["pack"], s["fmt"], STEP)
    out = {"w_hat": s["w_hat"].flat, "scale": s["scale"].flat}
    if case["bwd"]:
        if case["bi"]:
            gws.gws_sample_bwd_bi(s["pack"], s["bw"], STEP)
        elif case["basis"] != "bits":
            gws.gws_sample_bwd_basis(s["pack"], s["basis"], STEP)
        else:
            gws.gws_sample_bwd(s["pack"], STEP)
        out["dbt"] = s["dbt"].flat
        if case["copy"]:
            out["dw"] = s["dw"].flat
    return out


def _run_linear(s):
    case, d, fmt = s["case"], s["d"], FMT[s["case"]["fmt"]]
    if case["form"] == "ws":
        gws.gws_linear_fwd_ws(s["x"], d, s["y"], fmt, STEP, s["ws"], w_is_nk=case["nk"])
    elif case["form"] == "static":
        gws.gws_linear_fwd_static(s["x"], d, s["y"], fmt, STEP, w_is_nk=case["nk"])
    else:
        gws.gws_linear_fwd(s["x"], d, s["y"], fmt, STEP, w_is_nk=case["nk"])
    out = {"y": s["y"]}
    if case["form"] == "hat":
        out["w_hat"], out["scale"] = d.w_hat, d.scale
    if case["grad"]:
        gws.gws_gemm_bf16(s["dy"], (s.get("kept") or d).w_hat, s["dx"], w_is_nk=not case["nk"])
        out["dx"] = s["dx"]
    if case["grad"] == "xw":
        gws.gws_linear_bwd_w_ws(s["x"], s["dy"], d, STEP, s["bws"], w_is_nk=case["nk"])
        out["dw"], out["dbt"] = d.dw, d.dbt
    return out


def _run_gemm(s):
    gws.gws_gemm_bf16(s["x"], s["d"].w_hat, s["y"], w_is_nk=s["case"]["nk"])
    return {"y": s["y"]}


def _run_layer(s):
    layers, fmt = s["layers"], FMT[s["case"]["fmt"]]
    gws.gws_sample_fwd([layers[0]["qkv"]], fmt, STEP)
    for l, w in enumerate(layers):
        carried = {"qkv": [w["o"], w["gate"]] + ([layers[l + 1]["qkv"]] if l + 1 < len(layers) else []), "gate": [w["up"]], "up": [w["down"]]}
        for n in w:
            gws.gws_gemm_bf16_sample_next_n(s["x"][n], w[n].w_hat, s["y"][l][n], carried.get(n, []), fmt, STEP)
    return {"y": [[y[n] for n in y] for y in s["y"]], "w_hat": [[w[n].w_hat for n in w] for w in layers]}


# ---------------------------------------------------------------------------------------------------------------
# What a pass cannot do without, and what its results may differ by
# ---------------------------------------------------------------------------------------------------------------
def work(case):
    if case["kind"] == "sample":
        n = sum(r * c for r, c in _shapes(case))
        blocks = sum(_nb(r) * _nb(c) for r, c in _shapes(case))
        out = (1.0 if case["fmt"] == "fp8" else 0.75) if case["mx"] else 2.0
        nbytes = (2 + out) * n + (9 if case["mx"] else 8) * blocks
        if case["bwd"]:
            nbytes += (4 if case["copy"] else 2) * n + (12 if case["bi"] else 8) * blocks
        return {"bytes": nbytes, "flops": 0.0}
    M = case["M"]
    if case["kind"] == "layer":
        kn = [(k, n) for _, k, n in _layer_weights(case)]
        return {"bytes": case["layers"] * sum(2.0 * M * (k + n) + 4.0 * k * n + 8 * _nb(k) * _nb(n) for k, n in kn),
                "flops": case["layers"] * sum(2.0 * M * k * n for k, n in kn)}
    K, N = case["K"], case["N"]
    blocks = _nb(K) * _nb(N)
    nbytes, flops = 2.0 * (M * K + K * N + M * N), 2.0 * M * K * N
    if case["kind"] == "gemm":
        return {"bytes": nbytes, "flops": flops}
    nbytes += 4 * blocks + ((2 * K * N + 4 * blocks) if case["form"] == "hat" else 0)
    grads = len(case["grad"])
    # dX: dY and w_hat in, dX out; dW: X and dY again, dW and dL/db_t out
    nbytes += (2.0 * (M * N + K * N + M * K) if grads else 0) + (2.0 * (M * N + M * K + K * N) + 8 * blocks if grads == 2 else 0)
    return {"bytes": nbytes, "flops": flops * (1 + grads)}


def tolerance(case):
    # w_hat, codes and scales are the same bits for every implementation; dL/db_t is an fp32 sum of 1024 signed terms
    if case["kind"] == "sample":
        return {"rel": 5e-7, "max": 1e-4} if case["bwd"] else "exact"
    # BF16 results of fp32 sums: another order of the sums moves a result across a rounding boundary now and then
    return {"rel": 2e-3, "max": 2e-2}


# ---------------------------------------------------------------------------------------------------------------
# The same in 64 bits (plain torch)
# ---------------------------------------------------------------------------------------------------------------
def _mul_hi_lo(a, m):
    """High and low 32 bits of a * m for int64 tensors (or ints) below 2^32."""
    lo = (a * m) & 0xFFFFFFFF if not torch.is_tensor(a) else (a * (m & 0xFFFF) + (((a * (m >> 16)) & 0xFFFF) << 16)) & 0xFFFFFFFF
    hi = (a * (m >> 16) + ((a * (m & 0xFFFF)) >> 16)) >> 16
    return hi & 0xFFFFFFFF, lo


def _philox(rows, groups, seed):
    """Philox4x32-10 words [rows, groups] x 4 for the counters (group, row, step, 0)."""
    c0 = torch.arange(groups, device=DEV, dtype=torch.int64)[None, :].expand(rows, groups)
    c1 = torch.arange(rows, device=DEV, dtype=torch.int64)[:, None].expand(rows, groups)
    c2 = torch.full_like(c0, STEP)
    c3 = torch.zeros_like(c0)
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        h0, l0 = _mul_hi_lo(c0, 0xD2511F53)
        h1, l1 = _mul_hi_lo(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c0, c1, c2, c3


def _noise(rows, cols, seed, basis):
    """R [rows, cols] as float64 (the sign of a zero is lost: it only matters for w = -0)."""
    groups = (cols + 7) // 8
    x = _philox(rows, groups, seed)
    out = torch.empty(rows, groups, 8, dtype=torch.float64, device=DEV)
    for k in range(8):
        if basis == "bits":
            n = [(v >> (4 * ((k >> 1) + 4 * (k & 1)))) & 15 for v in x]
            two = (n[0] == 15) & (n[1] == 15) & ((n[2] & 3) != 0)
            one = ((n[2] & 12) != 0) & ((n[3] & 3) != 0) & ((n[3] & 4) != 0) & ~two
            out[:, :, k] = (two * 2 + one * 1) * (1 - 2 * (n[3] >> 3))
        elif basis == "uniform":
            out[:, :, k] = (2 * ((x[k // 4] >> (8 * (k % 4))) & 255) - 255).double() / 512
        else:
            u1 = ((x[k // 2] & 0xFFFF).double() + 0.5) / 65536
            u2 = ((x[k // 2] >> 16).double() + 0.5) / 65536
            z = torch.sqrt(-2 * torch.log(u1)) * (torch.sin if k & 1 else torch.cos)(2 * math.pi * u2)
            out[:, :, k] = torch.round(z / 2)
    return out.view(rows, groups * 8)[:, :cols]


def _per_block(v, rows, cols):
    return v.view(_nb(rows), _nb(cols)).repeat_interleave(32, 0).repeat_interleave(32, 1)[:rows, :cols]


def _block_view(v, rows, cols):
    """[block rows, 32, block columns, 32], zeros past the edges."""
    p = torch.zeros(_nb(rows) * 32, _nb(cols) * 32, dtype=v.dtype, device=DEV)
    p[:rows, :cols] = v
    return p.view(_nb(rows), 32, _nb(cols), 32)


def _sampled(w, bt, seed, fmt, basis="bits"):
    """(w_hat, scale, R) of a weight, everything in float64."""
    rows, cols = w.shape
    w = w.double()
    a = _block_view(w.abs(), rows, cols).amax((1, 3))
    s32 = a * torch.exp2(1 - bt.double().view_as(a))
    s = s32.float().to(torch.bfloat16).double()
    r = _noise(rows, cols, seed, basis)
    pqn = (r * _per_block(s, rows, cols)).float().to(torch.bfloat16).double()
    v = (w + pqn).float().to(torch.bfloat16).double()
    emax, emin, m, top = {"bf16": (0, 0, 0, 0), "fp8": (8, -6, 3, 448.0), "fp6": (4, -2, 2, 28.0)}[fmt]
    X = torch.exp2(torch.floor(torch.log2(a.clamp(min=2.0 ** -100))) + 1 - emax)
    if fmt != "bf16":
        q = v / _per_block(X, rows, cols)
        e = torch.floor(torch.log2(q.abs().clamp(min=2.0 ** emin))).clamp(min=emin)
        q = (torch.round(q / torch.exp2(e - m)) * torch.exp2(e - m)).clamp(-top, top)
        v = q * _per_block(X, rows, cols)
    return v, s32, r


def exact(case, seed):
    s = prepare(case, seed)
    return {"sample": _exact_sample, "linear": _exact_linear, "gemm": _exact_gemm, "layer": _exact_layer}[case["kind"]](case, s)


def _exact_sample(case, s):
    if sum(r * c for r, c in s["shapes"]) > 4e8 or case["mx"]:
        return None      # many seconds of integer arithmetic; codes are bytes, which are compared as they are
    out = {n: torch.zeros(s[n].flat.numel(), dtype=torch.float64, device=DEV) for n in ("w_hat", "scale")}
    if case["bwd"]:
        out["dbt"] = torch.zeros(s["dbt"].flat.numel(), dtype=torch.float64, device=DEV)
    for i, (r, c) in enumerate(s["shapes"]):
        ld = _up8(c)
        bt = s["bt"][i]
        if case["bi"]:
            bt = B_TARGET + bt * (B_INIT - B_TARGET)
        v, s32, noise = _sampled(s["w"][i].view(r, ld)[:, :c], bt, _weight_seed(s["seed"], i), case["fmt"], case["basis"])
        lo, n = s["w_hat"].off[i], r * ld
        out["w_hat"][lo:lo + n].view(r, ld)[:, :c] = v
        lo, n = s["scale"].off[i], _nb(r) * _nb(c)
        out["scale"][lo:lo + n] = s32.flatten()
        if case["bwd"]:
            g = s["g"][i].view(r, ld)[:, :c].double()
            grad = -math.log(2) * s32 * _block_view(g * noise, r, c).sum((1, 3))
            if case["bi"]:
                grad = (B_INIT - B_TARGET) * (grad + LAMBDA / n * torch.sign(bt.double().view_as(grad) - B_TARGET))
            out["dbt"][lo:lo + n] = grad.flatten()
    if case["copy"]:
        dw = torch.zeros(s["dw"].flat.numel(), dtype=torch.float64, device=DEV)
        for i, (r, c) in enumerate(s["shapes"]):
            lo, ld = s["dw"].off[i], _up8(c)
            dw[lo:lo + r * ld].view(r, ld)[:, :c] = s["g"][i].view(r, ld)[:, :c].double()
        out["dw"] = dw
    return out


def _product(a, b):
    """a b in float64, a part of the rows at a time."""
    return torch.cat([a[i:i + 2048].double() @ b for i in range(0, a.shape[0], 2048)])


def _exact_linear(case, s):
    d = s["d"]
    v, s32, r = _sampled(d.w, d.bt, d.seed, case["fmt"])
    kn = v.t().contiguous() if case["nk"] else v
    out = {"y": _product(s["x"], kn)}
    if case["form"] == "hat":
        out["w_hat"], out["scale"] = v, s32
    if case["grad"]:
        out["dx"] = _product(s["dy"], kn.t().contiguous())
    if case["grad"] == "xw":
        a, b = (s["dy"], s["x"]) if case["nk"] else (s["x"], s["dy"])
        dw = a.t().contiguous().double() @ b.double()
        out["dw"] = dw
        # Eq. 4 on the gradient as it is stored, in BF16
        out["dbt"] = -math.log(2) * s32 * _block_view(dw.float().to(torch.bfloat16).double() * r, d.rows, d.cols).sum((1, 3))
    return out


def _exact_gemm(case, s):
    d = s["d"]
    v = _sampled(d.w, d.bt, d.seed, case["fmt"])[0]
    return {"y": _product(s["x"], v.t().contiguous() if case["nk"] else v)}


def _exact_layer(case, s):
    names = [n for n, _, _ in _layer_weights(case)]
    hats = [[_sampled(w[n].w, w[n].bt, w[n].seed, case["fmt"])[0] for n in names] for w in s["layers"]]
    return {"y": [[_product(s["x"][n], h) for n, h in zip(names, row)] for row in hats], "w_hat": hats}
