"""Work that users of the tolerance engine have it do, through its public entry points.

A verifier re-executes traced FP32 operators and checks the proposer's claimed outputs against them:
for each operator a bound is formed and the claim is checked and profiled.  The cases below are such
operators, alone or in the small groups in which they occur, from the smallest single call to the
large operators of a decoder layer's prefill; one more is the adversary's side of the protocol, the
projection of a perturbation onto the admissible sets.

`prepare` makes what the verifier's program has in hand before the call: operands, its own outputs,
the claims, prepared images of committed weights (they never change), result buffers and
workspaces.  Activations arrive anew with every request, so their images are made inside `run`.
Everything is synthetic and made on the GPU from the seed.
"""
import ctypes
import math

import torch

import paper_2510_16028_amd as tao

U = 2.0 ** -24


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # one small linear layer, checked alone: launches and latency are all there is
        dict(name="linear_small", kind="linear", M=64, K=256, N=128, bias=False, route="stored", claim="honest"),
        # a decode step's projection: a handful of tokens against a large committed weight
        dict(name="linear_decode", kind="linear", M=8, K=4096, N=4096, bias=False, route="stored", claim="honest"),
        # the up projection of an encoder block at sequence length 512, weight prepared once
        dict(name="linear_encoder", kind="linear", M=512, K=768, N=3072, bias=True, route="prepared", claim="honest"),
        # sizes that fit no tile and no vector, both operands new, a proposer that leaves the bound in places
        dict(name="linear_ragged", kind="linear", M=1111, K=1001, N=3001, bias=True, route="checked", claim="perturbed"),
        # the gate projection of a decoder layer's prefill, sequence length 2048
        dict(name="linear_prefill", kind="linear", M=2048, K=4096, N=12288, bias=False, route="prepared", claim="honest"),
        # attention of an encoder block: scores, softmax and context of 12 heads
        dict(name="attention_encoder", kind="attention", heads=12, group=1, seq=512, dim=64, causal=False),
        # causal attention of a decoder layer with grouped queries (32 query heads on 8 key heads)
        dict(name="attention_decoder", kind="attention", heads=8, group=4, seq=2048, dim=128, causal=True),
        # normalisations: an encoder block's and a decoder layer's
        dict(name="layernorm_encoder", kind="norm", norm="layernorm", rows=512, cols=768),
        dict(name="rmsnorm_decoder", kind="norm", norm="rmsnorm", rows=2048, cols=4096),
        # the gated activation of a decoder layer: SiLU, then the product with the other branch
        dict(name="gated_decoder", kind="act", act="silu_mul", n=2048 * 12288),
        # a residual stage of a convolutional network: 3 x 3 convolution and the folded batch norm
        dict(name="conv_stage", kind="conv", batch=32, size=56, C=256, Cout=256, filter=3, stride=1),
        # one step of the adversary: error profile of a tentative output, then both projections
        dict(name="projection", kind="project", n=2048 * 4096),
    ]


def _spread(rng, lo, hi):
    """A whole number in [lo, hi], even over its logarithm, odd ones among them."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "attention", "norm", "act", "conv", "project"])
    if kind == "linear":
        while True:
            M, K, N = _spread(rng, 1, 2048), _spread(rng, 32, 8192), _spread(rng, 32, 12288)
            if rng.random() < 0.5:                      # widths of real layers are mostly multiples of 64
                K, N = (K + 63) // 64 * 64, (N + 63) // 64 * 64
            if M * K * N <= 2048 * 4096 * 12288:
                break
        route = "stored" if M < 256 else rng.choice(["prepared", "checked"])
        return dict(kind=kind, M=M, K=K, N=N, bias=rng.random() < 0.5, route=route,
                    claim=rng.choice(["honest", "honest", "perturbed"]) if K >= 256 and M * K * N <= 1 << 33 else "honest")
    if kind == "attention":
        while True:
            c = dict(kind=kind, heads=rng.choice([1, 2, 4, 8, 12, 16]), group=rng.choice([1, 1, 4]), seq=_spread(rng, 32, 2048),
                     dim=rng.choice([32, 64, 80, 96, 128]), causal=rng.random() < 0.6)
            if c["heads"] * c["group"] * c["seq"] ** 2 <= 32 * 2048 ** 2:
                return c
    if kind == "norm":
        cols = _spread(rng, 32, 12288)
        return dict(kind=kind, norm=rng.choice(["layernorm", "rmsnorm"]), rows=_spread(rng, 1, max(1, (1 << 24) // cols)), cols=cols)
    if kind == "act":
        return dict(kind=kind, act=rng.choice(["gelu", "gelu_tanh", "silu_mul", "add"]), n=_spread(rng, 1000, 2048 * 12288))
    if kind == "conv":
        while True:
            c = dict(kind=kind, batch=_spread(rng, 1, 32), size=_spread(rng, 7, 112), C=rng.choice([3, 32, 64, 100, 128, 256, 512]),
                     Cout=rng.choice([64, 96, 128, 256, 512]), filter=rng.choice([1, 3, 3, 7]), stride=rng.choice([1, 1, 2]))
            if c["filter"] == 7 and c["C"] != 3:
                continue
            if c["batch"] * c["size"] ** 2 * c["C"] * c["Cout"] * c["filter"] ** 2 <= 32 * 56 * 56 * 256 * 256 * 9:
                return c
    return dict(kind=kind, n=_spread(rng, 1000, 2048 * 4096))


# ------------------------------------------------------------------ inputs

def _randn(g, shape, std=1.0):
    return torch.randn(shape, generator=g, device=g.device) * std


def _product(A, Wkn, slabs):
    """A @ W in FP32, the reduction in `slabs` parts that are then added (another correct execution for slabs > 1)."""
    K = A.shape[-1]
    step = (K + slabs - 1) // slabs
    acc = None
    for k in range(0, K, step):
        part = torch.matmul(A[..., k:k + step].contiguous(), Wkn[..., k:k + step, :].contiguous())
        acc = part if acc is None else acc.add_(part)
    return acc


def _profile_buffer():
    # (zeroed: the struct has four bytes of padding, which the library has no reason to write)
    return tao.new_profile_buffer(torch.device("cuda", torch.cuda.current_device())).zero_()


def _scratch(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def _prepare_linear(c, g):
    M, K, N = c["M"], c["K"], c["N"]
    A, W = _randn(g, (M, K)), _randn(g, (N, K), 0.02)
    bias = _randn(g, (N,), 0.02) if c["bias"] else None
    Wkn = W.t().contiguous()
    y = _product(A, Wkn, 1)
    claimed = _product(A, Wkn, 4)
    if bias is not None:
        y += bias
        claimed += bias
    if c["claim"] == "perturbed":
        # +- f times the bound, f in {0, 0.5, 0.9, 1.1}: well inside, inside and outside
        k = K + (1 if bias is not None else 0)
        tau = A.double().abs() @ Wkn.double().abs()
        if bias is not None:
            tau += bias.double().abs()
        tau *= k * U / (1 - k * U)
        f = torch.tensor([0.0, 0.5, 0.9, 1.1, -0.5, -0.9, -1.1, 0.0], dtype=torch.float64, device="cuda")
        claimed = (y.double() + f[torch.randint(0, 8, y.shape, generator=g, device="cuda")] * tau).float()
    s = dict(A=A, bias=bias, y=y, claimed=claimed, out=_profile_buffer())
    if c["route"] == "stored":
        s.update(W=W, tau=torch.empty_like(y), ws=_scratch(tao.tao_check_workspace_bytes(y.numel())))
    elif c["route"] == "checked":
        s.update(W=W, ws=_scratch(tao.tao_bound_check_linear_workspace_bytes(M, N, K)))
    else:
        s.update(W_image=tao.tao_split_operand(W), A_image=_scratch(tao.tao_split_image_bytes(M, K)),
                 ws=_scratch(tao.lib().tao_check_linear_images_workspace_bytes(M, N, K, 1)))
    return s


def _run_linear(c, s):
    if c["route"] == "stored":
        tao.tao_bound_linear(s["A"], s["W"], s["bias"], out=s["tau"])
        tao.tao_check_and_profile(s["claimed"], s["y"], s["tau"], out=s["out"], ws=s["ws"], readback=False)
        return [s["tau"], s["out"]]
    if c["route"] == "checked":
        return [tao.tao_bound_check_linear(s["A"], s["W"], s["bias"], s["y"], s["claimed"], out=s["out"], ws=s["ws"], readback=False)]
    tao.tao_split_operand(s["A"], out=s["A_image"])
    return [tao.tao_bound_check_linear_images(s["A_image"], s["W_image"], c["M"], c["N"], c["K"], s["y"], s["claimed"], bias=s["bias"],
                                              out=s["out"], ws=s["ws"], readback=False)]


def _prepare_attention(c, g):
    B, rows, S, D = c["heads"], c["group"] * c["seq"], c["seq"], c["dim"]
    q, k, v = _randn(g, (B, rows, D), D ** -0.5), _randn(g, (B, S, D)), _randn(g, (B, S, D))
    kt = k.transpose(1, 2).contiguous()
    scores, scores_claimed = _product(q, kt, 1), _product(q, kt, 4)
    x = scores
    if c["causal"]:
        # the query heads of a group are stacked along the rows: row r is position r mod S
        above = torch.arange(S, device="cuda")[None, :] > (torch.arange(rows, device="cuda") % S)[:, None]
        x = scores.masked_fill(above[None], float("-inf"))
    e = torch.exp(x - x.amax(dim=-1, keepdim=True))
    p = e / e.sum(dim=-1, keepdim=True)
    p_claimed = e / e.flip(-1).contiguous().sum(dim=-1, keepdim=True)
    ctx, ctx_claimed = _product(p, v, 1), _product(p, v, 8)
    return dict(q=q, k=k, v=v, scores=scores, scores_claimed=scores_claimed, x=x, p=p, p_claimed=p_claimed, ctx=ctx, ctx_claimed=ctx_claimed,
                out=[_profile_buffer() for _ in range(3)],
                ws=_scratch(max(tao.tao_bound_check_linear_workspace_bytes(rows, S, D, B, B == 1), tao.tao_check_workspace_bytes(p.numel()),
                                tao.tao_bound_check_linear_workspace_bytes(rows, D, S, B, B == 1))))


def _run_attention(c, s):
    o, ws = s["out"], s["ws"]
    tao.tao_bound_check_linear(s["q"], s["k"], None, s["scores"], s["scores_claimed"], out=o[0], ws=ws, readback=False)
    tao.tao_bound_check_softmax(s["x"], s["p"], s["p_claimed"], out=o[1], ws=ws, readback=False)
    tao.tao_bound_check_linear(s["p"], s["v"], None, s["ctx"], s["ctx_claimed"], trans_w=True, out=o[2], ws=ws, readback=False)
    return o


def _prepare_norm(c, g):
    rows, cols = c["rows"], c["cols"]
    x = _randn(g, (rows, cols))
    gamma, beta = 1 + _randn(g, (cols,), 0.02), _randn(g, (cols,), 0.02)
    layer = c["norm"] == "layernorm"
    eps = 1e-5 if layer else 1e-6

    def execute(order):
        t = order(x)
        if layer:
            d = x - t.sum(dim=-1, keepdim=True) / cols
            r = torch.rsqrt((order(d) ** 2).sum(dim=-1, keepdim=True) / cols + eps)
            return d * r * gamma + beta
        return gamma * (x * torch.rsqrt((t * t).sum(dim=-1, keepdim=True) / cols + eps))

    y, claimed = execute(lambda t: t), execute(lambda t: t.flip(-1).contiguous())
    return dict(x=x, gamma=gamma, beta=beta, eps=eps, y=y, claimed=claimed, out=_profile_buffer(), ws=_scratch(tao.tao_check_workspace_bytes(x.numel())))


def _run_norm(c, s):
    kind = tao.NORM_LAYERNORM if c["norm"] == "layernorm" else tao.NORM_RMSNORM
    return [tao.tao_bound_check_norm(kind, s["x"], s["y"], s["claimed"], s["gamma"], s["beta"], eps=s["eps"], out=s["out"], ws=s["ws"], readback=False)]


def _prepare_act(c, g):
    n, act = c["n"], c["act"]
    x, x2 = _randn(g, (n,)), _randn(g, (n,))
    ws = _scratch(tao.tao_check_workspace_bytes(n))
    if act == "add":
        y = x + x2
        ops = [(tao.ACT_ADD, x, x2, y, y.clone())]                        # one rounding: every correct execution agrees
    elif act == "silu_mul":
        xd = x.double()
        y = x / (1 + torch.exp(-x))
        z = y * x2
        ops = [(tao.ACT_SILU, x, None, y, (xd / (1 + torch.exp(-xd))).float()), (tao.ACT_MUL, y, x2, z, z.clone())]
    else:
        xd = x.double()
        if act == "gelu":
            y = 0.5 * x * (1 + torch.erf(x * 0.5 ** 0.5))
            claimed = (0.5 * xd * (1 + torch.erf(xd * 0.5 ** 0.5))).float()
            ops = [(tao.ACT_GELU_ERF, x, None, y, claimed)]
        else:
            f = lambda t: 0.5 * t * (1 + torch.tanh((2 / math.pi) ** 0.5 * (t + 0.044715 * t * t * t)))
            ops = [(tao.ACT_GELU_TANH, x, None, f(x), f(xd).float())]
    return dict(ops=ops, out=[_profile_buffer() for _ in ops], ws=ws)


def _run_act(c, s):
    for (kind, x, x2, y, claimed), o in zip(s["ops"], s["out"]):
        tao.tao_bound_check_act(kind, x, y, claimed, x2=x2, out=o, ws=s["ws"], readback=False)
    return s["out"]


def _conv_dims(c):
    pad = c["filter"] // 2
    out = (c["size"] + 2 * pad - c["filter"]) // c["stride"] + 1
    return pad, out, c["filter"] ** 2 * c["C"]


def _prepare_conv(c, g):
    B, H, C, Cout, R = c["batch"], c["size"], c["C"], c["Cout"], c["filter"]
    pad, OH, K = _conv_dims(c)
    x = _randn(g, (B, H, H, C)).abs()                                     # after a ReLU
    w = _randn(g, (Cout, R, R, C), (2.0 / K) ** 0.5)
    # the verifier's execution and the claim: the sum over filter taps, in two orders
    xp = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad))
    taps = [(r, s) for r in range(R) for s in range(R)]
    span = (OH - 1) * c["stride"] + 1

    def execute(order):
        acc = torch.zeros((B * OH * OH, Cout), device="cuda")
        for r, t in order:
            acc += xp[:, r:r + span:c["stride"], t:t + span:c["stride"], :].reshape(-1, C) @ w[:, r, t, :].t().contiguous()
        return acc.view(B, OH, OH, Cout)

    y, claimed = execute(taps), execute(taps[::-1])
    scale, shift = 1 + _randn(g, (Cout,), 0.1), _randn(g, (Cout,), 0.1)
    z = y * scale + shift
    s = dict(x=x, w=w, y=y, claimed=claimed, scale=scale, shift=shift, z=z, z_claimed=z.clone(), pad=pad, z_tau=torch.empty_like(z),
             out=[_profile_buffer(), _profile_buffer()], check_ws=_scratch(tao.tao_check_workspace_bytes(y.numel())),
             fused=tao.tao_conv2d_split_supported(tuple(x.shape), tuple(w.shape), c["stride"], pad, 1))
    if s["fused"]:
        s["ws"] = _scratch(tao.lib().tao_conv2d_split_workspace_bytes(B, H, H, C, Cout, R, R, c["stride"], c["stride"], pad, pad, 1, 1, 1))
    else:
        s["tau"] = torch.empty_like(y)
    return s


def _run_conv(c, s):
    o = s["out"]
    if s["fused"]:
        tao.tao_bound_check_conv2d(s["x"], s["w"], None, s["y"], s["claimed"], c["stride"], s["pad"], out=o[0], ws=s["ws"], readback=False)
    else:                                                                 # shapes the one-pass entry point does not take
        tao.tao_bound_conv2d(s["x"], s["w"], None, c["stride"], s["pad"], out=s["tau"])
        tao.tao_check_and_profile(s["claimed"], s["y"], s["tau"], out=o[0], ws=s["check_ws"], readback=False)
    # the affine operator stores its bound, which is then checked
    tao.tao_bound_norm(tao.NORM_BN_AFFINE, s["y"], s["z"], s["scale"], s["shift"], out=s["z_tau"])
    tao.tao_check_and_profile(s["z_claimed"], s["z"], s["z_tau"], out=o[1], ws=s["check_ws"], readback=False)
    return [o[0], s["z_tau"], o[1]]


def _prepare_project(c, g):
    n = c["n"]
    ref = _randn(g, (n,))
    size = ctypes.sizeof(tao.ErrorProfile)
    ws = _scratch(tao.tao_profile_workspace_bytes(n))
    # committed thresholds: three times the envelope of four honest runs' profiles
    runs = torch.empty((4, size), dtype=torch.uint8, device="cuda")
    for r in range(4):
        tao.tao_profile_errors(ref * (1 + _randn(g, (n,), 1e-6)), ref, out=runs[r], ws=ws, readback=False)
    _, _, thr_abs, thr_rel = tao.tao_calibrate_thresholds(runs, 3.0)
    # a gradient step away from the honest output: part of the elements, a larger part at the top, leave the set
    delta = ref * _randn(g, (n,), 1e-6) * torch.exp(_randn(g, (n,)))
    tau = ref.abs() * 2e-6
    return dict(claimed=ref + delta, ref=ref, delta=delta, tau=tau, thr_abs=thr_abs, thr_rel=thr_rel, ws=ws,
                profile=torch.empty(size, dtype=torch.uint8, device="cuda"), project_ws=_scratch(tao.tao_project_workspace_bytes(n)),
                clipped=torch.empty_like(delta), capped=torch.empty_like(delta))


def _run_project(c, s):
    tao.tao_profile_errors(s["claimed"], s["ref"], thr_abs=s["thr_abs"], thr_rel=s["thr_rel"], out=s["profile"], ws=s["ws"], readback=False)
    tao.tao_project_clip(s["delta"], s["tau"], 1.0, out=s["clipped"])
    tao.tao_project_empirical(s["delta"], s["thr_abs"], 1.0, out=s["capped"], ws=s["project_ws"])
    return [s["profile"], s["clipped"], s["capped"]]


_PREPARE = dict(linear=_prepare_linear, attention=_prepare_attention, norm=_prepare_norm, act=_prepare_act, conv=_prepare_conv, project=_prepare_project)
_RUN = dict(linear=_run_linear, attention=_run_attention, norm=_run_norm, act=_run_act, conv=_run_conv, project=_run_project)


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return case, _PREPARE[case["kind"]](case, g)


def run(state):
    case, s = state
    return _RUN[case["kind"]](case, s)


# ------------------------------------------------------------------ what a pass cannot do without

_PROFILE = ctypes.sizeof(tao.Profile)


def work(case):
    """Bytes: operands, re-executed and claimed outputs read once, results (and bounds that are handed over) written once.
    Flops: the products' multiply-adds, and for the other operators a nominal dozen operations per element."""
    c, kind = case, case["kind"]
    if kind == "linear":
        M, K, N = c["M"], c["K"], c["N"]
        return dict(bytes=4 * (M * K + N * K + M * N * (3 if c["route"] == "stored" else 2)) + _PROFILE, flops=2 * M * K * N)
    if kind == "attention":
        B, R, S, D = c["heads"], c["group"] * c["seq"], c["seq"], c["dim"]
        scores, ctx = B * R * S, B * R * D
        # q, k, v; scores twice; softmax input, output and claim (its output is also the next product's operand); context twice
        return dict(bytes=4 * (ctx + 2 * B * S * D + 5 * scores + 2 * ctx) + 3 * _PROFILE, flops=4 * B * R * S * D + 12 * scores)
    if kind == "norm":
        n = c["rows"] * c["cols"]
        return dict(bytes=12 * n + 4 * c["cols"] + _PROFILE, flops=12 * n)
    if kind == "act":
        n = c["n"]
        per = dict(add=8, silu_mul=16, gelu=12, gelu_tanh=12)[c["act"]]
        return dict(bytes=per * n + _PROFILE, flops=12 * n)
    if kind == "conv":
        _, OH, K = _conv_dims(c)
        n = c["batch"] * OH * OH * c["Cout"]
        x = c["batch"] * c["size"] ** 2 * c["C"]
        # input, filters, output and claim; then the affine operator: its input, output, claim and the bound it hands over
        return dict(bytes=4 * (x + c["Cout"] * K + 2 * n + 3 * n) + 2 * _PROFILE, flops=2 * n * K + 12 * n)
    n = c["n"]
    # profile: two inputs; clip: two inputs, one output; capped projection: one input, one output
    return dict(bytes=4 * n * (2 + 3 + 2), flops=24 * n)


def tolerance(case):
    """Profiles are whole numbers and binary64 quotients of exact quantities, projections are bit-identical by contract: exact.
    A stored bound lies between the real-number value and 1e-6 above it, so two correct ones differ by no more than that
    (measured against the product in 64 bits: up to 7e-7 on the matrix cores, 1.2e-7 for the affine operator)."""
    if (case["kind"] == "linear" and case["route"] == "stored") or case["kind"] == "conv":
        return dict(rel=1e-6, max=1.1e-6)
    return "exact"
