"""The work that a serving or evaluation program has this library do, as cases that can be timed and checked.

A case is one linear layer of a transformer block: the packed weights are laid
out once (sdq.pack, offline), the program keeps the blob, its output buffers
and its workspace, and one pass quantizes a batch of activations per token and
multiplies it by the decomposed weights.  INT and MX layers go through
sdq.linear, dual layers through sdq.quantize_act_dual and sdq.gemm_dual.

The shapes are the LLaMA-7B and OPT-6.7B linear layers of the repository's
workloads (and shards and ragged sizes around them), from one token of decode
to thousands of tokens of prefill.
"""
import math

import torch

import paper_2406_13868_amd as sdq


def _case(name, family, M, N, K, n_o=1, m_o=8, fmt_o="e4m3", n_i=3, sfmt_i="", qv_i=0, y="f32", x="bf16"):
    c = dict(family=family, M=M, N=N, K=K, n_o=n_o, m_o=m_o, fmt_o=fmt_o, n_i=n_i, sfmt_i=sfmt_i, qv_i=qv_i, y=y, x=x)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one token of decode through an attention projection: the smallest call, launches and latency
        _case("int_m1_attn", "int", 1, 4096, 4096),
        # a few sequences decoded together through a gate projection, bf16 output for the activation that follows
        _case("int_m4_gate", "int", 4, 11008, 4096, y="bf16"),
        # a batch of 16 sequences decoded through an attention projection
        _case("int_m16_attn", "int", 16, 4096, 4096),
        # 64 sequences through the first FFN layer of an OPT-6.7B block, int8 outliers
        _case("int8o_m64_fc1", "int", 64, 16384, 4096, fmt_o="int8"),
        # a short prompt of odd length through a down projection, byte-sized inlier scales
        _case("int_m201_down", "int", 201, 4096, 11008, sfmt_i="e4m3", qv_i=32, y="bf16"),
        # a long prompt through an attention projection
        _case("int_m2048_attn", "int", 2048, 4096, 4096),
        # a batch of 16 sequences decoded through a gate projection, MX formats
        _case("mx_m16_gate", "mx", 16, 11008, 4096, n_i=2),
        # a prompt of odd length through a down projection, MX formats
        _case("mx_m301_down", "mx", 301, 4096, 11008, n_i=2, y="bf16"),
        # the prefill of 2048 tokens through a gate projection, MX formats (the default benchmark's layer)
        _case("mx_m2048_gate", "mx", 2048, 11008, 4096, n_i=2),
        # one token of decode, the paper's dual formats
        _case("dual_m1_attn", "dual", 1, 4096, 4096, fmt_o="int8", n_i=6),
        # a short prompt through an attention projection, two outliers in eight
        _case("dual_m256_attn", "dual", 256, 4096, 4096, n_o=2, fmt_o="int8", n_i=4, y="bf16"),
        # a batch of long prompts through a gate projection, the paper's dual formats: the largest call
        _case("dual_m4096_gate", "dual", 4096, 11008, 4096, fmt_o="int8", n_i=6),
    ]


_MOST_FLOPS = 2.0 * 4096 * 11008 * 4096


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["int", "int", "mx", "dual"])
    while True:
        M = _log(rng, 1, 4096)
        # whole layers and the shards of them that a tensor-parallel program holds; odd N is a padded vocabulary or head
        N = _log(rng, 512, 22016)
        K = 32 * _log(rng, 16, 512)
        if rng.random() < 0.5:
            N, K = N // 128 * 128, max(512, K // 128 * 128)
        if 2.0 * M * N * K <= _MOST_FLOPS and N * K <= 22016 * 4096:
            break
    y, x = rng.choice(["f32", "bf16"]), rng.choice(["bf16", "bf16", "f32"])
    if family == "dual":
        n_o, n_i = rng.choice([(1, 6), (2, 4), (1, 7)])
        return _case(None, "dual", M, N, K, n_o=n_o, fmt_o="int8", n_i=n_i, y=y, x=x)
    m_o, n_i = rng.choice([8, 8, 16]), rng.choice([2, 3])
    if family == "mx":
        return _case(None, "mx", M, N, K, m_o=m_o, n_i=n_i, y=y, x=x)
    sfmt_i = rng.choice(["", "", "e4m3", "ue6m2"])
    qv_i = rng.choice([0, 0, 32] + ([64] if K % 64 == 0 else []))
    return _case(None, "int", M, N, K, m_o=m_o, fmt_o=rng.choice(["e4m3", "int8"]), n_i=n_i, sfmt_i=sfmt_i, qv_i=qv_i,
                 y=y, x=x)


def _config(c):
    f = c["family"]
    return sdq.Config(f, c["n_o"], c["m_o"], c["fmt_o"], c["n_i"], 8, "int4" if f == "int" else "e2m1",
                      "e4m3" if f == "mx" else "int8", sfmt_i=c["sfmt_i"], y_dtype=c["y"], qv_i=c["qv_i"])


def _inputs(case, seed):
    """Weights [N, K] fp32 with a few heavy-tailed entries, activations [M, K] with a few loud channels."""
    dev = torch.device("cuda")
    M, N, K = case["M"], case["N"], case["K"]
    g = torch.Generator(device=dev).manual_seed(1000003 * int(seed) + 17)
    W = torch.randn((N, K), generator=g, device=dev) * 0.02
    n = max(1, int(0.002 * N * K))
    at = torch.randint(0, N * K, (n,), generator=g, device=dev)
    z = torch.randn((4, n), generator=g, device=dev)
    # Student's t with three degrees of freedom; entries hit twice would depend on the order of the writes
    heavy = torch.zeros(N * K, device=dev)
    heavy.scatter_reduce_(0, at, 0.2 * z[0] / ((z[1:] ** 2).sum(0) / 3).sqrt(), "amax", include_self=False)
    hit = torch.zeros(N * K, dtype=torch.bool, device=dev)
    hit[at] = True
    W = torch.where(hit.view(N, K), heavy.view(N, K), W)
    X = torch.randn((M, K), generator=g, device=dev)
    loud = torch.randperm(K, generator=g, device=dev)[: max(1, K // 1000)]
    X[:, loud] *= 30
    return W, X.to(torch.bfloat16 if case["x"] == "bf16" else torch.float32)


def prepare(case, seed):
    cfg, M, N, K = _config(case), case["M"], case["N"], case["K"]
    W, X = _inputs(case, seed)
    dev = X.device
    packed = torch.from_numpy(sdq.pack(W.cpu().numpy(), cfg)).to(dev)
    s = dict(cfg=cfg, N=N, K=K, X=X, packed=packed, Y=torch.empty((M, N), dtype=cfg.y_torch_dtype(), device=dev),
             Xq=torch.empty((M, K), dtype=torch.uint8, device=dev), s_a=torch.empty(M, device=dev))
    if cfg.family == "dual":
        s["Xi"] = torch.empty((M, K // 2), dtype=torch.uint8, device=dev)
        s["Ea"] = torch.empty((M, K // 32), dtype=torch.uint8, device=dev)
    else:
        nb = sdq.gemm_workspace_size(cfg, M, N, K)
        s["ws"] = torch.empty(nb, dtype=torch.uint8, device=dev) if nb else None
    return s


def run(s):
    if s["cfg"].family == "dual":
        q = sdq.quantize_act_dual(s["X"], s["cfg"], out=(s["Xq"], s["s_a"], s["Xi"], s["Ea"]))
        return (sdq.gemm_dual(*q, s["packed"], s["N"], s["K"], s["cfg"], out=s["Y"]), *q)
    return sdq.linear(s["X"], s["packed"], s["N"], s["K"], s["cfg"], out=s["Y"], xq=s["Xq"], scales=s["s_a"],
                      workspace=s["ws"])


def work(case):
    M, N, K = case["M"], case["N"], case["K"]
    acts = M * K * (2 if case["x"] == "bf16" else 4) + M * K + 4 * M
    if case["family"] == "dual":
        acts += M * K // 2 + M * K // 32
    y = M * N * (2 if case["y"] == "bf16" else 4)
    return {"bytes": sdq.logical_bytes(_config(case), N, K) + acts + y, "flops": 2.0 * M * N * K}


def tolerance(case):
    # Every product is exact; results differ by the order and rounding of fp32 sums (and, in the MX family, of the
    # matrix unit's own sums over a block), then by the output's type.  Against 64 bits fp32 outputs measure 3e-8 to
    # 8e-8 (INT, dual) and 1.6e-5 (MX), bf16 ones 1.7e-3; the limits are about four times that and room for long rows.
    if case["y"] == "bf16":
        return {"rel": 6e-3, "max": 1.6e-2}
    return {"rel": 6e-5, "max": 1e-3} if case["family"] == "mx" else {"rel": 4e-7, "max": 5e-6}


# ---------------------------------------------------------------- the same in 64 bits, from the formats' definitions
def _e4m3(v):
    """fp64 -> the nearest e4m3 value, ties to even, saturating at 448."""
    a = v.abs().clamp(max=448.0)
    e = torch.frexp(a.clamp(min=2.0 ** -6))[1].to(torch.float64) - 1
    step = torch.exp2(e - 3)
    return torch.copysign((torch.round(a / step) * step).clamp(max=448.0), v)


def _e2m1(v):
    a = v.abs().clamp(max=6.0)
    e = torch.frexp(a.clamp(min=1.0))[1].to(torch.float64) - 1
    step = torch.exp2(e - 1)
    return torch.copysign((torch.round(a / step) * step).clamp(max=6.0), v)


def _ue6m2(v):
    e = torch.frexp(v.clamp(min=2.0 ** -30))[1].to(torch.float64) - 1
    step = torch.exp2(e - 2)
    return torch.round(v / step) * step


def _floor_log2(a):
    return torch.frexp(a)[1].to(torch.float64) - 1


def _top(S, m, n, mask):
    """The n largest of every m along K where mask allows, ties to the lower k."""
    N, K = S.shape
    key = torch.where(mask, S, torch.full_like(S, -1.0)).view(N, K // m, m)
    at = torch.sort(key, dim=-1, descending=True, stable=True).indices[..., :n]
    return torch.zeros_like(key, dtype=torch.bool).scatter_(-1, at, True).view(N, K)


def _blocks(absW, mask, qv):
    N, K = absW.shape
    return torch.where(mask, absW, torch.zeros_like(absW)).view(N, K // qv, qv).amax(-1)


def _weights(W, case):
    """(outliers, inliers), dequantized, fp64 [N, K]."""
    N, K = W.shape
    absW, f = W.abs(), case["family"]
    everything = torch.ones_like(W, dtype=torch.bool)
    mo = _top(absW, case["m_o"], case["n_o"], everything) if case["n_o"] else ~everything
    mi = _top(absW, 8, case["n_i"], ~mo)
    zero = torch.zeros((), dtype=torch.float64, device=W.device)
    if f == "mx":
        a = _blocks(absW, mo, 32).double()
        s = torch.exp2((_floor_log2(a) - 8).clamp(-127, 127)).repeat_interleave(32, 1)
        out = torch.where(mo, _e4m3(W.double() / s) * s, zero)
    else:
        qmax = 127.0 if case["fmt_o"] == "int8" else 448.0
        s = torch.where(mo, absW, torch.zeros_like(W)).amax(1, keepdim=True) / torch.tensor(qmax, device=W.device)
        v = (W / torch.where(s == 0, torch.ones_like(s), s)).double()
        q = torch.round(v).clamp(-127, 127) if case["fmt_o"] == "int8" else _e4m3(v)
        out = torch.where(mo & (s != 0), q * s.double(), zero)
    qv = case["qv_i"] or (16 if f == "int" else 32)
    a = _blocks(absW, mi, qv)
    if f == "int":
        v = a / torch.tensor(7.0, device=W.device)
        if case["sfmt_i"] == "e4m3":
            top = v.double().amax(1, keepdim=True)
            E = _floor_log2(torch.where(top > 0, top, torch.ones_like(top))) - 8
            E = torch.where(top > 448 * torch.exp2(E), E + 1, E)
            s = _e4m3(v.double() / torch.exp2(E)) * torch.exp2(E)
        else:
            s = _ue6m2(v.double()) if case["sfmt_i"] else v.half().double()
        s = s.repeat_interleave(qv, 1)
        q = torch.round((W / torch.where(s == 0, torch.ones_like(s), s).float()).double()).clamp(-7, 7)
        return out, torch.where(mi & (s != 0), q * s, zero)
    E = torch.where(a > 0, (_floor_log2(a.double()) - 2).clamp(-127, 127), -127.0)
    s = torch.exp2(E).repeat_interleave(qv, 1)
    return out, torch.where(mi, _e2m1(W.double() / s) * s, zero)


def exact(case, seed):
    W, X = _inputs(case, seed)
    wo, wi = _weights(W, case)
    X = X.float()
    a = X.abs().amax(1, keepdim=True)
    qmax = torch.tensor(448.0 if case["family"] == "mx" else 127.0, device=X.device)
    s_a, inv = a / qmax, torch.where(a > 0, qmax / a, torch.zeros_like(a))
    v = (X * inv).double()
    q = _e4m3(v) if case["family"] == "mx" else torch.round(v).clamp(-127, 127)
    if case["family"] != "dual":
        Y = s_a.double() * (q @ (wo + wi).T)
        return Y, None, s_a[:, 0].double()
    M, K = X.shape
    b = X.abs().view(M, K // 32, 32).amax(-1).double()
    E = torch.where(b > 0, (_floor_log2(b) - 2).clamp(-127, 127), -127.0)
    s = torch.exp2(E).repeat_interleave(32, 1)
    Y = s_a.double() * (q @ wo.T) + (_e2m1(X.double() / s) * s) @ wi.T
    return Y, None, s_a[:, 0].double(), None, None
