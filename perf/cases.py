"""Timed workloads of the gated delta-rule forward, through its public entry points.

Every case is one call of ``forward``, ``frame_forward``, ``frame_forward_norm``,
``frame_forward_bidir`` or ``frame_forward_fused`` the way a streaming video
model makes it: device tensors in, library-cached workspace, outputs and the
carried states allocated by the call.  Sizes are those of 1280x704 video (a
latent frame is 44 x 80 = 3520 tokens, a streaming call three frames), of the
smaller 22 x 40 latent frame, and of the classifier-free-guidance batch; the
values follow the gates and feature maps of the model (unit or ReLU features,
Mamba-style decays, sigmoid write gates).
"""
import math

import torch

import paper_2605_30409_amd as gdn

# op: token | frame | fused; norm / bidir: the frame-wise variants (fused is
# always normalized); mu: mean of the decay gate's pre-activation (2 = heads
# that forget fast); state: whether the call continues a stream (states in).
_BASE = dict(op="token", dtype="bf16", B=1, T=0, F=0, N=0, H=16, Dk=128, Dv=128, norm=False, bidir=False,
             mu=0.0, state=True, lat_w=80, t0=0)


def _case(**kw):
    c = dict(_BASE)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a short fp32 sequence of two heads, all latency
        _case(name="token-tiny-f32", dtype="f32", T=256, H=2, Dk=64, Dv=64, state=False),
        # one 1280x704 latent frame, token-wise (the headline workload)
        _case(name="token-frame", T=3520),
        # the streaming call: three frames with the state carried in and out
        _case(name="token-stream3", T=10560),
        # the guidance batch: four branches, twenty narrow heads that forget fast
        _case(name="token-batch-d64", B=4, T=10560, H=20, Dk=64, Dv=64, mu=2.0),
        # twelve frames in one call, all heads of a wide model
        _case(name="token-long", T=42240, H=32),
        # a tensor-parallel shard of the streaming call: two heads, long sequence
        _case(name="token-shard-h2", T=10560, H=2),
        # fp32 with a length that is no multiple of the chunk
        _case(name="token-ragged-f32", dtype="f32", T=3557),
        # one small (22 x 40) latent frame, frame-wise, plain readout
        _case(name="frame-small", op="frame", F=1, N=880, lat_w=40),
        # the streaming call frame-wise, both directions, normalized readout
        _case(name="frame-bidir-norm", op="frame", F=3, N=3520, norm=True, bidir=True),
        # the whole block operator on the streaming call
        _case(name="fused", op="fused", F=3, N=3520, norm=True, t0=6),
        # the same for the guidance batch with narrow heads, both directions
        _case(name="fused-batch-d64", op="fused", B=4, F=3, N=3520, H=20, Dk=64, Dv=64, norm=True, bidir=True,
              mu=2.0),
        # the block operator in the fp32 precision mode
        _case(name="fused-f32", op="fused", dtype="f32", F=3, N=3520, norm=True),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    """One more case of the same ranges: any length from one token to twelve
    frames, 1 to 32 heads, batches up to four, every head size and option."""
    op = rng.choice(["token", "token", "frame", "fused"])
    f32 = rng.random() < 0.25
    Dk, Dv = rng.choice([(128, 128), (128, 128), (128, 128), (64, 64), (64, 64), (128, 64), (64, 128)])
    B, H = rng.choice([1, 1, 1, 2, 4]), _log_int(rng, 1, 32)
    # token rows x channels of the whole call, kept below the largest listed ones
    room = (10560 * 16 * 128 if f32 else 42240 * 32 * 128) // (B * H * max(Dk, Dv))
    c = _case(op=op, dtype="f32" if f32 else "bf16", B=B, H=H, Dk=Dk, Dv=Dv, mu=rng.choice([0.0, 2.0]),
              state=rng.random() < 0.75)
    if op == "token":
        c["T"] = _log_int(rng, 1, min(room, 10560 if f32 else 42240))
        return c
    c["N"] = _log_int(rng, 1, min(room, 3520))
    c["F"] = rng.randint(1, max(1, min(12, room // c["N"])))
    c["norm"] = True if op == "fused" else rng.random() < 0.5
    c["bidir"] = rng.random() < 0.5
    c["lat_w"] = rng.choice([80, 40, 1 + rng.randrange(96)])
    c["t0"] = rng.choice([0, c["F"], 60])
    return c


def _tokens(c):
    return c["T"] if c["op"] == "token" else c["F"] * c["N"]


def _rope(Dk):
    """Frequencies and axes of the 3D rotation: a quarter of the channel pairs
    turn with time, the rest with the latent row and column."""
    P = Dk // 2
    nt = P // 4
    ny = (P - nt) // 2
    freq, axis = [], []
    for a, n in ((0, nt), (1, ny), (2, P - nt - ny)):
        freq += [10000.0 ** (-j / n) for j in range(n)]
        axis += [a] * n
    return freq, axis


def prepare(case, seed):
    c = case
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    B, T, H, Dk, Dv = c["B"], _tokens(c), c["H"], c["Dk"], c["Dv"]
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32

    def randn(*shape):
        return torch.randn(shape, generator=gen, device=dev)

    def rand(*shape):
        return torch.rand(shape, generator=gen, device=dev)

    def keys():
        x = randn(B, T, H, Dk)
        if c["op"] == "fused":                       # raw projections of varying scale
            return (x * (0.2 + 4.8 * rand(B, T, H, 1))).to(dt)
        if c["norm"]:                                # non-negative features
            x = x.clamp_min(0.0)
        return (x / x.norm(dim=-1, keepdim=True).clamp_min(1e-6)).to(dt)

    s = dict(case=dict(c))
    s["q"], s["k"] = keys(), keys()
    s["v"] = randn(B, T, H, Dv).to(dt)
    rows = T if c["op"] == "token" else c["F"]
    s["alpha"] = torch.exp(-torch.nn.functional.softplus(randn(B, rows, H) + c["mu"]))
    s["beta"] = torch.sigmoid(randn(B, T, H))
    s["state"] = 0.02 * randn(B, H, Dk, Dv) if c["state"] else None
    s["z"] = (0.02 * randn(B, H, Dk)).abs() if c["state"] and c["norm"] else None
    if c["op"] == "fused":
        s["gate"] = randn(B, T, H, Dv).to(dt)
        s["w_o"] = (randn(H, Dv, Dv) / math.sqrt(Dv)).to(dt)
        s["gain_q"], s["gain_k"] = 0.5 + rand(H, Dk), 0.5 + rand(H, Dk)
        freq, axis = _rope(Dk)
        s["freq"] = torch.tensor(freq, dtype=torch.float32, device=dev)
        s["axis"] = torch.tensor(axis, dtype=torch.int32, device=dev)
    return s


def run(s):
    c = s["case"]
    if c["op"] == "token":
        return gdn.forward(s["q"], s["k"], s["v"], s["alpha"], s["beta"], s["state"])
    if c["op"] == "fused":
        return gdn.frame_forward_fused(s["q"], s["k"], s["v"], s["gate"], s["w_o"], s["alpha"], s["beta"],
                                       s["gain_q"], s["gain_k"], s["freq"], s["axis"], s["state"], s["z"],
                                       frame_tokens=c["N"], lat_w=c["lat_w"], t0=c["t0"], bidirectional=c["bidir"])
    args = (s["q"], s["k"], s["v"], s["alpha"], s["beta"], s["state"])
    if c["bidir"]:
        return gdn.frame_forward_bidir(*args, s["z"], frame_tokens=c["N"], normalized=c["norm"])
    if c["norm"]:
        return gdn.frame_forward_norm(*args, s["z"], frame_tokens=c["N"])
    return gdn.frame_forward(*args, frame_tokens=c["N"])


def work(case):
    """Inputs once in, outputs once out; the recurrence's own products (a Gram
    matrix counted once for its symmetry)."""
    c = case
    esz = 2 if c["dtype"] == "bf16" else 4
    BH, Dk, Dv = c["B"] * c["H"], c["Dk"], c["Dv"]
    n = BH * _tokens(c)
    state = 4 * BH * (Dk * Dv + (Dk if c["norm"] else 0))
    by = n * (2 * Dk + 2 * Dv) * esz + 4 * n + 4 * (n if c["op"] == "token" else BH * c["F"])
    by += state * (2 if c["state"] else 1)
    if c["op"] == "token":
        return {"bytes": by, "flops": n * 6 * Dk * Dv}
    fl = n * (Dk * Dk + 4 * Dk * Dv)
    fl += BH * c["F"] * 2 * Dk * Dk * Dv * (2 if c["bidir"] else 1)
    if c["op"] == "fused":
        by += n * Dv * esz + c["H"] * Dv * Dv * esz + 8 * c["H"] * Dk
        fl += n * (Dk * Dk + 2 * Dv * Dv)
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # about four times the largest distance from the fp64 results: 4.2e-7 seen
    # in fp32 (the fused operator's state), 3.4e-3 in bf16 (token-wise outputs)
    if case["dtype"] == "f32":
        return {"rel": 1.7e-6}
    return {"rel": 1.4e-2}


def _exact_token(s):
    """The recurrence, one token at a time."""
    q, k, v = (s[n].double() for n in ("q", "k", "v"))
    alpha, beta = s["alpha"].double(), s["beta"].double()
    B, T, H, Dk = q.shape
    Dv = v.shape[-1]
    S = torch.zeros(B, H, Dk, Dv, dtype=torch.float64, device=q.device) if s["state"] is None else s["state"].double()
    out = torch.empty(B, T, H, Dv, dtype=torch.float64, device=q.device)
    for t in range(T):
        kt = k[:, t].unsqueeze(-1)
        S = S * alpha[:, t, :, None, None]
        u = beta[:, t].unsqueeze(-1) * (v[:, t] - (S * kt).sum(2))
        S = torch.addcmul(S, kt, u.unsqueeze(2))
        torch.sum(S * q[:, t].unsqueeze(-1), 2, out=out[:, t])
    return out, S


def _features(s, x, gain):
    """RMSNorm with gain and ReLU, and its rotation by the token's coordinates."""
    c = s["case"]
    F, N = c["F"], c["N"]
    x = x.double()
    x = (gain.double() * x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-6)).clamp_min(0.0)
    n = torch.arange(F * N, device=x.device)
    pos = torch.stack([c["t0"] + n // N, n % N // c["lat_w"], n % N % c["lat_w"]]).double()
    ang = s["freq"].double() * pos[s["axis"].long()].t()               # [T, Dk / 2]
    cs, sn = torch.cos(ang)[None, :, None], torch.sin(ang)[None, :, None]
    a, b = x[..., 0::2], x[..., 1::2]
    return x, torch.stack([a * cs - b * sn, a * sn + b * cs], -1).flatten(-2)


def _exact_frame(s):
    c = s["case"]
    B, H, F, N, Dk, Dv = (c[n] for n in ("B", "H", "F", "N", "Dk", "Dv"))
    ks = 1.0 / math.sqrt(Dk * N)
    if c["op"] == "fused":
        qt, qh = _features(s, s["q"], s["gain_q"])
        kt, kh = _features(s, s["k"], s["gain_k"])
    else:
        qt = qh = s["q"].double()
        kt = kh = s["k"].double()

    def frames(x):                                   # [B, T, H, D] -> [F, B, H, N, D]
        return x.reshape(B, F, N, H, -1).permute(1, 0, 3, 2, 4).contiguous()

    qt, qh, kt, kh, v = (frames(x) for x in (qt, qh, ks * kt, ks * kh, s["v"].double()))
    be = frames(s["beta"].double().unsqueeze(-1))
    al = s["alpha"].double().permute(1, 0, 2)[..., None, None]
    A = torch.stack([kh[f].mT.contiguous() @ (be[f] * v[f]) for f in range(F)])
    G = torch.stack([kh[f].mT.contiguous() @ (be[f] * kh[f]) for f in range(F)])
    Gz = torch.stack([kt[f].mT.contiguous() @ (be[f] * kt[f]) for f in range(F)])
    Az = torch.stack([kt[f].mT.contiguous() @ be[f] for f in range(F)])

    def step(f, S, P, R):
        return al[f] * (S - P[f] @ S) + R[f]

    S = torch.zeros_like(A[0]) if s["state"] is None else s["state"].double()
    z = torch.zeros_like(Az[0]) if s["z"] is None else s["z"].double().unsqueeze(-1)
    back = [(torch.zeros_like(S), torch.zeros_like(z)) for _ in range(F)]
    if c["bidir"]:
        for f in range(F - 1, 0, -1):
            back[f - 1] = (step(f, back[f][0], G, A), step(f, back[f][1], Gz, Az))
    outs = []
    for f in range(F):
        S, z = step(f, S, G, A), step(f, z, Gz, Az)
        o = qh[f] @ (S + back[f][0])
        if c["norm"]:
            o = o / (qt[f] @ (z + back[f][1]) + 1e-6)
        outs.append(o)
    out = torch.stack(outs).permute(1, 0, 3, 2, 4).reshape(B, F * N, H, Dv)
    if c["op"] == "fused":
        y = torch.nn.functional.silu(s["gate"].double()) * out
        w = s["w_o"].double().mT.contiguous()        # [H, in, out]
        out = (y.permute(0, 2, 1, 3).contiguous() @ w).permute(0, 2, 1, 3).contiguous()
    return (out, S, z.squeeze(-1)) if c["norm"] else (out, S)


def exact(case, seed):
    s = prepare(case, seed)
    return _exact_token(s) if case["op"] == "token" else _exact_frame(s)
