"""Performance cases of the scheduled denoiser step.

A user of this library does two things with it: builds a schedule from a model's weights once,
and runs denoising steps, one after another, with that schedule or without one.  The cases are
those calls over the sizes they meet: single evaluations of one to three blocks of every
architecture (a block is the unit the library schedules), whole scheduled trajectories with
frozen units and cached updates, a replayed trajectory graph, and schedule builds, from
latency-bound single samples to full batches.

Weights and inputs are drawn on the GPU from the seed.  ``exact`` evaluates the same network in
float64 with plain torch.
"""
import math

import numpy as np
import torch

import paper_2609_29505_amd as P
import synth

GATED = ("llada", "sdxl", "sdxl_unet")
CROSS = ("sdxl", "sdxl_unet")


def _case(**kw):
    """A case with every field set.  ``kind`` "step": one unscheduled evaluation per pass,
    "trajectory": T scheduled steps from z_1, "graph": the same as one replayed HIP graph,
    "schedule": one schedule build.  ``rows``: first token the sampler updates (LLaDA's prompt
    rows stay fixed)."""
    c = dict(kind="step", arch="dit", dtype="bf16", B=1, N=256, d=1024, dh=64, F=4096, L=1, T=50, budget=100,
             granularity="block", ctx_len=0, ctx_dim=0, grid=0, rows=0)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest calls: the fp32 network, a whole 10-step trajectory at half the layer-steps
        # (kernels of a few microseconds; launches count)
        _case(name="tiny_trajectory", kind="trajectory", arch="tiny", dtype="f32", N=256, d=256, F=1024, L=4, T=10,
              budget=50),
        # a short prompt of a language-model denoiser: 200 ragged tokens, bound by its weights
        _case(name="llada_short", arch="llada", N=200, d=4096, dh=128, F=12288, L=2, T=64, rows=100),
        # the same blocks at the 1024 tokens the 8B-shaped workload runs
        _case(name="llada_block", arch="llada", N=1024, d=4096, dh=128, F=12288, L=2, T=64, rows=512),
        # its scheduled trajectory at half the layer-steps: active units, frozen runs, cache stores
        _case(name="llada_trajectory", kind="trajectory", arch="llada", N=1024, d=4096, dh=128, F=12288, L=4, T=6,
              rows=512, budget=50),
        # class-conditional image generation: a full batch of 32 samples
        _case(name="dit_block", arch="dit", B=32, N=256, d=1152, dh=72, F=4608, L=2),
        # one image with classifier-free guidance (two samples), every branch a unit of its own,
        # the whole trajectory replayed as one graph
        _case(name="dit_pair_graph", kind="graph", arch="dit", B=2, N=256, d=1152, dh=72, F=4608, L=4, T=6, budget=50,
              granularity="branch"),
        # U-ViT's in-, mid- and out-block with the long skip: 258 tokens (ragged against any tile)
        _case(name="uvit_stack", arch="uvit", B=32, N=258, d=1024, F=4096, L=3),
        # SDXL's 32 x 32 stage: self-attention, cross-attention to 77 text tokens, gated MLP
        _case(name="sdxl_block", arch="sdxl", B=8, N=1024, d=1280, F=5120, ctx_len=77, ctx_dim=2048),
        # the UNet stage unit in front of it: two 3 x 3 convolutions and GroupNorms as well
        _case(name="sdxl_unet_block", arch="sdxl_unet", B=8, N=1024, d=1280, F=5120, ctx_len=77, ctx_dim=2048,
              grid=32),
        # the same unit for one image on an odd 25 x 25 grid
        _case(name="sdxl_unet_single", arch="sdxl_unet", B=1, N=625, d=1280, F=5120, ctx_len=77, ctx_dim=2048,
              grid=25),
        # schedule builds: a small fp32 stack (24 matrices of 256 x 256 to 1024 x 256), and one
        # full-width bf16 block (4 of 1152 x 1152, 2 of 4608 x 1152)
        _case(name="schedule_small", kind="schedule", arch="tiny", dtype="f32", d=256, F=1024, L=4, T=10, budget=50),
        _case(name="schedule_block", kind="schedule", arch="dit", d=1152, dh=72, F=4608, L=1, T=50, budget=50),
    ]


def draw(rng):
    """One more case of the same ranges; sizes are spread over their logarithm."""
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def traj(c, most):
        """Turns a step case into a trajectory of up to ``most`` active block evaluations."""
        if rng.random() < 0.4:
            c["kind"] = rng.choice(["trajectory", "trajectory", "graph"])
            c["granularity"] = rng.choice(["block", "branch"])
            c["T"] = rng.randint(3, max(3, most // c["L"]))
            c["budget"] = rng.choice([50, 70])
        return c

    arch = rng.choice(["tiny", "llada", "llada", "dit", "dit", "uvit", "sdxl", "sdxl_unet", "schedule"])
    if arch == "tiny":
        d = 128 * rng.randint(1, 4)
        return _case(kind="trajectory", arch="tiny", dtype="f32", B=rng.randint(1, 3), N=logint(16, 400), d=d,
                     F=128 * logint(d // 128, d // 32), L=rng.randint(2, 5), T=rng.randint(4, 10),
                     budget=rng.choice([50, 70]))
    if arch == "llada":
        d = 128 * rng.randint(8, 32)
        n = logint(32, 1024)
        return traj(_case(arch="llada", N=n, d=d, dh=128, F=64 * int(round(d * rng.uniform(2.5, 3.0) / 64)),
                          L=rng.randint(1, 2), T=64, rows=rng.randint(0, n // 2)), 6)
    if arch == "dit":
        d, dh = rng.choice([(1152, 72), (1024, 64), (768, 64)])
        return traj(_case(arch="dit", B=logint(1, 32), N=logint(64, 256), d=d, dh=dh, F=4 * d, L=rng.randint(1, 3)), 12)
    if arch == "uvit":
        return traj(_case(arch="uvit", B=logint(1, 32), N=2 + logint(64, 256), d=rng.choice([512, 768, 1024]), F=4096,
                          L=3), 12)
    if arch == "schedule":
        d = logint(96, 1152)
        return _case(kind="schedule", arch=rng.choice(["dit", "uvit"]), dtype=rng.choice(["bf16", "f32"]), d=d,
                     F=logint(2 * d, 4 * d), L=3 if d <= 400 else 1, T=50, budget=rng.choice([50, 70]))
    d = rng.choice([640, 1280])
    g = rng.randint(8, 32)
    n = g * g if arch == "sdxl_unet" else logint(64, 1024)
    return traj(_case(arch=arch, B=logint(1, 8), N=n, d=d, F=4 * d, ctx_len=77, ctx_dim=rng.choice([768, 2048]),
                      grid=g if arch == "sdxl_unet" else 0), 3)


# ------------------------------------------------------------------ inputs

def _config(c):
    return synth.Config(c["arch"], c["arch"], c["dtype"], c["B"], c["N"], c["d"], c["d"] // c["dh"], c["dh"], c["F"],
                        c["L"], c["T"], ctx_len=c["ctx_len"], ctx_dim=c["ctx_dim"], prompt_rows=c["rows"],
                        grid=c["grid"])


def _rng(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _weights(c, seed):
    """Per block, the device tensors of its parameters (names of sgd_unit_weights): Gaussian
    matrices of gain one, gains around one, small biases."""
    g = _rng(seed)
    d, F, arch = c["d"], c["F"], c["arch"]
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    fo = 2 * F if arch in GATED else F

    def mat(m, n):
        return torch.randn(m, n, generator=g, device="cuda").mul_(n ** -0.5).to(dt)

    def vec(n, center=0.0, scale=0.02):
        return torch.randn(n, generator=g, device="cuda").mul_(scale).add_(center)

    blocks = []
    for l in range(c["L"]):
        w = dict(w_qkv=mat(3 * d, d), w_o=mat(d, d), w1=mat(fo, d), w2=mat(d, F))
        if arch == "dit":
            w.update(w_ada=mat(6 * d, d), b_ada=vec(6 * d), b_qkv=vec(3 * d))
        else:
            w.update(norm1_w=vec(d, 1.0, 0.1), norm2_w=vec(d, 1.0, 0.1))
        if arch in ("uvit",) + CROSS:
            w.update(norm1_b=vec(d), norm2_b=vec(d))
        if arch not in ("tiny", "llada"):
            w.update(b_o=vec(d), b1=vec(fo), b2=vec(d))
        if arch == "uvit" and l > c["L"] // 2:
            w.update(w_skip=mat(d, 2 * d), b_skip=vec(d))
        if arch in CROSS:
            w.update(normx_w=vec(d, 1.0, 0.1), normx_b=vec(d), w_xq=mat(d, d), w_xkv=mat(2 * d, c["ctx_dim"]),
                     w_xo=mat(d, d), b_xo=vec(d))
        if arch == "sdxl_unet":
            w.update(gn1_w=vec(d, 1.0, 0.1), gn1_b=vec(d), w_conv1=mat(d, 9 * d), b_conv1=vec(d), w_temb=mat(d, d),
                     b_temb=vec(d), gn2_w=vec(d, 1.0, 0.1), gn2_b=vec(d), w_conv2=mat(d, 9 * d), b_conv2=vec(d))
        blocks.append(w)
    return blocks


def _inputs(c, seed):
    g = _rng(seed + 7919)
    x = dict(z=torch.randn(c["B"], c["N"], c["d"], generator=g, device="cuda"))
    if c["arch"] in ("dit", "sdxl_unet"):
        x["class_emb"] = torch.randn(c["B"], c["d"], generator=g, device="cuda")
    if c["arch"] in CROSS:
        ctx = torch.randn(1, c["ctx_len"], c["ctx_dim"], generator=g, device="cuda").bfloat16()
        x["ctx"] = ctx.expand(c["B"], -1, -1).contiguous()
    return x


def _lifetimes(c, units):
    """Nested lifetimes in 1..T with mean near budget % of T, in a fixed mixed order."""
    T = c["T"]
    spread = [(i * 7 + 3) % units for i in range(units)]
    lo = max(1.0, 2.0 * c["budget"] / 100 * T - T)
    hi = min(float(T), 2.0 * c["budget"] / 100 * T)
    return [min(T, max(1, int(round(lo + (hi - lo) * (r + 0.5) / units)))) for r in spread]


def _host(t):
    """Storage array of a tensor as DeviceModel takes it (bf16 as uint16 bit patterns)."""
    return t.view(torch.int16).cpu().numpy().view(np.uint16) if t.dtype == torch.bfloat16 else t.cpu().numpy()


def _scored(c, seed):
    """Per unit, the scored matrices of a block with decaying column norms (spectra between flat
    and concentrated, as in trained weights)."""
    g = _rng(seed + 104729)
    d = c["d"]
    units = []
    for w in _weights(c, seed):
        mats = [("q", w["w_qkv"][:d]), ("k", w["w_qkv"][d:2 * d]), ("v", w["w_qkv"][2 * d:]), ("o", w["w_o"]),
                ("w1", w["w1"]), ("w2", w["w2"])]
        unit = []
        for role, m in mats:
            decay = 0.3 + 1.2 * torch.rand(1, generator=g, device="cuda")
            n = m.shape[1]
            col = torch.arange(1, n + 1, device="cuda").float().pow(-decay)
            col = col * (n / col.square().sum()).sqrt()
            unit.append((role, (m.float() * col).to(m.dtype).contiguous()))
        units.append(unit)
    return units


def prepare(case, seed):
    c = dict(_case(), **case)
    if c["kind"] == "schedule":
        return dict(case=c, units=_scored(c, seed))
    x = _inputs(c, seed)
    weights = [{k: _host(v) for k, v in w.items()} for w in _weights(c, seed)]
    model = P.DeviceModel(_config(c), weights, {k: _host(v) for k, v in x.items() if k != "z"},
                          granularity=c["granularity"])
    s = dict(case=c, model=model, z1=x["z"], z=x["z"].clone())
    if c["kind"] != "step":
        s["sched"] = P.schedule_from_lifetimes(_lifetimes(c, model.n_units), c["T"])
        s["cache"] = P.Cache(model)
    if c["kind"] == "graph":
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        s["graph"] = model.capture(s["z"], s["sched"], s["cache"], side)
        torch.cuda.synchronize()
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "schedule":
        sch = P.schedule_build(s["units"], [c["dh"]] * c["L"], c["T"], budget_pct=c["budget"])
        names = ("e_top", "e_tail", "frob", "scr", "g", "sigma1_sq")
        out = {n: sch.mat_stats[:, i] for i, n in enumerate(names)}
        return dict(out, raw=sch.unit_raw, lifetimes=sch.lifetimes)
    m, z = s["model"], s["z"]
    if c["kind"] == "step":
        # the state moves on by alpha z - beta eps at every pass, as a sampler moves it
        m.step(z, 1, None, None, alpha=1.0, beta=1.0 / c["T"])
        return z
    z.copy_(s["z1"])
    if c["kind"] == "graph":
        s["graph"].launch(torch.cuda.current_stream())
        return z
    s["cache"].reset()
    for step in range(1, c["T"] + 1):
        m.step(z, step, s["sched"], s["cache"])
    return z


# ------------------------------------------------------------------ work and tolerance

def _branches(c):
    """Per branch of a block: (flops of one evaluation, weight bytes)."""
    M, N, d, F, es = c["B"] * c["N"], c["N"], c["d"], c["F"], 2 if c["dtype"] == "bf16" else 4
    fo = 2 * F if c["arch"] in GATED else F
    out = []
    if c["arch"] == "sdxl_unet":
        out.append((2 * 2.0 * M * 9 * d * d + 2.0 * c["B"] * d * d, (18 * d * d + d * d) * es))
    ada = 2.0 * c["B"] * 6 * d * d if c["arch"] == "dit" else 0.0
    out.append((2.0 * M * 4 * d * d + 4.0 * M * N * d + ada / 2, (4 + (3 if ada else 0)) * d * d * es))
    if c["arch"] in CROSS:
        out.append((2.0 * M * 2 * d * d + 4.0 * M * c["ctx_len"] * d +
                    2.0 * c["B"] * c["ctx_len"] * 2 * d * c["ctx_dim"], (2 * d * d + 2 * d * c["ctx_dim"]) * es))
    out.append((2.0 * M * (fo + F) * d + ada / 2, (fo + F + (3 * d if ada else 0)) * d * es))
    return out


def work(case):
    c = dict(_case(), **case)
    d, F = c["d"], c["F"]
    if c["kind"] == "schedule":
        es = 2 if c["dtype"] == "bf16" else 4
        fo = 2 * F if c["arch"] in GATED else F
        # the Gram matrix of the short side and its reduction to tridiagonal form
        shapes = [(d, d)] * 4 + [(fo, d), (d, F)]
        flops = sum(float(max(m, n)) * min(m, n) ** 2 + 4.0 / 3.0 * min(m, n) ** 3 for m, n in shapes)
        return {"bytes": float(c["L"] * es * sum(m * n for m, n in shapes)), "flops": c["L"] * flops}
    M = c["B"] * c["N"]
    br = _branches(c)
    skips = (c["L"] // 2) * 2 * d * d if c["arch"] == "uvit" else 0
    skip_f, skip_b = 2.0 * M * skips, 2.0 * skips
    if c["kind"] == "step":
        return {"bytes": c["L"] * sum(b for _, b in br) + skip_b + 8.0 * M * d,
                "flops": c["L"] * sum(f for f, _ in br) + skip_f}
    units = c["L"] * (len(br) if c["granularity"] == "branch" else 1)
    per = br if c["granularity"] == "branch" else [(sum(f for f, _ in br), sum(b for _, b in br))]
    byts, flops = 8.0 * M * d + c["T"] * skip_b, c["T"] * skip_f
    for u, life in enumerate(_lifetimes(c, units)):
        f, b = per[u % len(per)]
        flops += life * f
        # weights at every active step, the cached update written once and read at frozen steps
        byts += life * b + (4.0 * M * d * (1 + c["T"] - life) if life < c["T"] else 0.0)
    return {"bytes": byts, "flops": flops}


# about four times the relative error of one evaluation's output against float64 (bf16 weights and
# activations): 0.0021 LLaDA, 0.0023-0.0032 SDXL, 0.0039 U-ViT, 0.0049 DiT
_BF16_REL = {"llada": 0.01, "sdxl": 0.015, "sdxl_unet": 0.015, "uvit": 0.016, "dit": 0.02}


def tolerance(case):
    c = dict(_case(), **case)
    if c["kind"] == "schedule":
        # float64 throughout: 1e-15 to 6e-15 measured; another backward-stable eigenvalue method
        # is off by some multiple of the short side (up to 1152) times 1e-16
        return {"rel": 1e-12}
    if c["dtype"] == "f32":
        return {"rel": 2e-6}  # 2.9e-7 measured over ten steps
    # every evaluation enters the state times beta = 1/T
    steps = 1 if c["kind"] == "step" else c["T"]
    return {"rel": _BF16_REL[c["arch"]] * steps / c["T"]}


# ------------------------------------------------------------------ float64 reference

def _emb(t, dim):
    half = dim // 2
    f = torch.exp(-math.log(10000.0) * torch.arange(half, dtype=torch.float64, device="cuda") / half)
    return torch.cat([torch.cos(t * f), torch.sin(t * f)])


def _ln(x, eps, w=None, b=None):
    x = x - x.mean(-1, keepdim=True)
    y = x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps)
    return y if w is None else y * w + b


def _heads(x, H):
    return x.view(x.shape[0], x.shape[1], H, -1).transpose(1, 2)


def _attend(q, k, v):
    """softmax(q k^T / sqrt(dh)) v, sample by sample; [B, H, N, dh] -> [B, N, d]."""
    out = []
    for i in range(q.shape[0]):
        p = torch.softmax(q[i] @ k[i].transpose(1, 2).contiguous() / math.sqrt(q.shape[-1]), -1)
        out.append((p @ v[i].contiguous()).transpose(0, 1).reshape(q.shape[2], -1))
    return torch.stack(out)


def _rope(x):
    half = x.shape[-1] // 2
    inv = 10000.0 ** (-torch.arange(half, dtype=torch.float64, device="cuda") / half)
    a = torch.arange(x.shape[2], dtype=torch.float64, device="cuda")[:, None] * inv
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * a.cos() - x2 * a.sin(), x2 * a.cos() + x1 * a.sin()], -1)


def _gelu_tanh(x):
    return 0.5 * x * (1 + torch.tanh(math.sqrt(2 / math.pi) * (x + 0.044715 * x ** 3)))


def _gelu(x):
    return 0.5 * x * (1 + torch.erf(x / math.sqrt(2)))


def _silu(x):
    return x * torch.sigmoid(x)


def _group_norm(x, groups, w, b):
    B, N, C = x.shape
    y = x.view(B, N, groups, C // groups)
    y = y - y.mean((1, 3), keepdim=True)
    y = y * torch.rsqrt(y.square().mean((1, 3), keepdim=True) + 1e-5)
    return y.reshape(B, N, C) * w + b


def _conv(x, w, side):
    B, N, C = x.shape
    pad = torch.zeros(B, side + 2, side + 2, C, dtype=x.dtype, device=x.device)
    pad[:, 1:-1, 1:-1] = x.view(B, side, side, C)
    out = 0
    for k in range(9):
        ky, kx = divmod(k, 3)
        tap = pad[:, ky:ky + side, kx:kx + side].reshape(B * N, C)
        out = out + tap @ w[:, k * C:(k + 1) * C].t().contiguous()
    return out.view(B, N, -1)


def _branch(c, name, w, h, x, t):
    """The update of one residual branch on the stream h, in float64."""
    d, H, F, arch = c["d"], c["d"] // c["dh"], c["F"], c["arch"]

    def lin(v, m, bias=None):
        y = v @ w[m].t().contiguous()
        return y if bias is None or bias not in w else y + w[bias]

    def norm(which, mod=None):
        if arch in ("tiny", "llada"):
            return h * torch.rsqrt(h.square().mean(-1, keepdim=True) + 1e-5) * w[which + "_w"]
        if arch == "dit":
            return _ln(h, 1e-6) * (1 + mod[1][:, None]) + mod[0][:, None]
        return _ln(h, 1e-5, w[which + "_w"], w[which + "_b"])

    if name == "resnet":
        temb = lin(_silu(_emb(t, d)[None] + x["class_emb"]), "w_temb", "b_temb")
        u = _silu(_group_norm(h, 32, w["gn1_w"], w["gn1_b"]))
        u = _conv(u, w["w_conv1"], c["grid"]) + w["b_conv1"] + temb[:, None]
        return _conv(_silu(_group_norm(u, 32, w["gn2_w"], w["gn2_b"])), w["w_conv2"], c["grid"]) + w["b_conv2"]
    mod = lin(_silu(_emb(t, d)[None] + x["class_emb"]), "w_ada", "b_ada").split(d, -1) if arch == "dit" else None
    if name == "attn":
        q, k, v = (_heads(p, H) for p in lin(norm("norm1", mod), "w_qkv", "b_qkv").split(d, -1))
        if arch == "llada":
            q, k = _rope(q), _rope(k)
        a = lin(_attend(q, k, v), "w_o", "b_o")
        return a if mod is None else mod[2][:, None] * a
    if name == "xattn":
        k, v = (_heads(p, H) for p in (x["ctx"] @ w["w_xkv"].t().contiguous()).split(d, -1))
        return lin(_attend(_heads(lin(norm("normx"), "w_xq"), H), k, v), "w_xo", "b_xo")
    y = lin(norm("norm2", mod[3:] if mod else None), "w1", "b1")
    if arch == "llada":
        y = _silu(y[..., :F]) * y[..., F:]
    elif arch in CROSS:
        y = _gelu(y[..., :F]) * y[..., F:]
    else:
        y = _gelu_tanh(y) if arch == "dit" else _gelu(y)
    y = lin(y, "w2", "b2")
    return y if mod is None else mod[5][:, None] * y


def _exact_schedule(c, seed):
    cols = []
    for unit in _scored(c, seed):
        for _, m in unit:
            m = m.double().cpu()
            m = m if m.shape[0] <= m.shape[1] else m.t()
            gram = (m @ m.t()).numpy()
            lam = np.sort(np.maximum(np.linalg.eigvalsh(gram), 0.0))[::-1]
            n = len(lam)
            k = min(n, max(1, n // 10))
            frob = float(np.trace(gram))
            top, tail = float(lam[:k].sum()), float(lam[k:].sum())
            a, b = top + 1e-6 * frob, tail + 1e-6 * frob
            cols.append([top, tail, frob, math.log(a / b), math.sqrt(frob * a / (a + b)), float(lam[0])])
    st = np.array(cols)
    names = ("e_top", "e_tail", "frob", "scr", "g", "sigma1_sq")
    return dict({n: st[:, i].copy() for i, n in enumerate(names)}, raw=None, lifetimes=None)


def exact(case, seed):
    c = dict(_case(), **case)
    if c["kind"] == "schedule":
        return _exact_schedule(c, seed)
    x = {k: v.double() for k, v in _inputs(c, seed).items()}
    blocks = [{k: v.double() for k, v in w.items()} for w in _weights(c, seed)]
    names = (["resnet"] if c["arch"] == "sdxl_unet" else []) + ["attn"] + \
        (["xattn"] if c["arch"] in CROSS else []) + ["mlp"]
    nb = len(names) if c["granularity"] == "branch" else 1
    L, T, uvit = c["L"], c["T"], c["arch"] == "uvit"
    steps = 1 if c["kind"] == "step" else T
    life = [T] * (L * nb) if c["kind"] == "step" else _lifetimes(c, L * nb)
    r0 = c["rows"] if c["arch"] == "llada" else 2 if uvit else 0
    z, cache = x["z"], {}
    for s in range(1, steps + 1):
        t = 1000.0 * (T - s + 1) / T
        h = z.clone()
        if uvit:
            h[:, 0] = _emb(t, c["d"])
        saved = {}
        for l, w in enumerate(blocks):
            if uvit and l > L // 2:
                h = torch.cat([h, saved[L - 1 - l]], -1) @ w["w_skip"].t().contiguous() + w["b_skip"]
            for part in (names if nb > 1 else [names]):
                u = l * nb + (names.index(part) if nb > 1 else 0)
                if s <= life[u]:
                    before = h
                    for name in ([part] if nb > 1 else part):
                        h = h + _branch(c, name, w, h, x, t)
                    cache[u] = h - before
                else:
                    h = h + cache[u]
            if uvit and l < L // 2:
                saved[l] = h
        z = z.clone()
        z[:, r0:] -= h[:, r0:] / T
    return z
