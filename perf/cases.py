"""Performance cases of the stream-batched rectified-flow step.

Each case is one call that a program makes through the package's entry points: whole
stream steps and velocity calls of the workload networks, shallow networks of the wider
shapes (their blocks are all alike, so two to four stand for twenty-eight), and the
layers that can be called alone (self-attention, the timestep conditioning, the latent
update). `listed()` names the ones that are followed, `draw()` gives more of the same
ranges, `prepare()` builds what a program holds before the call (the loaded model, the
device buffers), `run()` is the call, `exact()` its result in 64-bit arithmetic written
out in plain torch.

Weights are those of the synthetic workloads with the timestep path at 1 / fan_in
variance (every linear map N(0, 0.02), the fixed sin-cos position table), so the adaLN
gates have the size of a trained network's and every block counts in the result.
"""
import math
import struct

import numpy as np
import torch

from paper_2511_22009_amd import Cond, Model, Precision

GUIDANCE = 7.5
# the schedule of the PeRFlow time windows: count, length, first and last beta
WINDOWS, TRAIN_STEPS, BETA0, BETA1 = 4, 1000, 0.00085, 0.012


def _net(name, kind, H, W, D, L, heads, mlp, B, prec="bf16", C=4, p=2, tdim=128, ctx_len=0, ctx_dim=0, guided=False,
         fill=False, windows=False, graph=False):
    return {"name": name, "kind": kind, "C": C, "H": H, "W": W, "p": p, "D": D, "L": L, "heads": heads, "mlp": mlp,
            "tdim": tdim, "ctx_len": ctx_len, "ctx_dim": ctx_dim, "B": B, "prec": prec, "guided": guided, "fill": fill,
            "windows": windows, "graph": graph}


def listed():
    return [
        # the smallest network of the workloads, a full queue of four latents: all
        # launches, no work (interactive previews, tests of a pipeline)
        _net("tiny_step", "step", 16, 16, 128, 2, 4, 512, 4),
        # 512^2, one latent: a queue that starts to fill, or sampling one image alone
        _net("one_512", "velocity", 64, 64, 768, 12, 12, 3072, 1),
        # 512^2, four slots in flight, replayed from a captured graph: the framework's
        # steady state
        _net("stream_512", "step", 64, 64, 768, 12, 12, 3072, 4, graph=True),
        # 512^2, text-conditioned, eight slots doubled by guidance
        _net("guided_512", "step", 64, 64, 768, 12, 12, 3072, 8, ctx_len=77, ctx_dim=1024, guided=True),
        # 512^2, the width-1152 network (head dim 72), four slots, four of its blocks
        _net("wide_512", "velocity", 64, 64, 1152, 4, 16, 4608, 4),
        # 1024^2, the width-1152 network, four slots, two of its blocks
        _net("wide_1024", "velocity", 128, 128, 1152, 2, 16, 4608, 4),
        # a 640 x 368 picture (920 tokens, no multiple of any tile) with a queue of three
        # that still fills, updated through the time windows
        _net("ragged_fill", "step", 46, 80, 768, 4, 12, 3072, 3, fill=True, windows=True),
        # the 32-bit mode: 512^2, four slots, two blocks
        _net("fp32_512", "velocity", 64, 64, 768, 2, 12, 3072, 4, prec="fp32"),
        # the 32-bit mode on a small ragged network (140 tokens, head dim 48)
        _net("fp32_ragged", "step", 20, 28, 192, 2, 4, 768, 3, prec="fp32"),
        # one self-attention layer of the 1024^2 network, two rows
        _net("attention_1024", "attention", 128, 128, 1152, 1, 16, 1152, 2),
        # the timestep conditioning of eight slots: embedding, MLP, every adaLN projection
        _net("modulation_512", "modulation", 64, 64, 768, 12, 12, 3072, 8),
        # the update and shift of a deep queue of 1024^2 latents, for a given velocity
        _net("update_1024", "update", 128, 128, 128, 1, 4, 512, 32),
    ]


# drawn networks stay below the work of the largest listed case (guided_512), the 32-bit
# ones below that of fp32_512
_MOST = {"bf16": 4.0e12, "fp32": 1.4e11}


def draw(rng):
    while True:
        kind = rng.choice(["step", "step", "velocity", "velocity", "velocity", "attention", "modulation", "update"])
        prec = "fp32" if rng.random() < 0.25 else "bf16"
        dh = rng.choice([32, 48, 64, 64, 64, 72, 72, 96, 128])
        heads = max(1, min(int(round(math.exp(rng.uniform(math.log(2), math.log(16))))), 1536 // dh))
        D = heads * dh
        # tokens from 24 to 4096, odd sides among them
        n = math.exp(rng.uniform(math.log(24), math.log(4096)))
        aspect = math.exp(rng.uniform(-0.6, 0.6))
        gh = max(3, int(round(math.sqrt(n * aspect))))
        gw = max(3, int(round(n / gh)))
        B = int(round(math.exp(rng.uniform(0.0, math.log(16)))))
        L = rng.randint(1, 4)
        cross = kind in ("step", "velocity") and rng.random() < 0.35
        guided = cross and rng.random() < 0.7
        steps = kind == "step"
        c = _net("", kind, 2 * gh, 2 * gw, D, L, heads, 4 * D, B, prec=prec, ctx_len=rng.randint(16, 128) if cross else 0,
                 ctx_dim=rng.choice([64, 256, 768, 1024]) if cross else 0, guided=guided,
                 fill=steps and rng.random() < 0.25, windows=steps and rng.random() < 0.25, graph=steps and rng.random() < 0.35)
        if kind == "attention":
            c["L"], c["mlp"] = 1, D
        elif kind == "modulation":
            c["L"] = rng.randint(2, 12)
            c["H"] = c["W"] = 16
        elif kind == "update":
            c["D"], c["L"], c["heads"], c["mlp"], c["prec"] = 64, 1, 2, 64, "bf16"
            c["B"] = rng.randint(1, 32)
            c["fill"], c["windows"] = rng.random() < 0.3, rng.random() < 0.3
        if work(c)["flops"] <= _MOST[c["prec"]]:
            del c["name"]
            return c


# ------------------------------------------------------------------------- sizes

def _tokens(c):
    return (c["H"] // c["p"]) * (c["W"] // c["p"])


def _rows(c):
    return 2 * c["B"] if c["guided"] else c["B"]


def _specs(c):
    """The tensors of a weight blob in its order, with the standard deviation each is
    drawn with (None: the position table)."""
    D, P, F, N, x = c["D"], c["p"] * c["p"] * c["C"], c["mlp"], _tokens(c), c["ctx_dim"]
    s = 0.02
    out = [("W_pe", (D, P), s), ("b_pe", (D,), s), ("pos", (N, D), None), ("W_t1", (D, c["tdim"]), c["tdim"] ** -0.5),
           ("b_t1", (D,), s), ("W_t2", (D, D), D ** -0.5), ("b_t2", (D,), s)]
    for i in range(c["L"]):
        b = [("W_mod", (6 * D, D), D ** -0.5), ("b_mod", (6 * D,), s), ("W_qkv", (3 * D, D), s), ("b_qkv", (3 * D,), s),
             ("W_o", (D, D), s), ("b_o", (D,), s)]
        if x:
            b += [("W_qx", (D, D), s), ("b_qx", (D,), s), ("W_kvx", (2 * D, x), s), ("b_kvx", (2 * D,), s),
                  ("W_ox", (D, D), s), ("b_ox", (D,), s)]
        b += [("W_fc1", (F, D), s), ("b_fc1", (F,), s), ("W_fc2", (D, F), s), ("b_fc2", (D,), s)]
        out += [("%d.%s" % (i, n), sh, sd) for n, sh, sd in b]
    return out + [("W_fmod", (2 * D, D), D ** -0.5), ("b_fmod", (2 * D,), s), ("W_f", (P, D), s), ("b_f", (P,), s)]


def work(c):
    """Weights, latents and contexts read once, outputs written once; products of the
    network without padding (a context's keys and values once, the null context's too)."""
    es = 2 if c["prec"] == "bf16" else 4
    N, D, F, L, R, B = _tokens(c), c["D"], c["mlp"], c["L"], _rows(c), c["B"]
    E, P = c["C"] * c["H"] * c["W"], c["p"] * c["p"] * c["C"]
    if c["kind"] == "attention":
        return {"bytes": 4.0 * B * N * D * es, "flops": 4.0 * B * N * N * D}
    if c["kind"] == "update":
        return {"bytes": 4.0 * E * (2 * B + 1 + B + 1), "flops": 2.0 * B * E}
    tpath = c["tdim"] * D + D * D + (6 * L + 2) * D * D
    if c["kind"] == "modulation":
        return {"bytes": 4.0 * (c["tdim"] * D + D * D) + es * (6.0 * L + 2) * D * D + 4.0 * B * (6 * L + 2) * D,
                "flops": 2.0 * B * tpath}
    per_block = 2.0 * N * D * (4 * D + 2 * F) + 4.0 * N * N * D
    flops = 2.0 * B * tpath + R * (L * per_block + 4.0 * N * P * D)
    weights = 4.0 * (c["tdim"] * D + D * D + 2 * P * D + N * D) + es * (6.0 * L + 2) * D * D + es * L * (4.0 * D * D + 2 * D * F)
    if c["ctx_len"]:
        entries = B + (1 if c["guided"] else 0)
        flops += R * L * (4.0 * N * D * D + 4.0 * N * c["ctx_len"] * D) + entries * L * 4.0 * c["ctx_len"] * c["ctx_dim"] * D
        weights += es * L * (2.0 * D * D + 2 * D * c["ctx_dim"]) + 4.0 * entries * c["ctx_len"] * c["ctx_dim"]
    return {"bytes": weights + 4.0 * E * (2 * B + (2 if c["kind"] == "step" else 0)), "flops": flops}


def tolerance(c):
    """About four times what this path was measured off `exact()` by: 16-bit mode 1.8e-3
    in a velocity, 2.9e-3 in an attention layer, 5e-4 (1.2e-3 guided) in an updated queue,
    where the latents outweigh the step; 32-bit mode 2.6e-7. Guidance multiplies the
    difference of two rows' errors by its weight."""
    if c["kind"] == "update":
        return {"rel": 1e-6, "max": 1e-5}
    if c["kind"] == "modulation":
        return {"rel": 4e-6, "max": 1e-4}  # sums in 32 bits, whatever the weights' type
    if c["prec"] == "fp32":
        return {"rel": 1e-5 if c["guided"] else 2e-6, "max": 1e-4}
    if c["kind"] == "attention":
        return {"rel": 1.2e-2, "max": 0.2}
    if c["kind"] == "step":
        return {"rel": 5e-3 if c["guided"] else 2e-3, "max": 0.1}
    return {"rel": 1.6e-2 if c["guided"] else 8e-3, "max": 0.2}


# ------------------------------------------------------------------------ inputs

def _pos_table(c):
    """The fixed 2-D sin-cos position table (half the width for the patch row, half for
    the column)."""
    gh, gw, q = c["H"] // c["p"], c["W"] // c["p"], c["D"] // 4
    omega = 1.0 / 10000.0 ** (torch.arange(q, dtype=torch.float64, device="cuda") / q)
    r = torch.arange(gh, dtype=torch.float64, device="cuda").repeat_interleave(gw)[:, None] * omega
    k = torch.arange(gw, dtype=torch.float64, device="cuda").repeat(gh)[:, None] * omega
    return torch.cat([r.sin(), r.cos(), k.sin(), k.cos()], 1).float()


def _weights(c, seed):
    """One flat fp32 tensor on the GPU in blob order, and a view of every tensor in it."""
    specs = _specs(c)
    total = sum(int(np.prod(sh)) for _, sh, _ in specs)
    g = torch.Generator(device="cuda").manual_seed(1000003 * seed + 17)
    flat = torch.randn(total, generator=g, device="cuda")
    views, off = {}, 0
    for name, sh, sd in specs:
        n = int(np.prod(sh))
        v = views[name] = flat[off:off + n].view(sh)
        if sd is None:
            v.copy_(_pos_table(c))
        else:
            v.mul_(sd)
        off += n
    return flat, views


def _load(c, seed, max_rows):
    flat, _ = _weights(c, seed)
    head = struct.pack("<4sI12IQ", b"SFW1", 1, c["C"], c["H"], c["W"], c["p"], c["D"], c["L"], c["heads"], c["mlp"], c["tdim"],
                       c["ctx_len"], c["ctx_dim"], 1 if c["ctx_len"] else 0, seed)
    blob = np.empty(64 + 4 * flat.numel(), np.uint8)
    blob[:64] = np.frombuffer(head, np.uint8)
    torch.from_numpy(blob[64:].view(np.float32)).copy_(flat)
    return Model(blob, Precision.FP32 if c["prec"] == "fp32" else Precision.BF16, max_rows)


def _inputs(c, seed):
    """Latents, noise, times and contexts. Slot k of a queue of B sits at t = 1 - k / B,
    moved by up to a third of a step: every slot at a time of its own."""
    g = torch.Generator(device="cuda").manual_seed(1000003 * seed + 29)
    rng = np.random.default_rng([seed, 31])
    B, latent = c["B"], (c["C"], c["H"], c["W"])
    s = {}
    s["x"] = torch.randn((B + 1,) + latent, generator=g, device="cuda")
    s["z"] = torch.randn(latent, generator=g, device="cuda")
    t = 1.0 - (np.arange(B) + rng.uniform(0.0, 1.0 / 3.0, B)) / B
    if c["windows"]:  # a noise prediction is updated inside its window, not at its end
        t = np.clip(t, 0.02, 1.0)
    s["t"] = t.astype(np.float32)
    s["dt"] = (np.append(t[1:], 0.0) - t).astype(np.float32)
    if c["ctx_len"]:
        s["ctx"] = torch.randn((B, c["ctx_len"], c["ctx_dim"]), generator=g, device="cuda")
        s["null"] = torch.randn((c["ctx_len"], c["ctx_dim"]), generator=g, device="cuda") if c["guided"] else None
    if c["kind"] == "update":
        s["v"] = torch.randn((B,) + latent, generator=g, device="cuda")
    if c["kind"] == "attention":
        dt = torch.float32 if c["prec"] == "fp32" else torch.bfloat16
        sh = (B, c["heads"], _tokens(c), c["D"] // c["heads"])
        s["q"], s["k"], s["v"] = (torch.randn(sh, generator=g, device="cuda").to(dt) for _ in range(3))
    return s


def prepare(c, seed):
    s = _inputs(c, seed)
    rows = 1 if c["kind"] in ("attention", "update") else _rows(c)
    m = s["model"] = _load(c, seed, rows)
    s["case"] = c
    if c["windows"]:
        m.set_scheduler(WINDOWS, TRAIN_STEPS, BETA0, BETA1)
    if c["ctx_len"]:
        s["cond"] = Cond(s["ctx"], s["null"], GUIDANCE)
    if c["kind"] in ("step", "update"):
        s["done"] = None if c["fill"] else torch.empty_like(s["z"])
    if c["graph"]:
        m.graph_enable(True)
        s["stream"] = torch.cuda.Stream()
    if c["kind"] == "attention":
        # v as the library's projections leave it: transposed, keys past the last one
        # zero, in 16-bit mode with bits 2 and 3 of the key index swapped
        n, col = _tokens(c), torch.arange(_tokens(c), device="cuda")
        if m.info["vt_key_perm"]:
            col = (col & ~12) | ((col & 4) << 1) | ((col & 8) >> 1)
        v = s["v"]
        vt = torch.zeros(v.shape[:2] + (v.shape[3], m.info["vt_ld"]), dtype=v.dtype, device="cuda")
        vt[..., col] = v.transpose(2, 3)
        s["vt"] = vt
    torch.cuda.synchronize()
    return s


def run(s):
    c, m, B = s["case"], s["model"], s["case"]["B"]
    if c["kind"] == "velocity":
        return m.velocity(s["x"][:B], s["t"], s.get("cond"))
    if c["kind"] == "step":
        m.stream_step(s["x"], s["t"], s["dt"], B, s["z"], s["done"], s.get("cond"), s.get("stream"))
    elif c["kind"] == "update":
        m.scheduler_shift(s["x"], s["v"], s["t"], s["dt"], B, s["z"], s["done"])
    elif c["kind"] == "attention":
        return m.attention(s["q"], s["k"], s["vt"])
    else:
        return m.modulation(s["t"])
    return {"x": s["x"]} if c["fill"] else {"x": s["x"], "done": s["done"]}


# ----------------------------------------------------------------- 64-bit results

def _silu(z):
    return z / (1.0 + torch.exp(-z))


def _lin(x, W, b):
    return x @ W.double().t() + b.double()


def _ln(z):
    d = z - z.mean(-1, keepdim=True)
    return d / torch.sqrt((d * d).mean(-1, keepdim=True) + 1e-6)


def _softmax_attention(q, k, v):
    """[heads, n, dh] each, in blocks of queries."""
    out = torch.empty_like(q)
    kt = k.transpose(1, 2).contiguous()
    step = max(1, (1 << 27) // (q.shape[0] * k.shape[1]))
    for i in range(0, q.shape[1], step):
        p = torch.softmax(torch.bmm(q[:, i:i + step].contiguous(), kt) / math.sqrt(q.shape[2]), -1)
        out[:, i:i + step] = torch.bmm(p, v)
    return out


def _heads(z, h):
    return z.view(z.shape[0], h, -1).transpose(0, 1).contiguous()


def _attend(q, k, v, h):
    o = _softmax_attention(_heads(q, h), _heads(k, h), _heads(v, h))
    return o.transpose(0, 1).reshape(q.shape)


def _conditioning(c, w, t):
    """SiLU(c) of each time: phases rounded to 32 bits as the network's input defines
    them, the rest in 64."""
    half = c["tdim"] // 2
    f = np.exp(-math.log(10000.0) * np.arange(half, dtype=np.float64) / half).astype(np.float32)
    phi = ((np.float32(1000.0) * t)[:, None] * f[None]).astype(np.float32).astype(np.float64)
    e = torch.from_numpy(np.concatenate([np.cos(phi), np.sin(phi)], 1)).cuda()
    return _silu(_lin(_silu(_lin(e, w["W_t1"], w["b_t1"])), w["W_t2"], w["b_t2"]))


def _forward(c, w, x, s, ctx):
    """The network on one latent; s = SiLU(c) [1, D]."""
    C, H, W, p, D, h = c["C"], c["H"], c["W"], c["p"], c["D"], c["heads"]
    tok = x.double().view(C, H // p, p, W // p, p).permute(1, 3, 2, 4, 0).reshape(-1, p * p * C)
    z = _lin(tok, w["W_pe"], w["b_pe"]) + w["pos"].double()
    for i in range(c["L"]):
        b = {n: w["%d.%s" % (i, n)] for n in ("W_mod", "b_mod", "W_qkv", "b_qkv", "W_o", "b_o", "W_fc1", "b_fc1", "W_fc2", "b_fc2")}
        m = _lin(s, b["W_mod"], b["b_mod"]).view(6, D)
        a = _lin(_ln(z) * (1.0 + m[1]) + m[0], b["W_qkv"], b["b_qkv"])
        z = z + m[2] * _lin(_attend(a[:, :D], a[:, D:2 * D], a[:, 2 * D:], h), b["W_o"], b["b_o"])
        if ctx is not None:
            x_ = {n: w["%d.%s" % (i, n)] for n in ("W_qx", "b_qx", "W_kvx", "b_kvx", "W_ox", "b_ox")}
            kv = _lin(ctx.double(), x_["W_kvx"], x_["b_kvx"])
            z = z + _lin(_attend(_lin(_ln(z), x_["W_qx"], x_["b_qx"]), kv[:, :D], kv[:, D:], h), x_["W_ox"], x_["b_ox"])
        u = _lin(_ln(z) * (1.0 + m[4]) + m[3], b["W_fc1"], b["b_fc1"])
        u = 0.5 * u * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (u + 0.044715 * u ** 3)))
        z = z + m[5] * _lin(u, b["W_fc2"], b["b_fc2"])
    m = _lin(s, w["W_fmod"], w["b_fmod"]).view(2, D)
    out = _lin(_ln(z) * (1.0 + m[1]) + m[0], w["W_f"], w["b_f"])
    return out.view(H // p, W // p, p, p, C).permute(4, 0, 2, 1, 3).reshape(C, H, W)


def _update(c, s, v):
    """The queue after the update and shift, for the network's output v."""
    B, x = c["B"], s["x"].double()
    new = []
    for k in range(B):
        t, dt = float(s["t"][k]), float(s["dt"][k])
        if c["windows"]:
            beta = np.linspace(math.sqrt(np.float32(BETA0)), math.sqrt(np.float32(BETA1)), TRAIN_STEPS) ** 2
            abar = np.cumprod(1.0 - beta)
            kw = max(1, sum(t > j / WINDOWS + 1e-6 for j in range(WINDOWS)))
            ts, te = kw / WINDOWS, (kw - 1) / WINDOWS
            at = lambda u: abar[int(np.rint(u * (TRAIN_STEPS - 1)))]  # noqa: E731
            g = math.sqrt(at(ts) / at(te))
            den = (t - ts) / g + (te - t)
            pred = (te - ts) / g / den * x[k] + (-math.sqrt(1.0 - g * g) / g * (te - t) / den) * v[k]
            new.append(x[k] + dt * (pred - x[k]) / (te - t))
        else:
            new.append(x[k] + dt * v[k])
    z = s["z"].double()
    if c["fill"]:
        return {"x": torch.stack([z] + new)}
    return {"x": torch.stack([z] + new[:-1] + [x[B]]), "done": new[-1]}


def exact(c, seed):
    s = _inputs(c, seed)
    if c["kind"] == "update":
        return _update(c, s, s["v"].double())
    if c["kind"] == "attention":
        o = [_softmax_attention(s["q"][r].double(), s["k"][r].double(), s["v"][r].double()) for r in range(c["B"])]
        return torch.stack([r.transpose(0, 1).reshape(_tokens(c), c["D"]) for r in o])
    _, w = _weights(c, seed)
    sc = _conditioning(c, w, s["t"])
    if c["kind"] == "modulation":
        parts = [_lin(sc, w["%d.W_mod" % i], w["%d.b_mod" % i]) for i in range(c["L"])]
        return torch.cat(parts + [_lin(sc, w["W_fmod"], w["b_fmod"])], 1)
    v = []
    for k in range(c["B"]):
        one = _forward(c, w, s["x"][k], sc[k:k + 1], s["ctx"][k] if c["ctx_len"] else None)
        if c["guided"]:
            null = _forward(c, w, s["x"][k], sc[k:k + 1], s["null"])
            one = null + GUIDANCE * (one - null)
        v.append(one)
    v = torch.stack(v)
    return _update(c, s, v) if c["kind"] == "step" else v
