"""Per-kernel parity on the GPU: each kernel's output against the oracle applied to the
SAME inputs the kernel saw (read back from the library's workspace), so an error is
pinned to one kernel instead of the whole network."""
import numpy as np
import pytest

import oracle
import workloads as W
from conftest import oracle_model
from helpers import bf16_round, rel_l2

pytestmark = pytest.mark.gpu

from gpu_util import dev, host, model, torch  # noqa: E402
from paper_2511_22009_amd import Buffer  # noqa: E402

# tolerance of a kernel fed exactly its own inputs: fp32 arithmetic, or a bf16 output
ISO = {"fp32": 1e-5, "bf16": 1e-2}
TOL = {"fp32": 1e-4, "bf16": 2e-2}


def _run_block0(name, prec):
    cfg = W.get_config(name)
    t, _ = W.slot_times(cfg)
    x = W.latents(cfg, cfg.K)
    m = model(name, prec)
    R, N, D, H, dh = cfg.K, cfg.N, cfg.D, cfg.heads, cfg.dh
    h1 = host(m.residual(dev(x), t, 1))
    ldv = m.info["vt_ld"]
    assert ldv % 64 == 0 and ldv >= N
    # column of each key: the head-dim-64 bf16 layout swaps bits 2 and 3 of the key index
    tok = np.arange(N)
    col = (tok & ~12) | ((tok & 4) << 1) | ((tok & 8) >> 1) if m.info["vt_key_perm"] else tok
    assert m.info["vt_key_perm"] == (prec == "bf16")
    bufs = dict(
        q=host(m.debug_read(Buffer.Q, (R, H, N, dh))).transpose(0, 2, 1, 3).reshape(R, N, D),
        k=host(m.debug_read(Buffer.K, (R, H, N, dh))).transpose(0, 2, 1, 3).reshape(R, N, D),
        v=host(m.debug_read(Buffer.VT, (R, H, dh, ldv)))[..., col].transpose(0, 3, 1, 2).reshape(R, N, D),
        attn=host(m.debug_read(Buffer.ATTN, (R, N, D))),
        ln2=host(m.debug_read(Buffer.ACT, (R, N, D))),
        mlp=host(m.debug_read(Buffer.MLP, (R, N, cfg.mlp))),
        h_out=h1,
    )
    om = oracle_model(name)
    traces = []
    for k in range(R):
        tr = {}
        oracle.residual_one(om, x[k], t[k], None, 1, trace=tr)
        traces.append(tr)
    return cfg, om, bufs, traces


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("name", ["tiny_tsens", "ragged", "dh72", "dh64"])
def test_block0_intermediates(name, prec):
    cfg, om, g, tr = _run_block0(name, prec)
    b = om.blocks[0]
    report = {}
    for k in range(cfg.K):
        # end-to-end intermediates vs the oracle's own chain
        for key in ("q", "k", "v", "attn", "ln2", "mlp", "h_out"):
            report.setdefault(key, []).append(rel_l2(g[key][k], tr[k][key]))
        # each kernel on its own inputs
        a_iso = oracle.attention(g["q"][k].astype(np.float64), g["k"][k].astype(np.float64),
                                 g["v"][k].astype(np.float64), cfg.heads)
        report.setdefault("attn_iso", []).append(rel_l2(g["attn"][k], a_iso))
        f_iso = oracle.gelu_tanh(g["ln2"][k].astype(np.float64) @ b["W_fc1"].T.astype(np.float64) + b["b_fc1"])
        report.setdefault("fc1_iso", []).append(rel_l2(g["mlp"][k], f_iso))
    worst = {k: max(v) for k, v in report.items()}
    print(name, prec, {k: f"{v:.2e}" for k, v in worst.items()})
    assert worst["attn_iso"] <= ISO[prec], worst
    assert worst["fc1_iso"] <= ISO[prec], worst
    for key in ("q", "k", "v", "attn", "ln2", "mlp", "h_out"):
        assert worst[key] <= TOL[prec], worst


@pytest.mark.parametrize("D,heads", [(192, 4), (336, 6)], ids=["dh48", "dh56"])
@pytest.mark.parametrize("gh,gw", [(1, 1), (1, 3), (1, 5), (3, 5), (3, 7), (5, 6), (7, 9), (5, 13), (9, 22), (21, 25)])
def test_transposed_values_of_any_token_count(gh, gw, D, heads):
    """The transposed values that the QKV projection leaves, where token counts are no
    multiples of 4 or 16: groups of four tokens start at any row of a tile, reach from one
    group of 16 rows into the next, and are cut by tiles and network rows. Every row of a
    batch holds the bits it has alone, the columns of keys past the last stay zero, and a
    row agrees with the oracle."""
    from paper_2511_22009_amd import Model, Precision
    B = 7
    cfg = W.Config("vt", C=4, H=2 * gh, W=2 * gw, p=2, D=D, L=1, heads=heads, mlp=64, K=1, schedule="uniform1")
    blob = W.make_blob(cfg, init="tsens")
    m = Model(blob, Precision.BF16, B)
    x = W.latents(cfg, B, seed=61)
    t = np.random.default_rng(62).uniform(0.0, 1.0, B).astype(np.float32)
    shape = (heads, D // heads, m.info["vt_ld"])
    tok = np.arange(cfg.N)
    col = (tok & ~12) | ((tok & 4) << 1) | ((tok & 8) >> 1)
    past = np.setdiff1d(np.arange(shape[2]), col)
    m.residual(dev(x), t, 1)
    batch = host(m.debug_read(Buffer.VT, (B,) + shape))
    assert (batch[..., past] == 0).all()
    for k in range(B):
        m.residual(dev(x[k:k + 1]), t[k:k + 1], 1)
        np.testing.assert_array_equal(host(m.debug_read(Buffer.VT, (1,) + shape))[0], batch[k])
    tr = {}
    oracle.residual_one(oracle.load_blob(blob), x[B - 1], t[B - 1], None, 1, trace=tr)
    v = batch[B - 1][..., col].transpose(2, 0, 1).reshape(cfg.N, D)
    assert rel_l2(v, tr["v"]) <= TOL["bf16"]
    m.close()


@pytest.mark.parametrize("HW", [(32, 64), (10, 12), (8, 8)], ids=["512tok", "30tok", "16tok"])
@pytest.mark.parametrize("D,heads", [(128, 2), (144, 2), (96, 2), (64, 2), (48, 2), (208, 2), (240, 2), (256, 2)],
                         ids=["dh64", "dh72", "dh48", "dh32", "dh24", "dh104", "dh120", "dh128"])
def test_attention_scores_far_from_zero(D, heads, HW):
    """Scores whose level per query lies far outside [-64, 64] in exp2 units, on both
    sides: every key entry is 128 plus a small exact integer step, so a query's scores are
    a large offset (its product with the shared part, spread about +-185 exp2 units over
    the queries) plus a spread of a few units between keys. Softmax does not depend on the
    offset, so the result is well conditioned, while the kernels' online softmax meets
    sums that overflow and underflow and maxima far from zero. bf16 attention alone
    (sf_attention) on exact bf16 inputs against the oracle's fp64 softmax: 64 rows run the
    two-query-block kernels (where the grid is large enough for them), four rows the
    one-block ones, and the four rows both ran agree bit for bit. At 30 and 16 tokens a
    single step holds every key: the second key half sees none (16) or only part of its
    keys (30), so the masked, partly empty step meets the offset moves too."""
    from paper_2511_22009_amd import Model, Precision
    cfg = W.Config(f"attn{D}", C=4, H=HW[0], W=HW[1], p=2, D=D, L=1, heads=heads, mlp=128)
    m = Model(W.make_blob(cfg), Precision.BF16, 64)
    N, dh, ldv, R = cfg.N, D // heads, m.info["vt_ld"], 64
    rng = np.random.default_rng(91)
    q = rng.standard_normal((R, heads, N, dh))
    k = 128.0 + rng.integers(-4, 5, (R, heads, N, dh))
    v = rng.standard_normal((R, heads, N, dh))
    qb, kb, vb = (torch.from_numpy(a.astype(np.float32)).to(torch.bfloat16) for a in (q, k, v))
    q64, k64, v64 = (a.float().numpy().astype(np.float64) for a in (qb, kb, vb))
    # the inputs are what this test says: offsets beyond +-64 exp2 units for most queries
    off = np.einsum("rhnd,d->rhn", q64, np.full(dh, 128.0)) / np.sqrt(dh) / np.log(2.0)
    assert (off > 64).mean() > 0.3 and (off < -64).mean() > 0.3
    tok = np.arange(N)
    col = (tok & ~12) | ((tok & 4) << 1) | ((tok & 8) >> 1) if m.info["vt_key_perm"] else tok
    vT = torch.zeros((R, heads, dh, ldv), dtype=torch.bfloat16)
    vT[..., torch.from_numpy(col)] = vb.transpose(2, 3)
    full = m.attention(qb.cuda(), kb.cuda(), vT.cuda()).float()
    part = m.attention(qb[:4].contiguous().cuda(), kb[:4].contiguous().cuda(), vT[:4].contiguous().cuda()).float()
    full, part = host(full), host(part)
    flat = lambda a: a.transpose(1, 0, 2).reshape(N, D)  # noqa: E731  [heads, N, dh] -> [N, D]
    errs = [rel_l2(full[r], oracle.attention(flat(q64[r]), flat(k64[r]), flat(v64[r]), heads)) for r in range(R)]
    assert max(errs) <= ISO["bf16"], max(errs)
    np.testing.assert_array_equal(full[:4], part)
    m.close()


@pytest.mark.parametrize("prec", ["bf16", "fp32"])
@pytest.mark.parametrize("D,heads", [(64, 1), (264, 3), (520, 5), (1032, 43), (1544, 193), (2048, 32)])
def test_modulation_of_many_samples(D, heads, prec):
    """One, four, five and nine samples in a call (one pass over the weights' rows, or several
    with the rows held) give each sample the bits it has alone, at widths of one to eight
    16-byte chunks per lane, and the table of 64-bit sums: fp32 sums of at most 2048 products
    behind two layers whose rounding passes through the sinusoids' phases, 4e-6."""
    from paper_2511_22009_amd import Model, Precision
    cfg = W.Config("mod", C=4, H=4, W=4, p=2, D=D, L=0, heads=heads, mlp=64)
    blob = W.make_blob(cfg, init="tsens")
    m = Model(blob, Precision[prec.upper()], 9)
    t = np.random.default_rng(3).uniform(0.0, 1.0, 9).astype(np.float32)
    full = host(m.modulation(t))
    for n in (1, 4, 5):
        np.testing.assert_array_equal(host(m.modulation(t[:n])), full[:n])
    np.testing.assert_array_equal(host(m.modulation(t[8:])), full[8:])
    om = oracle.load_blob(blob)
    if prec == "bf16":
        om.top["W_fmod"] = bf16_round(om.top["W_fmod"])
    ref = np.stack([oracle.modulation_table(om, t[k], dtype=np.float64).reshape(-1) for k in range(9)])
    assert rel_l2(full, ref) <= 4e-6
    m.close()
