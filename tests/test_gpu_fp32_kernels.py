"""The fp32 matrix-core kernels alone, at the sizes where their tiles can go wrong, against
64-bit results on the same inputs. An fp32 sum of n products has a relative error of about
sqrt(n) 2^-24 (n <= 4096: 4e-6); 1e-6 is what these shapes stay below by a factor of two
or more, and the bound of one element is forty times that."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

from gpu_util import host, torch  # noqa: E402
from helpers import rel_l2  # noqa: E402
from paper_2511_22009_amd import Buffer, Model, Precision  # noqa: E402


def _attention_model(heads, dh, H, Wd):
    D = heads * dh
    cfg = W.Config("attn", C=4, H=H, W=Wd, p=2, D=D, L=1, heads=heads, mlp=D, K=1, schedule="uniform1")
    return cfg, Model(W.make_blob(cfg), Precision.FP32, 1)


def _reference(q, k, v):
    s = np.einsum("rhqd,rhkd->rhqk", q, k, dtype=np.float64) / np.sqrt(q.shape[-1])
    p = np.exp(s - s.max(-1, keepdims=True))
    o = np.einsum("rhqk,rhkd->rhqd", p / p.sum(-1, keepdims=True), v, dtype=np.float64)
    return o.transpose(0, 2, 1, 3).reshape(q.shape[0], q.shape[2], -1)


def _run(m, q, k, v, shift=0):
    """Attention on device copies of q, k, v; shift > 0 moves every operand that many
    floats off its 16-byte boundary."""
    def put(a):
        buf = torch.empty(a.size + shift, device="cuda")
        t = buf[shift:].view(a.shape)
        t.copy_(torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)))
        return t
    vt = np.zeros(v.shape[:2] + (v.shape[3], m.info["vt_ld"]), np.float32)
    vt[..., :v.shape[2]] = v.transpose(0, 1, 3, 2)
    return host(m.attention(put(q), put(k), put(vt)))


@pytest.mark.parametrize("H,Wd", [(2, 2), (6, 10), (8, 8), (6, 22), (10, 26), (20, 28)],
                         ids=["n1", "n15", "n16", "n33", "n65", "n140"])
@pytest.mark.parametrize("heads,dh", [(1, 8), (3, 16), (2, 24), (1, 40), (2, 64), (2, 72), (1, 96), (1, 104), (2, 128)])
def test_attention_fp32(heads, dh, H, Wd):
    cfg, m = _attention_model(heads, dh, H, Wd)
    rng = np.random.default_rng([heads, dh, cfg.N])
    q, k, v = (rng.standard_normal((2, heads, cfg.N, dh)).astype(np.float32) for _ in range(3))
    q *= 3.0
    ref = _reference(q, k, v)
    got = _run(m, q, k, v)
    assert rel_l2(got, ref) < 1e-6
    assert np.max(np.abs(got - ref)) < 4e-5 * np.sqrt(np.mean(ref * ref))
    # operands off their 16-byte boundary take the general kernel: the same result within
    # the same bound
    assert rel_l2(_run(m, q, k, v, shift=1), ref) < 1e-6
    # each row alone gives the bits it has in the batch
    np.testing.assert_array_equal(_run(m, q[1:], k[1:], v[1:])[0], got[1])
    m.close()


def test_attention_fp32_score_levels_and_nan():
    """Scores far above, far below and moving through the row (the running max rises at
    late keys), and a NaN key: its head's outputs are NaN, the other head's are not."""
    cfg, m = _attention_model(2, 48, 20, 28)
    rng = np.random.default_rng(5)
    q, k, v = (rng.standard_normal((1, 2, cfg.N, 48)).astype(np.float32) for _ in range(3))
    q[..., 0], k[..., 0] = 40.0, np.linspace(-60.0, 60.0, cfg.N)  # scores from -350 to 350
    ref = _reference(q, k, v)
    # a score of 350 carries a rounding of about 350 2^-24 sqrt(48) = 1.4e-4 into its exponent
    assert rel_l2(_run(m, q, k, v), ref) < 1.5e-4
    k[0, 1, 70, 3] = np.nan
    got = _run(m, q, k, v)
    assert np.isnan(got[0, :, 48:]).all() and np.isfinite(got[0, :, :48]).all()
    m.close()


def test_gemm_fp32_tiles_and_ragged_k():
    """Widths that are multiples of neither fp32 tile nor of the 32-wide K slice (K 200,
    1032; N 200, 600, 1032). 64 rows of 84 tokens take 64 x 64 tiles for the QKV and MLP
    up-projections and 32 x 32 tiles for the other two, one row 32 x 32 tiles throughout:
    against the oracle (sums of at most 1032 products: 2e-6), and the same bits."""
    import oracle
    cfg = W.Config("odd", C=4, H=14, W=24, p=2, D=200, L=1, heads=5, mlp=1032)
    blob = W.make_blob(cfg, init="tsens")
    m = Model(blob, Precision.FP32, 64)
    x = W.latents(cfg, 64, seed=7)
    t = np.random.default_rng(8).uniform(0.0, 1.0, 64).astype(np.float32)
    put = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    got = host(m.velocity(put(x), t))
    om = oracle.load_blob(blob)
    for k in (0, 31, 63):
        assert rel_l2(got[k], oracle.forward_one(om, x[k], t[k], dtype=np.float64)) < 2e-6
        np.testing.assert_array_equal(host(m.velocity(put(x[k:k + 1]), t[k:k + 1]))[0], got[k])
    m.close()


@pytest.mark.parametrize("C,p,H,Wd,D,heads", [(4, 2, 14, 22, 192, 4), (8, 2, 6, 10, 128, 4), (3, 2, 10, 6, 72, 1),
                                              (1, 4, 20, 12, 200, 5), (4, 1, 3, 5, 1160, 29), (2, 4, 16, 8, 8, 1),
                                              (4, 2, 2, 2, 2048, 16)])
def test_head_fp32(C, p, H, Wd, D, heads):
    """Final LayerNorm, modulate and output map alone (a network without blocks): patches of
    4 to 32 values, widths that fill no column step, token counts that end inside a
    workgroup's four rows (and put each slot's rows elsewhere in it): against the oracle in 64
    bits, and every slot alone gives its bits in the batch."""
    import oracle
    cfg = W.Config("head", C=C, H=H, W=Wd, p=p, D=D, L=0, heads=heads, mlp=D, K=5, schedule="uniform5")
    tens = W.make_weights(cfg, init="tsens")
    tens["pos"] = np.random.default_rng(4).standard_normal((cfg.N, D)).astype(np.float32)
    blob = W.write_blob(cfg, tens)
    m = Model(blob, Precision.FP32, 5)
    x = W.latents(cfg, 5, seed=9)
    t = np.random.default_rng(10).uniform(0.0, 1.0, 5).astype(np.float32)
    put = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    got = host(m.velocity(put(x), t))
    om = oracle.load_blob(blob)
    for k in range(5):
        assert rel_l2(got[k], oracle.forward_one(om, x[k], t[k], dtype=np.float64)) < 2e-6
        np.testing.assert_array_equal(host(m.velocity(put(x[k:k + 1]), t[k:k + 1]))[0], got[k])
    m.close()


def _fma(a, b, c):
    """fp32 a * b + c with one rounding: the product is exact in 64 bits (whose own rounding of
    the sum, then to 32 bits, misses the single rounding about once in 2^29)."""
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(np.float32)


def _butterfly(x):
    """Sum over the 64 lanes of the last axis by xor 32, 16, 8, 4, 2, 1."""
    for d in (32, 16, 8, 4, 2, 1):
        x = x + x[..., np.arange(64) ^ d]
    return x[..., 0]


def _head_in_order(h, table, W_f, b_f):
    """The head in fp32 in its order of sums: h [rows, N, D], table [rows, 2D] (shift, scale)
    -> [rows, N, P]. Lane l of a wavefront holds columns 4 (l + 64 i) .. + 3."""
    R, N, D = h.shape
    one, nv = np.float32(1.0), (D + 255) // 256

    def lanes(a):  # [..., D] -> [..., nv, 64, 4], zeros past the end
        out = np.zeros(a.shape[:-1] + (nv * 256,), np.float32)
        out[..., :D] = a
        return out.reshape(a.shape[:-1] + (nv, 64, 4))

    def pairs(a, b):
        return _fma(a[..., 0], b[..., 0], a[..., 1] * b[..., 1]) + _fma(a[..., 2], b[..., 2], a[..., 3] * b[..., 3])

    v, live = lanes(h), lanes(np.ones(D, np.float32)) > 0
    s = np.zeros((R, N, 64), np.float32)
    for i in range(nv):
        s = s + ((v[:, :, i, :, 0] + v[:, :, i, :, 1]) + (v[:, :, i, :, 2] + v[:, :, i, :, 3]))
    d = v - (_butterfly(s) / np.float32(D))[..., None, None, None]
    q = np.zeros((R, N, 64), np.float32)
    for i in range(nv):
        q = np.where(live[i, :, 0], q + pairs(d[:, :, i], d[:, :, i]), q)
    rstd = one / np.sqrt(_butterfly(q) / np.float32(D) + np.float32(1e-6))
    shift, scale = lanes(table[:, :D])[:, None], lanes(table[:, D:])[:, None]
    y = np.where(live, _fma(d * rstd[..., None, None, None], one + scale, shift), np.float32(0.0))
    w, out = lanes(W_f), np.empty((R, N, W_f.shape[0]), np.float32)
    for f in range(W_f.shape[0]):
        t = np.zeros((R, N, 64), np.float32)
        for i in range(nv):
            t = t + pairs(y[:, :, i], np.broadcast_to(w[f, i], y[:, :, i].shape))
        out[..., f] = _butterfly(t) + b_f[f]
    return out


@pytest.mark.parametrize("prec", ["bf16", "fp32"])
@pytest.mark.parametrize("C,p,H,Wd,D,heads", [(4, 2, 14, 22, 768, 12), (8, 2, 6, 10, 256, 4), (3, 2, 10, 6, 264, 3),
                                              (1, 2, 20, 12, 1160, 29), (2, 4, 16, 8, 8, 1), (4, 2, 6, 2, 2048, 16)])
def test_head_order_of_sums(C, p, H, Wd, D, heads, prec):
    """The head's sums have one order, bit for bit: a stream step feeds its last bits back into
    the queue, where they travel through the roundings of later steps."""
    cfg = W.Config("head", C=C, H=H, W=Wd, p=p, D=D, L=0, heads=heads, mlp=D, K=3, schedule="uniform3")
    tens = W.make_weights(cfg, init="tsens")
    tens["pos"] = np.random.default_rng(14).standard_normal((cfg.N, D)).astype(np.float32)
    m = Model(W.write_blob(cfg, tens), Precision[prec.upper()], 3)
    x = W.latents(cfg, 3, seed=19)
    t = np.random.default_rng(20).uniform(0.0, 1.0, 3).astype(np.float32)
    got = host(m.velocity(torch.from_numpy(x).cuda(), t))
    h = host(m.debug_read(Buffer.H, (3, cfg.N, D)))
    table = host(m.debug_read(Buffer.TABLE, (3, 2 * D)))
    ref = _head_in_order(h, table, np.asarray(tens["W_f"], np.float32), np.asarray(tens["b_f"], np.float32))
    ref = ref.reshape(3, H // p, Wd // p, p, p, C).transpose(0, 5, 1, 3, 2, 4).reshape(got.shape)
    np.testing.assert_array_equal(got, ref)
    m.close()
