"""GPU parity for attention over at most 32 keys: the bf16 attention kernels split each
64-key step into two halves of 32 keys, so with 32 or fewer keys (a 4x8x8 latent, or a
short cross-attention context) the second half holds no key at all. Its wavefronts must
contribute nothing, not NaN. Velocity against the oracle, relative L2 per sample."""
import numpy as np
import pytest

import oracle
import workloads as W
from conftest import oracle_model
from helpers import TOL_BF16, TOL_FP32, rel_l2

pytestmark = pytest.mark.gpu

from gpu_util import dev, host, model  # noqa: E402

TOL = {"fp32": TOL_FP32, "bf16": TOL_BF16}
PRECS = ["fp32", "bf16"]


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("name", ["short16", "short16_dh72", "short32_dh64"])
def test_short_sequence_velocity_parity(name, prec):
    cfg = W.get_config(name)
    t, _ = W.slot_times(cfg)
    x = W.latents(cfg, cfg.K)
    got = host(model(name, prec).velocity(dev(x), t))
    assert np.isfinite(got).all()
    ref = oracle.velocity(oracle_model(name), x, t)
    errs = [rel_l2(got[k], ref[k]) for k in range(cfg.K)]
    assert max(errs) <= TOL[prec], errs


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("name", ["tiny_cfg_ctx20", "tiny_cfg_ctx32"])
def test_short_context_guided_velocity_parity(name, prec):
    from paper_2511_22009_amd import Cond
    cfg = W.get_config(name)
    t, _ = W.slot_times(cfg)
    x = W.latents(cfg, cfg.K)
    ctx, nctx = W.context(cfg, cfg.K), W.null_context(cfg)
    got = host(model(name, prec).velocity(dev(x), t, Cond(dev(ctx), dev(nctx), cfg.guidance)))
    assert np.isfinite(got).all()
    ref = oracle.velocity(oracle_model(name), x, t, ctx, nctx, cfg.guidance)
    errs = [rel_l2(got[k], ref[k]) for k in range(cfg.K)]
    assert max(errs) <= TOL[prec], errs


@pytest.mark.parametrize("D,heads", [(1152, 16), (512, 8), (640, 10), (192, 4)])
@pytest.mark.parametrize("H,Wd", [(2, 2), (4, 4), (8, 8)], ids=["n1", "n4", "n16"])
def test_fewer_tokens_than_a_row_block(H, Wd, D, heads):
    """One row of 1, 4 or 16 tokens in a model that holds one row: the gated residual
    projections end inside the first of a tile's 32-row blocks, so later blocks lie past the
    matrix and past the only row of the modulation table."""
    from paper_2511_22009_amd import Model, Precision
    cfg = W.Config("few", C=4, H=H, W=Wd, p=2, D=D, L=2, heads=heads, mlp=4 * D, K=1, schedule="uniform1")
    blob = W.make_blob(cfg, init="tsens")
    om = oracle.load_blob(blob)
    x, t = W.latents(cfg, 1, seed=31), np.array([0.7], np.float32)
    m = Model(blob, Precision.BF16, 1)
    assert rel_l2(host(m.velocity(dev(x), t))[0], oracle.velocity(om, x, t)[0]) <= TOL_BF16
    h = host(m.residual(dev(x), t, 2))[0]
    ref, _ = oracle.residual_one(om, x[0], t[0], None, 2)
    assert rel_l2(h, ref) <= TOL_BF16
    m.close()
