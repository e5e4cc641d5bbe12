"""bf16 projections at sizes that end inside a tile in every direction (rows, columns, K
slices), on the tiles that a batch of rows takes and the ones a single row takes: the
residual stream against the oracle, and the same bits for a row alone and in the batch."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

from gpu_util import dev, host  # noqa: E402
from helpers import TOL_BF16, rel_l2  # noqa: E402
from paper_2511_22009_amd import Model, Precision  # noqa: E402

# (width, heads, MLP width, latent H, W, rows) and the tiles of the batch
CASES = {
    # QKV 1536: 128 x 128, fragments ahead; output and down-projection 512: 128 x 128 with both
    # halves in a wavefront, K 512 and 520; up-projection 520: 128 x 128, register-staged
    "w512": (512, 8, 520, 26, 30, 64),
    # QKV 3480 and up-projection 3080: 256 x 192, K 1160, the second register-staged; output 1160: 128 x 128 registers
    "w1160": (1160, 29, 3080, 26, 30, 16),
    # up-projection 7000: 128 x 192, K 200; the others 64 x 64, the last with K 7000
    "mlp7000": (200, 5, 7000, 26, 30, 8),
    # output and down-projection 384: 128 x 192 with both halves in a wavefront (K 384, 776),
    # QKV 1152: 128 x 192; 748 tokens: v leaves in groups of four tokens
    "w384": (384, 6, 776, 44, 68, 64),
    # QKV 2280: 128 x 288 (4095 rows, 195 tokens, K 760)
    "w760": (760, 19, 520, 26, 30, 21),
    # output and down-projection 640: 128 x 128 with the halves over two wavefronts
    "w640": (640, 10, 640, 16, 24, 64),
}


@pytest.mark.parametrize("name", CASES)
def test_projection_tiles(name):
    D, heads, mlp, H, Wd, B = CASES[name]
    cfg = W.Config(name, C=4, H=H, W=Wd, p=2, D=D, L=1, heads=heads, mlp=mlp)
    blob = W.make_blob(cfg, init="tsens")
    om = oracle.load_blob(blob)
    m = Model(blob, Precision.BF16, B)
    x = W.latents(cfg, B, seed=21)
    t = np.random.default_rng(22).uniform(0.0, 1.0, B).astype(np.float32)
    got = m.residual(dev(x), t, 1)
    for k in (0, B // 2 - 1, B - 1):
        alone = host(m.residual(dev(x[k:k + 1]), t[k:k + 1], 1))[0]
        mine = host(got[k])
        np.testing.assert_array_equal(alone, mine)
    ref, _ = oracle.residual_one(om, x[B - 1], t[B - 1], None, 1)
    assert rel_l2(mine, ref) <= TOL_BF16
    # the block's own contribution, too: the stream is mostly the embedding
    h0 = host(m.residual(dev(x[B - 1:]), t[B - 1:], 0))[0]
    ref0, _ = oracle.residual_one(om, x[B - 1], t[B - 1], None, 0)
    assert rel_l2(mine - h0, ref - ref0) <= TOL_BF16
    m.close()
