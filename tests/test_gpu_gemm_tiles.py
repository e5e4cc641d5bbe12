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

# (width, heads, MLP width, latent H, W, rows); the tiles that the batch's QKV, output, up- and
# down-projection take (a CPU test holds the rule to them); a row alone takes kPipe64, and
# kHalf64 where the sums over K go in halves
CASES = {
    # K 512 and 520
    "w512": (512, 8, 520, 26, 30, 64, "kTile128 kPipeHalf128 kTile128 kPipeHalf128"),
    # K 1160 and 3080
    "w1160": (1160, 29, 3080, 26, 30, 16, "kPipe128x192 kTile128 kTile256x192 kTile128"),
    # K 200 and 7000
    "mlp7000": (200, 5, 7000, 26, 30, 8, "kPipe64 kPipe64 kTile128 kPipe64"),
    # K 384 and 776; 748 tokens: v leaves in groups of four tokens
    "w384": (384, 6, 776, 44, 68, 64, "kPipe128x192 kPipeHalf128x192 kTile128 kPipeHalf128x192"),
    # 4095 rows of 195 tokens, K 760
    "w760": (760, 19, 520, 26, 30, 21, "kTile128x288 kTile128 kTile128 kTile128"),
    # K 640
    "w640": (640, 10, 640, 16, 24, 64, "kPipe128x192 kHalf128 kHalf128 kHalf128"),
    # 5070 rows, K 480 and 776
    "w480": (480, 10, 776, 26, 30, 26, "kTile128 kHalf128x96 kTile128 kHalf128x96"),
    # 6825 rows, K 840 and 1160
    "w840": (840, 35, 1160, 26, 30, 35, "kPipe128x192 kPipe128 kTile256x192 kPipe128"),
    # 7800 rows, K 1128 and 520
    "w1128": (1128, 47, 520, 26, 30, 40, "kPipe128x192 kTile128x288 kTile128 kTile128x288"),
    # 2145 rows, K 648 and 776
    "w648": (648, 27, 776, 26, 30, 11, "kPipe128 kPipe64 kPipe64 kPipe64"),
    # 8190 rows, K 552 and 3064
    "w552": (552, 23, 3064, 26, 30, 42, "kTile128 kTile128 kPipe128x192 kPipe128"),
}


@pytest.mark.parametrize("name", CASES)
def test_projection_tiles(name):
    D, heads, mlp, H, Wd, B, _ = CASES[name]
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
