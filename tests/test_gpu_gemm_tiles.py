"""Every tile shape, ring depth and k split of the tiled contraction against the oracle: one
linear layer (fp32 output) at widths and batches on both sides of the plan's lines, with ragged
rows, ragged output features and a last k-stage that is not whole."""
import numpy as np
import pytest

import synth
from oracle import forward as oracle_forward
from tests.common import infer, log, make_runtime

pytestmark = pytest.mark.gpu

# (width = features = k, batch, the plan: features and rows of a tile, k-stages in the ring, k splits); a width of a
# multiple of 128 has blocked weights
SHAPES = [
    (64, 33, (32, 32, 4, 1)),
    (72, 35, (32, 32, 4, 1)),
    (200, 65, (32, 32, 4, 1)),
    (512, 40, (32, 32, 6, 1)),
    (1000, 131, (32, 32, 6, 1)),
    (1152, 240, (32, 32, 4, 1)),
    (1000, 700, (64, 32, 5, 1)),
    (1024, 390, (64, 32, 5, 1)),
    (2400, 40, (64, 32, 5, 4)),
    (2560, 50, (64, 32, 5, 4)),
    (64, 20000, (64, 64, 4, 1)),
    (776, 1000, (64, 64, 4, 1)),
    (1024, 800, (64, 64, 4, 1)),
    (776, 2600, (64, 64, 2, 1)),
    (1152, 1900, (64, 64, 2, 1)),
    (1224, 2570, (128, 128, 3, 1)),
    (1280, 2570, (128, 128, 3, 1)),
    (520, 8010, (128, 128, 2, 1)),
    (512, 8510, (128, 128, 2, 1)),
    (1032, 8010, (256, 128, 3, 1)),
    (2048, 4000, (256, 128, 3, 1)),
    (4088, 4000, (256, 256, 2, 1)),
    (4096, 4090, (256, 256, 2, 1)),
]


@pytest.mark.parametrize("width,batch,plan", SHAPES, ids=["%dx%d-%dx%d-ring%d-split%d" % (w, b, *p) for w, b, p in SHAPES])
def test_linear_layer(width, batch, plan):
    log(f"linear {batch} x {width} x {width}: {plan}")
    m = synth.mlp(1, width, "bf16", "none", seed=900 + width, bias_std=0.5)
    x = synth.mlp_input(batch, width, "bf16", 901 + batch)
    rt, (mid,) = make_runtime([m], batch_max=batch)
    got = infer(rt, mid, m, x)
    again = infer(rt, mid, m, x)
    rt.close()
    assert np.all(np.isfinite(got))
    assert np.array_equal(got, again)
    # every row of the first and last tiles, a sample of the others
    rows = np.unique(np.concatenate([np.arange(min(batch, 70)), np.arange(max(0, batch - 290), batch),
                                     np.arange(0, batch, 37)]))
    ref = oracle_forward.forward(m, x[rows])
    err = oracle_forward.normwise_error(got[rows], ref).max()
    # exact products, fp32 sums in some order: |error| <= width 2^-24 sum |w x|, and that sum is
    # about 0.64 sqrt(width) where the row's largest output is at least 2
    tol = width * 2.0 ** -24 * 0.64 * np.sqrt(width) / 2 + 2.0 ** -23
    log(f"  normwise error {err:.2e} (tol {tol:.2e})")
    assert err <= tol
