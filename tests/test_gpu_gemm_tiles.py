"""Every tile shape, ring depth and k split of the tiled contraction against the oracle: one
linear layer (fp32 output) at widths and batches on both sides of the plan's lines, with ragged
rows, ragged output features and a last k-stage that is not whole."""
import numpy as np
import pytest

import synth
from oracle import forward as oracle_forward
from tests.common import infer, log, make_runtime

pytestmark = pytest.mark.gpu

# (width = features = k, batch, what the plan makes of it)
SHAPES = [
    (64, 33, "32 x 32, one stage"),
    (72, 35, "32 x 32, ragged stage of 8"),
    (200, 65, "32 x 32, ragged"),
    (512, 40, "32 x 32, six stages, blocked weights"),
    (1000, 131, "32 x 32, six stages, ragged"),
    (1152, 240, "32 x 32, four stages, blocked weights"),
    (1000, 700, "64 x 32, five stages, ragged"),
    (1024, 390, "64 x 32, five stages, blocked weights"),
    (2400, 40, "64 x 32 split over k, ragged"),
    (2560, 50, "64 x 32 split over k, blocked weights"),
    (64, 20000, "64 x 64, four stages, few features"),
    (776, 1000, "64 x 64, four stages, ragged"),
    (1024, 800, "64 x 64, four stages, blocked weights"),
    (776, 2600, "64 x 64, two stages, ragged"),
    (1152, 1900, "64 x 64, two stages, blocked weights"),
    (1224, 2570, "128 x 128, three stages, ragged"),
    (1280, 2570, "128 x 128, three stages, blocked weights"),
    (520, 8010, "128 x 128, two stages, ragged"),
    (512, 8510, "128 x 128, two stages, blocked weights"),
    (1032, 8010, "256 x 128, ragged"),
    (2048, 4000, "256 x 128, blocked weights"),
    (4088, 4000, "256 x 256, ragged"),
    (4096, 4090, "256 x 256, blocked weights"),
]


@pytest.mark.parametrize("width,batch,plan", SHAPES)
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
