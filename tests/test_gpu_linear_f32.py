"""The fp32 linear layer's two kernels (few rows; matrix tiles of 16, 32 or 64 rows) against the
oracle, on both sides of the lines between them, with ragged features, rows and k."""
import numpy as np
import pytest

import synth
from oracle import forward as oracle_forward
from tests.common import infer, log, make_runtime

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,batch", [(64, 4), (64, 5), (72, 17), (136, 255), (256, 16), (520, 33), (1000, 64),
                                         (1000, 100), (1000, 250), (1024, 256), (1032, 33), (2000, 6)])
def test_linear_layer(width, batch):
    log(f"fp32 linear {batch} x {width} x {width}")
    m = synth.mlp(1, width, "f32", "none", seed=700 + width, bias_std=0.5)
    x = synth.mlp_input(batch, width, "f32", 701 + batch)
    rt, (mid,) = make_runtime([m], batch_max=batch)
    got = infer(rt, mid, m, x)
    again = infer(rt, mid, m, x)
    rt.close()
    assert np.array_equal(got, again)
    err = oracle_forward.normwise_error(got, oracle_forward.forward(m, x)).max()
    # a sum over k is 64 partial sums of width / 64 products each, joined in 6 steps, plus the bias:
    # |error| <= (width / 64 + 8) 2^-24 sum |w x|, that sum about 0.64 sqrt(width), outputs of 2 and more
    tol = (width / 64 + 8) * 2.0 ** -24 * max(1.0, 0.64 * np.sqrt(width) / 2)
    log(f"  normwise error {err:.2e} (tol {tol:.2e})")
    assert err <= tol


@pytest.mark.parametrize("batch", [3, 5, 8])
def test_rows_do_not_depend_on_each_other(batch):
    # infinities in one row stay in that row, also where another row or k beyond the width is padded
    m = synth.mlp(1, 136, "f32", "none", seed=3)
    x = synth.mlp_input(batch, 136, "f32", 4)
    rt, (mid,) = make_runtime([m], batch_max=batch)
    clean = infer(rt, mid, m, x)
    x[0, 0] = np.inf
    got = infer(rt, mid, m, x)
    rt.close()
    assert np.array_equal(got[1:], clean[1:])
    assert np.all(np.isinf(got[0]))
