"""The fp32 linear layer's two kernels (few rows; matrix tiles of 16, 32 or 64 rows) against the
oracle, on both sides of the lines between them, with ragged features, rows and k."""
import numpy as np
import pytest

import synth
from oracle import forward as oracle_forward
from tests.common import infer, log, make_runtime, to_device, torch_dev

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


def test_more_rows_than_one_grid_dimension_holds():
    # 64 rows per workgroup, 65536 workgroups in a grid dimension: the last rows take another, in a pass launched
    # layer by layer and in a replayed graph whose buffers change
    torch, dev = torch_dev()
    width, batch = 8, 65536 * 64 + 70
    rng = np.random.default_rng(5)
    x = rng.standard_normal((batch, width), dtype=np.float32)
    rows = np.r_[0:3, 65536 * 64 - 2:batch]
    for layers in (1, 16):
        log(f"fp32 {layers} x {width}, batch {batch}")
        m = synth.mlp(layers, width, "f32", "none", seed=6)
        rt, (mid,) = make_runtime([m], batch_max=batch)
        ref = oracle_forward.forward(m, x[rows])
        for _ in range(2):                       # the second pass has other buffers
            err = oracle_forward.normwise_error(infer(rt, mid, m, x)[rows], ref).max()
            log(f"  normwise error {err:.2e}")
            assert err <= 1e-4
        xd = to_device(x)
        out = torch.full((batch, width), float("nan"), dtype=torch.float32, device=dev)
        torch.cuda.synchronize()
        s = torch.cuda.Stream(device=dev)
        rt.infer(mid, xd, out, stream=s)
        s.synchronize()
        assert oracle_forward.normwise_error(out.cpu().numpy()[rows], ref).max() <= 1e-4
        rt.close()
