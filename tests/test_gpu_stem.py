"""The ResNet stem and its max-pool, through the whole network, at several pooled rows per workgroup (1 to 8, also where
the last workgroup has fewer) and one or two column segments, against the oracle on samples of the batch: dense images,
which a fault in one row or column moves by less than the tolerance, and images that are zero but for a few rows
or columns, which it moves by several times as much (tests/test_oracle_stem_probes.py)."""
import numpy as np
import pytest

import synth
from oracle import forward as oracle_forward
from tests import stem_probes as sp
from tests.common import infer, log, make_runtime

pytestmark = pytest.mark.gpu

TOL = 2e-2          # 50 layers of bf16 activations


def rows_per_workgroup(image, batch):
    """Pooled rows a workgroup of the stem owns: as few as make at most 512 workgroups, up to 8."""
    hp = image // 4
    segs = -(-hp // sp.SEGMENT)
    return min(8, -(-segs * hp * batch // 512))


@pytest.mark.parametrize("image,batch,rows", [(64, 16, 1), (64, 60, 2), (96, 64, 3), (128, 30, 4), (128, 50, 7), (160, 45, 8),
                                              (160, 38, 6), (224, 12, 3), (224, 32, 7)])
def test_edges(image, batch, rows):
    assert rows_per_workgroup(image, batch) == rows
    log(f"stem edges: {batch} x {image} x {image}, {rows} pooled rows per workgroup")
    m = sp.model(image)
    x, at = sp.inputs(image, rows, batch, 56)
    rt, (mid,) = make_runtime([m], batch_max=batch)
    got = infer(rt, mid, m, x)
    rt.close()
    assert np.all(np.isfinite(got))
    pick = [0] + [b for _, b in at]
    err = oracle_forward.normwise_error(got[pick], oracle_forward.forward(m, x[pick]))
    for (name, _), e in zip([("dense", 0)] + at, err):
        log(f"  {name}: {e:.2e}")
    assert err.max() <= TOL


@pytest.mark.parametrize("image,batch", [(32, 2), (64, 84), (64, 160), (96, 64), (128, 70), (160, 25), (224, 9)])
def test_batches(image, batch):
    log(f"stem: {batch} x {image} x {image}")
    m = synth.resnet50(seed=55, classes=10, image=image)
    x = synth.resnet_input(batch, 56, image=image)
    rt, (mid,) = make_runtime([m], batch_max=batch)
    got = infer(rt, mid, m, x)
    rt.close()
    assert np.all(np.isfinite(got))
    pick = sorted({0, batch // 2, batch - 1})
    err = oracle_forward.normwise_error(got[pick], oracle_forward.forward(m, x[pick])).max()
    log(f"  normwise error {err:.2e}")
    assert err <= TOL
