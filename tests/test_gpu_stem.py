"""The ResNet stem and its max-pool at several pooled rows per workgroup (1 to 8, also where the last
workgroup has fewer) and one or two column segments, against the oracle on samples of the batch."""
import numpy as np
import pytest

import synth
from oracle import forward as oracle_forward
from tests.common import infer, log, make_runtime

pytestmark = pytest.mark.gpu


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
    assert err <= 2e-2
