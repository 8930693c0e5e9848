"""Two 1x1 convolutions of a ResNet block's input in one launch: warm requests (which may take it)
give the same bits as cold ones (a launch each), at sizes on both sides of the rule (rows of the
smaller convolution past 32, both convolutions' tiles within 1024) and with ragged last tiles."""
import numpy as np
import pytest

import synth
from oracle import forward as oracle_forward
from tests.common import infer, log, make_runtime

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("image,batch", [(32, 1), (64, 3), (64, 9), (96, 5), (160, 3), (224, 1), (224, 2)])
def test_same_bits(image, batch):
    log(f"block inputs of {batch} x {image} x {image}")
    m = synth.resnet50(seed=57, classes=10, image=image)
    x = synth.resnet_input(batch, 58, image=image)
    rt, (mid,) = make_runtime([m], batch_max=batch)
    cold = infer(rt, mid, m, x)
    warm = infer(rt, mid, m, x)
    rt.close()
    assert np.array_equal(cold, warm)
    err = oracle_forward.normwise_error(warm[:1], oracle_forward.forward(m, x[:1])).max()
    log(f"  normwise error {err:.2e}")
    assert err <= 2e-2
