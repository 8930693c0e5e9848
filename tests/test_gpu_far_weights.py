"""Requests that read the weights over the host link in place (a first request under direct_max_bytes, zero-copy
contexts), past the rows of the skinny kernels: other orders of tiles, other tiles and padded grids, and the bits of
warm requests; also where a graph captured on one side serves the other."""
import numpy as np
import pytest

import paper_2306_03622_amd as tp
import synth
from tests.common import check_parity, infer, log, make_runtime

pytestmark = pytest.mark.gpu

MODELS = [
    (lambda: synth.mlp(2, 512, "bf16", "gelu", seed=81), 300),
    (lambda: synth.mlp(1, 200, "bf16", "none", seed=82), 1000),
    (lambda: synth.mlp(16, 128, "bf16", "gelu", seed=83), 200),          # replayed as a graph
    (lambda: synth.mlp(1, 696, "f32", "none", seed=84), 64),
    (lambda: synth.mlp(1, 696, "f32", "none", seed=84), 16),
    (lambda: synth.mlp(2, 136, "f32", "relu", seed=85), 200),
    (lambda: synth.mlp(16, 136, "f32", "none", seed=86), 40),            # replayed as a graph
    (lambda: synth.bert(seed=87, layers=3, d=128, heads=2, ffn=512, seq=64, vocab=300, maxpos=64), 3),
    (lambda: synth.bert(seed=87, layers=3, d=128, heads=2, ffn=512, seq=64, vocab=300, maxpos=64), 12),    # too many rows for it
]


@pytest.mark.parametrize("k", range(len(MODELS)))
def test_direct_requests_equal_warm_ones(k):
    m, batch = MODELS[k][0](), MODELS[k][1]
    log(f"{m.arch} {m.dtype} {m.dims}, batch {batch}: {m.total_bytes} bytes read in place")
    assert m.total_bytes <= 2 << 20
    x = synth.config_input(m, batch, 91)
    rt, (mid,) = make_runtime([m], batch_max=batch, direct_max_bytes=2 << 20)
    direct = infer(rt, mid, m, x)
    check_parity(direct, m, x, 1e-4 if m.dtype == "f32" else 2e-2)
    assert np.array_equal(infer(rt, mid, m, x), direct)                  # warm
    rt.evict(mid)
    assert np.array_equal(infer(rt, mid, m, x), direct)                  # direct again
    assert np.array_equal(infer(rt, mid, m, x), direct)
    rt.close()


@pytest.mark.parametrize("make,batch", [(lambda: synth.mlp(2, 1000, "bf16", "gelu", seed=88), 300),
                                        (lambda: synth.mlp(2, 1000, "f32", "relu", seed=89), 130),
                                        (lambda: synth.mlp(2, 2056, "f32", "relu", seed=89), 30),
                                        (lambda: synth.mlp(2, 72, "f32", "relu", seed=89), 6),
                                        (lambda: synth.resnet50(seed=90, classes=10, image=64), 9),
                                        (lambda: synth.resnet50(seed=90, classes=10, image=224), 4)])
def test_zero_copy_equals_warm(make, batch):
    m = make()
    x = synth.config_input(m, batch, 92)
    rt, (mid,) = make_runtime([m], batch_max=batch)
    infer(rt, mid, m, x)
    warm = infer(rt, mid, m, x)
    rt.close()
    rt, (mid,) = make_runtime([m], batch_max=batch, copy_method=tp.TP_COPY_ZERO)
    log(f"{m.arch} {m.dtype} {m.dims}, batch {batch}: zero copy")
    assert np.array_equal(infer(rt, mid, m, x), warm)
    rt.close()
