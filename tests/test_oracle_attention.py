"""The GPU test of attention sees what it is for: with a mistake planted in the oracle's attention (the first or last 16
keys left out, half the scale, a query tile given to another one) its models' outputs move by several times its
tolerance at every sequence length."""
import numpy as np
import pytest

import synth
from oracle import forward as oracle_forward
from oracle import ops
from tests.test_gpu_attention import TOL, encoder

PLANTS = {
    "last keys": lambda q, k, v: PLAIN(q, k[..., :-16, :], v[..., :-16, :]),
    "first keys": lambda q, k, v: PLAIN(q, k[..., 16:, :], v[..., 16:, :]),
    "half the scale": lambda q, k, v: PLAIN(q / 2, k, v),
    "query tile": lambda q, k, v: PLAIN(np.concatenate([q[..., :-16, :], q[..., -32:-16, :]], axis=-2), k, v),
}
PLAIN = ops.attention


@pytest.mark.parametrize("seq", [32, 64, 96, 128, 160, 192, 224, 256])
def test_planted_mistakes_fail(seq, monkeypatch):
    m = encoder(seq)
    ids = synth.bert_input(1, 62 + seq, seq=seq, vocab=300)
    good = oracle_forward.forward(m, ids)
    for name, f in PLANTS.items():
        monkeypatch.setattr(ops, "attention", f)
        err = oracle_forward.normwise_error(oracle_forward.forward(m, ids), good)[0]
        print(f"{seq}, {name}: {err:.2f}")
        assert err > 5 * TOL, (name, err)
