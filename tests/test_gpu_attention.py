"""Self-attention at every sequence length and every number of waves per workgroup, through one
encoder layer, against the oracle; each sample alone equals the sample in its batch.
tests/test_oracle_attention.py shows that a lost key tile or another scale exceeds the tolerance."""
import numpy as np
import pytest

import synth
from tests.common import check_parity, infer, log, make_runtime

pytestmark = pytest.mark.gpu

TOL = 2e-2


def encoder(seq):
    # Weights of std w give queries and keys of std 16 w and exponents q k / 8 of std 256 w^2, 2.56 at 0.1, so that
    # attention singles keys out (at 0.05, 0.64, it is nearly uniform: a lost key tile moved the output by less
    # than the tolerance). Rounding q and k to bf16 moves an exponent by 2.56 sqrt(2) 2^-9 / sqrt(3) = 4e-3 rms, a
    # probability by as much of itself; the values' and the output's own rounding adds 2^-9 each.
    return synth.bert(seed=61, layers=1, d=256, heads=4, ffn=64, seq=seq, vocab=300, maxpos=256, std=0.1)


# 4 heads: workgroups of 4 waves; of 8 from 24 samples on beyond 128; of a wave per 16 queries from 48
# samples on up to 192
@pytest.mark.parametrize("seq,batch", [(32, 3), (64, 2), (96, 3), (128, 3), (160, 3), (160, 24), (160, 48), (192, 23),
                                       (192, 25), (192, 49), (224, 2), (224, 24), (256, 2), (256, 26)])
def test_sequence_lengths(seq, batch):
    log(f"attention: {batch} x {seq}, 4 heads")
    m = encoder(seq)
    ids = synth.bert_input(batch, 62 + seq, seq=seq, vocab=300)
    rt, (mid,) = make_runtime([m], batch_max=batch)
    got = infer(rt, mid, m, ids)
    check_parity(got, m, ids, TOL)
    alone = infer(rt, mid, m, ids[-1:])
    rt.close()
    # other batches may take other tiles and waves, which round sums otherwise: within bf16 rounding
    assert np.abs(alone[0] - got[-1]).max() <= TOL * np.abs(got[-1]).max()
