"""Self-attention at every sequence length and every number of waves per workgroup, through one
encoder layer, against the oracle; each sample alone equals the sample in its batch."""
import numpy as np
import pytest

import synth
from tests.common import check_parity, infer, log, make_runtime

pytestmark = pytest.mark.gpu


# 4 heads: workgroups of 4 waves; of 8 from 24 samples on beyond 128; of a wave per 16 queries from 48
# samples on up to 192
@pytest.mark.parametrize("seq,batch", [(32, 3), (64, 2), (96, 3), (128, 3), (160, 3), (160, 24), (160, 48), (192, 23),
                                       (192, 25), (192, 49), (224, 2), (224, 24), (256, 2), (256, 26)])
def test_sequence_lengths(seq, batch):
    log(f"attention: {batch} x {seq}, 4 heads")
    # Weights of std w give queries and keys of std 16 w and exponents q k / 8 of std 256 w^2; rounding q and k to bf16 moves a score by up to 2^-8 of it. At 0.05 (scores of
    # 0.64, moved by 2.5e-3) a probability is off by 0.3%, at 0.2 (10, by 0.04) by more than the 2e-2 allowed.
    m = synth.bert(seed=61, layers=1, d=256, heads=4, ffn=64, seq=seq, vocab=300, maxpos=256, std=0.05)
    ids = synth.bert_input(batch, 62 + seq, seq=seq, vocab=300)
    rt, (mid,) = make_runtime([m], batch_max=batch)
    got = infer(rt, mid, m, ids)
    check_parity(got, m, ids, 2e-2)
    alone = infer(rt, mid, m, ids[-1:])
    rt.close()
    # other batches may take other tiles and waves, which round sums otherwise: within bf16 rounding
    assert np.abs(alone[0] - got[-1]).max() <= 2e-2 * np.abs(got[-1]).max()
