"""The stem probes of the GPU test see what they are for: with a mistake planted in the oracle's max-pool (a row or column
of the map lost, a window without its shared column or row), the probe named for it is off by several times the
tolerance of that test."""
import numpy as np
import pytest

from oracle import forward as oracle_forward
from oracle import ops
from tests import stem_probes as sp
from tests.test_gpu_stem import TOL


def lose(rows=None, cols=None):
    def f(y, x):
        y = y.copy()
        if rows is not None:
            y[:, rows] = 0
        if cols is not None:
            y[:, :, cols] = 0
        return y
    return f


def short_window(axis, at, d):
    """Pooled row or column `at` without element d (0, 1, 2) of its window."""
    def f(y, x):
        y = y.copy()
        xs = np.moveaxis(x, axis, 0)
        taps = [2 * at - 1 + e for e in range(3) if e != d and 0 <= 2 * at - 1 + e < xs.shape[0]]
        line = np.maximum.reduce([xs[t] for t in taps])                # [n][other][c], the max over this axis
        pad = np.full((line.shape[0], line.shape[1] + 2, line.shape[2]), -np.inf)
        pad[:, 1:-1] = line
        n = y.shape[3 - axis]
        pooled = np.maximum.reduce([pad[:, e:e + 2 * n - 1:2] for e in range(3)])
        np.moveaxis(y, axis, 0)[at] = pooled
        return y
    return f


@pytest.mark.parametrize("image,rows", [(64, 2), (128, 7)])
def test_planted_mistakes_fail(image, rows, monkeypatch):
    m = sp.model(image)
    n = len(sp.probes(image, rows))
    x, at = sp.inputs(image, rows, n, 56)
    at = dict(at)
    good = oracle_forward.forward(m, x)
    hp = image // 4
    last = (hp - 1) // rows * rows
    plants = {"last column": lose(cols=hp - 1), "last row": lose(rows=hp - 1), "first column": lose(cols=0),
              "first row": lose(rows=0), "corner": lose(rows=hp - 1, cols=hp - 1), "last block": lose(rows=slice(last, hp)),
              "row line": short_window(1, last, 0)}
    if hp > sp.SEGMENT:
        plants.update({"seam, left": lose(cols=sp.SEGMENT - 1), "seam": short_window(2, sp.SEGMENT, 0),
                       "seam, right": lose(cols=sp.SEGMENT)})
    if "first line" in at:
        plants["first line"] = short_window(1, rows - 1, 2)
    plain = ops.maxpool_nhwc
    assert set(plants) == set(at)
    # the plants' own pooling, with nothing planted, is the oracle's
    ident = short_window(1, 0, 0)                    # row 0's window has no element 0
    monkeypatch.setattr(ops, "maxpool_nhwc", lambda t, k, s, p: ident(plain(t, k, s, p), t))
    assert np.allclose(oracle_forward.forward(m, x[-1:]), good[-1:], rtol=1e-12)
    for name, f in plants.items():
        b = at[name]
        monkeypatch.setattr(ops, "maxpool_nhwc", lambda t, k, s, p: f(plain(t, k, s, p), t))
        err = oracle_forward.normwise_error(oracle_forward.forward(m, x[b:b + 1]), good[b:b + 1])[0]
        print(f"{image}, {name}: {err:.2f}")
        assert err > 3 * TOL, (name, err)
