"""Images that are zero but for a few rows or columns, so that what the network makes of them hangs on a few pooled rows
or columns of its stem: its last and first ones, those at the seam of two column segments, and those at the line
between two row blocks. With zero biases the logits are linear in scale, and a lost row or column shows in full."""
import numpy as np

import synth

SEGMENT = 31        # pooled columns of a workgroup


def probes(image, rows):
    """(name, row or None, column or None) of the nonzero input, for `rows` pooled rows per workgroup."""
    hp = image // 4
    out = [("last column", None, image - 1), ("last row", image - 1, None), ("first column", None, 0),
           ("first row", 0, None), ("corner", image - 1, image - 1)]
    if hp > SEGMENT:
        # convolution column 2 SEGMENT - 1 belongs to the windows of both segments
        out += [("seam, left", None, 4 * SEGMENT - 4), ("seam", None, 4 * SEGMENT - 2), ("seam, right", None, 4 * SEGMENT)]
    if rows < hp:
        last = (hp - 1) // rows * rows              # first pooled row of the last workgroup
        out += [("last block", 4 * last, None), ("row line", 4 * last - 2, None)]
        if rows < last:
            out += [("first line", 4 * rows - 2, None)]
    return out


def model(image):
    return synth.resnet50(seed=55, classes=10, image=image, bias_std=0.0)


def inputs(image, rows, batch, seed):
    """A batch that ends in one sample per probe, the others dense; the probes' names with their samples."""
    x = synth.resnet_input(batch, seed, image=image)
    ps = probes(image, rows)
    assert len(ps) < batch or batch == len(ps)
    at = []
    for i, (name, row, col) in enumerate(ps):
        b = batch - len(ps) + i
        keep = np.zeros((image, image), bool)
        if row is None:
            keep[:, col] = True
        elif col is None:
            keep[row, :] = True
        else:
            keep[row - 1:row + 1, col - 1:col + 1] = True
        x[b][~keep] = 0
        at.append((name, b))
    return x, at
