"""Inputs and outputs off a 16-byte boundary give the bits of aligned ones. bf16 MLP inputs at 2-byte residues
of 16, past the skinny kernel's rows, launched one by one and replayed as a graph, with row-major and blocked
weights; fp32 MLP outputs at 4-byte residues."""
import numpy as np
import pytest

import synth
from tests.common import check_parity, infer, log, make_runtime, to_device, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,width,batch", [(1, 72, 35), (3, 200, 65), (2, 512, 40), (2, 776, 300), (16, 64, 33)])
def test_mlp_input_at_any_element(layers, width, batch):
    torch, dev = torch_dev()
    m = synth.mlp(layers, width, "bf16", "gelu", seed=71)
    x = synth.mlp_input(batch, width, "bf16", 72)
    rt, (mid,) = make_runtime([m], batch_max=batch)
    aligned = infer(rt, mid, m, x)
    check_parity(aligned, m, x, 2e-2)
    flat = to_device(x).reshape(-1)
    s = torch.cuda.Stream(device=dev)
    for shift in (1, 2, 4, 7, 0, 3):
        log(f"{layers} x {width}, batch {batch}: input {2 * shift} bytes past a 16-byte boundary")
        buf = torch.zeros(flat.numel() + 16, dtype=flat.dtype, device=dev)
        buf[shift:shift + flat.numel()] = flat
        xs = buf[shift:shift + flat.numel()].view(batch, width)
        assert xs.data_ptr() % 16 == 2 * shift
        for _ in range(2):
            out = torch.full((batch, width), float("nan"), dtype=torch.float32, device=dev)
            torch.cuda.synchronize()
            rt.infer(mid, xs, out, stream=s)
            s.synchronize()
            assert np.array_equal(out.cpu().numpy(), aligned), shift
    rt.evict(mid)                                     # cold, from an unaligned input
    out = torch.full((batch, width), float("nan"), dtype=torch.float32, device=dev)
    torch.cuda.synchronize()
    rt.infer(mid, xs, out, stream=s)
    s.synchronize()
    assert np.array_equal(out.cpu().numpy(), aligned)
    rt.close()


@pytest.mark.parametrize("layers,width,batch", [(1, 136, 5), (1, 72, 64), (2, 520, 33)])
def test_fp32_output_at_any_element(layers, width, batch):
    # the matrix tiles store whole vectors where the output starts at a 16-byte boundary, else element by element
    torch, dev = torch_dev()
    m = synth.mlp(layers, width, "f32", "relu", seed=73)
    x = synth.mlp_input(batch, width, "f32", 74)
    rt, (mid,) = make_runtime([m], batch_max=batch)
    aligned = infer(rt, mid, m, x)
    check_parity(aligned, m, x, 1e-4)
    xd = to_device(x)
    s = torch.cuda.Stream(device=dev)
    n = batch * width
    for shift in (1, 2, 3):
        log(f"{layers} x {width}, batch {batch}: output {4 * shift} bytes past a 16-byte boundary")
        buf = torch.full((n + 8,), float("nan"), dtype=torch.float32, device=dev)
        out = buf[shift:shift + n].view(batch, width)
        assert out.data_ptr() % 16 == 4 * shift
        torch.cuda.synchronize()
        rt.infer(mid, xd, out, stream=s)
        s.synchronize()
        got = buf.cpu().numpy()
        assert np.array_equal(got[shift:shift + n].reshape(batch, width), aligned)
        assert np.all(np.isnan(got[:shift])) and np.all(np.isnan(got[shift + n:]))
    rt.close()
