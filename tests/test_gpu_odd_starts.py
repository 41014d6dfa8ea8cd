"""Inputs, z, theta0 and outputs that start at an odd element of a larger buffer (views of a flat vector): the same
bits as from buffers of their own, for every kind and both sizes of FFD's block."""
import pytest
import torch

from test_gpu_parity import dev, rand_inputs  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [(1, 2 ** 16 + 1), (3, 1001)]
QK = [(64, 256, 16, 32), (33, 70, 5, 7)]


def odd(x):
    b = torch.empty(x.numel() + 1, dtype=x.dtype, device=x.device)
    b[1:] = x.flatten()
    return b[1:].view(x.shape)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("kind,lgD", [("fjl", 10), ("ffd", 12), ("ffd", 14), ("ffd", 17), ("ffd", 20), ("affd", 12),
                                      ("afjl", 9), ("afjl", 12), ("afjl", 17), ("qk", 0), ("afjlq", 12), ("qkh", 12),
                                      ("affdq", 12), ("afjlf", 12)])
def test_odd_starts(kind, lgD, dtype, dev):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    shapes = QK if kind == "qk" else SHAPES
    D = sum(s[2] * s[3] for s in shapes) if kind == "qk" else 1 << lgD
    s = Sketch(kind, shapes, D, 11, device=dev)
    for batch in (1, 3):
        xs = [x.to(dev) for x in rand_inputs(shapes, batch, 11, dtype=dtype)]
        assert torch.equal(s.apply(xs), s.apply([odd(x) for x in xs], out=odd(torch.zeros((batch, D), device=dev))))
        g = torch.Generator().manual_seed(12)
        z = torch.randn((batch, D), generator=g).to(dev)
        th = [torch.randn(n, generator=g).to(dev) for n in s.numels]
        ref = s.apply_T(z, out_dtype=dtype, theta0=th)
        outs = [odd(torch.zeros_like(r)) for r in ref]
        s.apply_T(odd(z), out_dtype=dtype, theta0=[odd(t) for t in th], outs=outs)
        assert all(torch.equal(o, r) for o, r in zip(outs, ref))
    s.close()
