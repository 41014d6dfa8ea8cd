"""The random-orthogonal contractions where K is divided over four or eight waves
(the rule's edge at K = 256, and K that leaves some waves short or empty), against
the fp64 oracle at the kind's fp32 tolerance; inputs at odd element offsets."""
import pytest
import torch

import oracle as O
from test_gpu_qhaar import TOL, dev, rel_err, sketch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,D,batch", [
    ("affdq", 301 * 1024 + 77, 4096, 3),  # K = 302 live rows: the last waves have less or none
    ("affdq", 255 * 1024 + 1, 2048, 1),   # K = 256 live rows, the last with one element
    ("affdq", 250 * 1024, 2048, 2),       # K = 250: four waves
    ("afjlq", 2 ** 19 - 3, 1 << 18, 2),   # K = 512 forward, 256 transposed
    ("qkh", 2 ** 18 - 1, 1 << 17, 2),     # K = 256 forward, 128 transposed
])
@pytest.mark.parametrize("bf16", [False, True])
def test_k_division(kind, n, D, batch, bf16, dev):  # noqa: F811
    g = torch.Generator().manual_seed(n)
    dt = torch.bfloat16 if bf16 else torch.float32
    buf = torch.randn(batch * n + 1, generator=g).to(dt)
    x = buf.to(dev)[1:].view(batch, n)  # first element at an odd offset
    s = sketch(kind, [(1, n)], D, 21, dev)
    xin = buf[1:].float().numpy().reshape(batch, n)
    y = s.apply([x]).cpu().numpy()
    assert rel_err(y, O.apply(kind, [(1, n)], D, 21, [xin])) < TOL
    z = torch.randn((batch, D), generator=g)
    out = s.apply_T(z.to(dev))[0].cpu().numpy()
    assert rel_err(out, O.apply_T(kind, [(1, n)], D, 21, z.double().numpy())[0]) < TOL


@pytest.mark.parametrize("kind,n,D,batch", [
    ("afjlq", 2 ** 19 - 3, 1 << 18, 9),   # 576 blocks of K = 512 and 1024: four waves
    ("affdq", 301 * 1024 + 77, 4096, 9),  # 720 blocks of the stacked rows, 144 to 288 of the others
    ("qkh", 2 ** 21 + 5, 1 << 16, 33),    # 528 blocks of K = 1024, three slabs
])
def test_more_blocks_than_two_per_cu(kind, n, D, batch, dev):  # noqa: F811
    g = torch.Generator().manual_seed(n)
    x = torch.randn((batch, n), generator=g)
    s = sketch(kind, [(1, n)], D, 22, dev)
    y = s.apply([x.to(dev)]).cpu().numpy()
    assert rel_err(y, O.apply(kind, [(1, n)], D, 22, [x.numpy()])) < TOL
    z = torch.randn((batch, D), generator=g)
    out = s.apply_T(z.to(dev))[0].cpu().numpy()
    assert rel_err(out, O.apply_T(kind, [(1, n)], D, 22, z.double().numpy())[0]) < TOL
