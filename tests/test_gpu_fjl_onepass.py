"""FJL layers of 2^14 <= N' <= 2^21 with D <= 2^13, forward and transposed, against
the fp64 oracle at the kinds' fp32 tolerance: the smallest and largest tile splits,
cells that several samples share (D = 2^13 of 2^14 positions), D below a workgroup,
ragged lengths, bf16, theta0, several layers."""
import pytest
import torch

import oracle as O
from test_gpu_qhaar import TOL, dev, rel_err, sketch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,D,batch", [
    ([16384], 8192, 2),
    ([16383, 8193], 4096, 3),
    ([40_001, 131_072], 4096, 1),
    ([262_145], 8192, 1),
    ([2 ** 21], 16, 2),
    ([2 ** 20 + 1], 128, 1),
])
@pytest.mark.parametrize("bf16", [False, True])
def test_fjl_onepass(ns, D, batch, bf16, dev):  # noqa: F811
    g = torch.Generator().manual_seed(D + batch)
    shapes = [(1, n) for n in ns]
    xs = [torch.randn((batch, n), generator=g).to(torch.bfloat16 if bf16 else torch.float32) for n in ns]
    s = sketch("fjl", shapes, D, 17, dev)
    y = s.apply([x.to(dev) for x in xs]).cpu().numpy()
    assert rel_err(y, O.apply("fjl", shapes, D, 17, [x.float().numpy() for x in xs])) < TOL
    z = torch.randn((batch, D), generator=g)
    th = [torch.randn(n, generator=g) if i == 0 else None for i, n in enumerate(ns)]
    outs = s.apply_T(z.to(dev), theta0=[None if t is None else t.to(dev) for t in th])
    refs = O.apply_T("fjl", shapes, D, 17, z.double().numpy(), theta0=[None if t is None else t.numpy() for t in th])
    for o, r in zip(outs, refs):
        assert rel_err(o.cpu().numpy(), r) < TOL
