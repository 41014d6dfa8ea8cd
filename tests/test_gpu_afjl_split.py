"""AFJL: the transpose's column and output kernels (D >= 1024: every number of destination rows, register and pass
columns, one, a few and more than eight vectors); and forward calls whose fold items are split over several workgroups (small calls), and rows that start at any
element (odd sizes in fp32 and bf16): against the fp64 oracle, one to 33 vectors, accumulated and in chunks of a
small workspace."""
import numpy as np
import pytest
import torch

import oracle as O
from test_gpu_parity import TOL_BF16, TOL_F32, dev, oracle_in, rand_inputs, rel_err  # noqa: F401

pytestmark = pytest.mark.gpu

# D = 256 (Lw < 1024), 1024 (one destination row), 4096 (R = 4) and 65536 (R = 64, two threads per column);
# items of one row, of a full 256 and a 257th, and layers that pad to N' = D
LAYERS = [(1, 2), (1, 769), (33, 1024), (257, 1024), (3, 100001)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D,batch,ws_mb", [(256, 1, None), (256, 3, None), (1024, 1, None), (1024, 9, None),
                                           (4096, 1, None), (4096, 2, None), (4096, 33, None), (8192, 8, 16),
                                           (65536, 1, None), (65536, 5, 16)])
def test_afjl_split_items(D, batch, ws_mb, dtype, dev, monkeypatch):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    if ws_mb is not None:
        monkeypatch.setenv("SK_WORKSPACE_MB", str(ws_mb))
    seed = 17
    xs = rand_inputs(LAYERS, batch, seed, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
    ref = O.apply("afjl", LAYERS, D, seed, [oracle_in(x)[0] for x in xs], dtype=dtype)
    s = Sketch("afjl", LAYERS, D, seed, device=dev)
    xd = [x.to(dev) for x in xs]
    y = s.apply(xd)
    assert rel_err(y.cpu().numpy(), ref) < TOL_F32
    y2 = s.apply(xd[:2])
    s.apply(xd[2:], out=y2, first_layer=2, accumulate=True)
    assert rel_err(y2.cpu().numpy(), ref) < TOL_F32
    s.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("lgD,batch", [(10, 1), (10, 3), (11, 1), (12, 9), (13, 2), (14, 1), (15, 10), (16, 1), (16, 3),
                                       (17, 1), (18, 2), (20, 1)])
def test_afjl_transpose_rows(lgD, batch, dtype, dev):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    D, seed = 1 << lgD, 40 + lgD
    s = Sketch("afjl", LAYERS, D, seed, device=dev)
    g = torch.Generator().manual_seed(seed)
    z = torch.randn((batch, D), generator=g)
    th = [torch.randn(r * c, generator=g) * 0.02 if i % 2 else None for i, (r, c) in enumerate(LAYERS)]
    outs = s.apply_T(z.to(dev), out_dtype=torch.bfloat16 if dtype == "bf16" else torch.float32,
                     theta0=[None if t is None else t.to(dev) for t in th])
    refs = O.apply_T("afjl", LAYERS, D, seed, z.numpy().astype(np.float64),
                     theta0=[None if t is None else t.numpy() for t in th])
    for o, r in zip(outs, refs):
        assert rel_err(o.float().cpu().numpy(), r) < (TOL_BF16 if dtype == "bf16" else TOL_F32)
    s.close()


# shares of items with 16 rows or more for every R up to 64 (one item per destination row, several layers and one, so
# that the tail shares them out too), beside layers of one live row and of a part of a destination row's rows
@pytest.mark.parametrize("lgD,batch", [(11, 1), (13, 3), (14, 1), (14, 9), (15, 1), (15, 2), (16, 1), (16, 3)])
@pytest.mark.parametrize("layers", [[(1, 2 ** 21 + 5)], [(1, 2), (1025, 1025), (3, 2 ** 20 + 7), (1, 769)]])
def test_afjl_split_shares(lgD, batch, layers, dev):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    D, seed = 1 << lgD, 70 + lgD
    xs = rand_inputs(layers, batch, seed, dtype=torch.float32)
    ref = O.apply("afjl", layers, D, seed, [oracle_in(x)[0] for x in xs], dtype="f32")
    s = Sketch("afjl", layers, D, seed, device=dev)
    y = s.apply([x.to(dev) for x in xs])
    assert rel_err(y.cpu().numpy(), ref) < TOL_F32
    s.close()
