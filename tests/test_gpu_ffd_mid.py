"""FFD with 2^14 <= D <= 2^19 (row and column passes): every column-tile width, one to nine blocks (places on the
XCDs beyond a multiple of 8), ragged ends of rows and blocks, several layers added into one output, one to five
vectors in fp32 and bf16 at odd starts, theta0, and a small workspace (chunks of vectors), against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from test_gpu_parity import TOL_BF16, TOL_F32, dev, oracle_in, rand_inputs, rel_err  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [(14, [(1, 9 * 2 ** 14 - 5), (1, 3)], 3, None), (15, [(1, 2 ** 15 + 1), (3, 5001)], 1, None),
         (16, [(1, 5 * 2 ** 16 + 1025)], 5, None), (16, [(1, 8 * 2 ** 16)], 1, None),
         (17, [(1, 2 ** 17 - 1023)], 2, None), (18, [(1, 2 ** 18 + 1024), (1, 7)], 1, None),
         (19, [(1, 2 ** 19 + 2 ** 18 + 3)], 2, None), (16, [(1, 17 * 2 ** 16 + 3)], 5, 24)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_ffd_mid(case, dtype, dev, monkeypatch):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    lgD, shapes, batch, ws_mb = CASES[case]
    if ws_mb is not None:
        monkeypatch.setenv("SK_WORKSPACE_MB", str(ws_mb))
    D, seed = 1 << lgD, 700 + case
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    s = Sketch("ffd", shapes, D, seed, device=dev)
    xs = rand_inputs(shapes, batch, seed, dtype=tdt)
    ref = O.apply("ffd", shapes, D, seed, [oracle_in(x)[0] for x in xs], dtype=dtype)
    xd = [x.to(dev) for x in xs]
    y = s.apply(xd)
    assert rel_err(y.cpu().numpy(), ref) < TOL_F32
    s.apply(xd, out=y, accumulate=True)
    assert rel_err(y.cpu().numpy(), 2 * ref) < TOL_F32
    g = torch.Generator().manual_seed(seed)
    z = torch.randn((batch, D), generator=g)
    th = [torch.randn(r * c, generator=g) * 0.02 if i % 2 == 0 else None for i, (r, c) in enumerate(shapes)]
    outs = s.apply_T(z.to(dev), out_dtype=tdt, theta0=[None if t is None else t.to(dev) for t in th])
    refs = O.apply_T("ffd", shapes, D, seed, z.numpy().astype(np.float64),
                     theta0=[None if t is None else t.numpy() for t in th])
    for o, r in zip(outs, refs):
        assert rel_err(o.float().cpu().numpy(), r) < (TOL_BF16 if dtype == "bf16" else TOL_F32)
    s.close()


def parity(lgD, shapes, batch, seed, dtype, dev):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    D = 1 << lgD
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    s = Sketch("ffd", shapes, D, seed, device=dev)
    xs = rand_inputs(shapes, batch, seed, dtype=tdt)
    ref = O.apply("ffd", shapes, D, seed, [oracle_in(x)[0] for x in xs], dtype=dtype)
    assert rel_err(s.apply([x.to(dev) for x in xs]).cpu().numpy(), ref) < TOL_F32
    g = torch.Generator().manual_seed(seed)
    z = torch.randn((batch, D), generator=g)
    outs = s.apply_T(z.to(dev), out_dtype=tdt)
    refs = O.apply_T("ffd", shapes, D, seed, z.numpy().astype(np.float64))
    for o, r in zip(outs, refs):
        assert rel_err(o.float().cpu().numpy(), r) < (TOL_BF16 if dtype == "bf16" else TOL_F32)
    s.close()


# blocks beyond the last eight, with 2^19 values per block and call or more: none to seven of them
@pytest.mark.parametrize("lgD,blocks,batch", [(19, 1, 1), (18, 2, 3), (17, 9, 4), (15, 12, 16), (17, 5, 5), (16, 15, 8)])
def test_ffd_mid_few_blocks(lgD, blocks, batch, dev):  # noqa: F811
    parity(lgD, [(1, (blocks << lgD) - 1021)], batch, 800 + lgD + blocks, "f32", dev)


# No intermediate may overflow where inputs and results are far from the end of the type: 2^112 times the vectors gives
# 2^112 times the results, bit for bit (an unnormalised pair of transforms grows by D).
@pytest.mark.parametrize("lgD", [14, 16, 17, 19])
def test_ffd_mid_large_values(lgD, dev):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    D = 1 << lgD
    s = Sketch("ffd", [(1, 2 * D - 3)], D, 19, device=dev)
    x = rand_inputs([(1, 2 * D - 3)], 2, 19)[0].to(dev)
    y = s.apply([x])
    assert torch.isfinite(y).all() and torch.equal(s.apply([x * 2.0 ** 112]), y * 2.0 ** 112)
    z = torch.randn((2, D), generator=torch.Generator().manual_seed(20)).to(dev)
    o = s.apply_T(z)[0]
    assert torch.isfinite(o).all() and torch.equal(s.apply_T(z * 2.0 ** 112)[0], o * 2.0 ** 112)
    s.close()


# More blocks than workgroups are wanted for: a workgroup goes on to a second and third vector (every gridDim.y-th), in
# the row, column and output passes, the column tiles of 2^13 and 2^14 values, whole blocks and a ragged last one
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("lgD,blocks,batch", [(14, 1025, 3), (16, 137, 4), (19, 17, 5)])
def test_ffd_mid_vector_turns(lgD, blocks, batch, dtype, dev):  # noqa: F811
    # row passes 2064, 1152 and 1088 workgroups per vector, column passes 2064, 1152 and 544, of 2048 in all
    parity(lgD, [(1, (blocks << lgD) - 4099)], batch, 900 + lgD, dtype, dev)
