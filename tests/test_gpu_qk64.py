"""QK contractions with fp64 sums (fp32 inputs, bf16 inputs off the bf16 matrix-core tiling, transposes) at the
edges of their tiles, against the fp64 oracle.

Bound: a result is an fp64 sum of products of fp32 values, rounded to fp32, over an intermediate rounded to fp32,
with factors within a few fp32 ulp of the oracle's: 1e-6 of max(|o|, rms) leaves a factor of about four."""
import numpy as np
import pytest
import torch

import oracle as O
from test_gpu_parity import dev, oracle_in, rand_inputs, rel_err  # noqa: F401

pytestmark = pytest.mark.gpu
TOL = 1e-6
TOL_BF16 = 2.0 ** -8  # one rounding to bf16 of the transpose's outputs (2^-9 of the value), and its edges

# (rows, cols, dA, dB): both orders, one to five 16-row tiles, ends of 16 and 64 in every index, single rows,
# columns and blocks, contractions longer than one k range (1024) in both orders
SHAPES = {
    "tiny": [(1, 1, 1, 1), (1, 300, 1, 9), (300, 1, 9, 1), (2, 3, 2, 3), (15, 17, 15, 17)],
    "tiles": [(16, 16, 16, 16), (64, 64, 17, 33), (65, 63, 33, 16), (48, 68, 31, 5), (130, 70, 64, 48)],
    "wide": [(96, 2051, 8, 40), (2051, 96, 40, 8), (33, 1029, 3, 12), (1029, 130, 70, 3)],
    "many": [(5 + i % 7, 9 + i % 5, 1 + i % 5, 1 + i % 9) for i in range(70)],
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name,batch,ws_mb", [(n, b, None) for n in SHAPES for b in (1, 3)] + [("wide", 40, 16)])
def test_qk_fp64_sums(name, batch, ws_mb, dtype, dev, monkeypatch):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    if ws_mb is not None:  # fewer k ranges than wanted, several vector chunks
        monkeypatch.setenv("SK_WORKSPACE_MB", str(ws_mb))
    shapes = SHAPES[name]
    D, seed = sum(s[2] * s[3] for s in shapes), 5
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    s = Sketch("qk", shapes, D, seed, device=dev)
    xs = rand_inputs(shapes, batch, seed, dtype=tdt)
    ref = O.apply("qk", shapes, D, seed, [oracle_in(x)[0] for x in xs], dtype=dtype)
    xd = [x.to(dev) for x in xs]
    y = s.apply(xd)
    assert rel_err(y.cpu().numpy(), ref) < TOL
    s.apply(xd, out=y, accumulate=True)
    assert rel_err(y.cpu().numpy(), 2 * ref) < TOL
    g = torch.Generator().manual_seed(seed)
    z = torch.randn((batch, D), generator=g)
    th = [torch.randn(r * c, generator=g) * 0.02 if i % 2 else None for i, (r, c, _, _) in enumerate(shapes)]
    outs = s.apply_T(z.to(dev), out_dtype=tdt, theta0=[None if t is None else t.to(dev) for t in th])
    refs = O.apply_T("qk", shapes, D, seed, z.numpy().astype(np.float64),
                     theta0=[None if t is None else t.numpy() for t in th])
    for o, r in zip(outs, refs):
        assert rel_err(o.float().cpu().numpy(), r) < (TOL_BF16 if dtype == "bf16" else TOL)
    s.close()


# One-row matrices of many vectors: every vector is the first one times a power of two
def test_qk_thin_transpose(dev):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    shapes, batch, seed = [(1, 2 ** 19, 1, 1)] * 9, 256, 6
    s = Sketch("qk", shapes, 9, seed, device=dev)
    g = torch.Generator().manual_seed(seed)
    z0 = torch.randn((1, 9), generator=g)
    p2 = 2.0 ** (torch.arange(batch) % 7)
    outs = s.apply_T((z0 * p2[:, None]).contiguous().to(dev))
    refs = O.apply_T("qk", shapes, 9, seed, z0.numpy().astype(np.float64))
    for o, r in zip(outs, refs):
        assert rel_err(o[:1].cpu().numpy(), r) < TOL
        assert torch.equal(o, o[:1] * p2.to(dev)[:, None])
    s.close()


# More workgroups of 32 rows than one launch takes (8 layers to a group: 33 million), forward
def test_qk_many_workgroups(dev):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    shapes, batch, seed = [(2 ** 19, 4, 4, 1)] * 9, 256, 6
    s = Sketch("qk", shapes, 36, seed, device=dev)
    x0 = rand_inputs(shapes[:1], 1, seed, dtype=torch.bfloat16)[0]
    p2 = (2.0 ** (torch.arange(batch) % 7)).to(dev)
    x = x0.to(dev) * p2.to(torch.bfloat16)[:, None]
    y = s.apply([x] * 9)
    ref = O.apply("qk", shapes, 36, seed, [oracle_in(x0)[0]] * 9, dtype="bf16")
    assert rel_err(y[:1].cpu().numpy(), ref) < TOL
    assert torch.equal(y, y[:1] * p2[:, None])
    s.close()


# Transposes with thin outputs (a thread per output) beside layers on the matrix cores: one and few rows and columns,
# short and long sums, one vector and groups of four with a rest
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("batch", [1, 4, 7])
def test_qk_thin_outputs(batch, dtype, dev):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    shapes = [(1, 4099, 1, 64), (4099, 1, 64, 1), (96, 130, 40, 33), (3, 1027, 2, 20), (1027, 5, 33, 3), (12, 700, 4, 64),
              (700, 24, 8, 4), (257, 255, 3, 3), (160, 192, 48, 64)]
    D, seed = sum(s[2] * s[3] for s in shapes), 8
    s = Sketch("qk", shapes, D, seed, device=dev)
    g = torch.Generator().manual_seed(seed)
    z = torch.randn((batch, D), generator=g)
    th = [torch.randn(r * c, generator=g) * 0.02 if i % 2 else None for i, (r, c, _, _) in enumerate(shapes)]
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    outs = s.apply_T(z.to(dev), out_dtype=tdt, theta0=[None if t is None else t.to(dev) for t in th])
    refs = O.apply_T("qk", shapes, D, seed, z.numpy().astype(np.float64),
                     theta0=[None if t is None else t.numpy() for t in th])
    for o, r in zip(outs, refs):
        assert rel_err(o.float().cpu().numpy(), r) < (TOL_BF16 if dtype == "bf16" else TOL)
    s.close()
