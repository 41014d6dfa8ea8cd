"""AFFD transposes of layer groups (rows of z, columns, output rows), and forwards of few vectors by the same passes
(and of three vectors, whose output pass shares the layers out): every tile width of the one-slab layers
(second digit of 2 to 512 values), one- and several-slab layers with the stored M tables, layers in between that
take the pass-based chain (no tables), more layers than one launch takes, odd sizes and bf16 outputs at odd
starts, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from test_gpu_parity import TOL_BF16, TOL_F32, dev, oracle_in, rand_inputs, rel_err  # noqa: F401

pytestmark = pytest.mark.gpu

# (D, shapes, flags, SK_WORKSPACE_MB)
CASES = [(2048, [(1, 3), (3, 1000), (1, 4099), (5, 3001), (33, 1023), (1, 100003)], 0, None),
         (16384, [(1, 768), (1, 16384), (3, 10001), (1, 2 ** 17 + 3), (1, 2 ** 19 - 5), (1, 2 ** 18 + 1)], 0, None),
         (4096, [(1, 2 ** 20 - 3), (1, 77), (1, 2 ** 20 + 5), (3, 2 ** 20 + 11), (1, 9 * 2 ** 20 + 5)], 0, None),
         (1 << 17, [(1, 2 ** 20 + 5), (1, 70001), (1, 2 ** 20)], 1, None),
         (1 << 20, [(1, 9), (1, 2 ** 21 + 7)], 0, None),
         (2048, [(1, 100 + 37 * i) for i in range(70)] + [(1, 2 ** 20 + 1)], 0, None),
         (65536, [(1, 2 ** 20 + 5), (1, 768), (1, 2 ** 21 + 9), (2, 2305)], 0, 22)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case,batch", [(i, b) for i in range(len(CASES)) for b in ((1, 3) if i != 4 else (1,))])
def test_affd_transpose_groups(case, batch, dtype, dev, monkeypatch):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    D, shapes, flags, ws_mb = CASES[case]
    if ws_mb is not None:  # one layer of three vectors in several chunks and groups
        monkeypatch.setenv("SK_WORKSPACE_MB", str(ws_mb))
    seed = 900 + case
    s = Sketch("affd", shapes, D, seed, device=dev, flags=flags)
    g = torch.Generator().manual_seed(seed)
    z = torch.randn((batch, D), generator=g)
    th = [torch.randn(r * c, generator=g) * 0.02 if i % 2 else None for i, (r, c) in enumerate(shapes)]
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    outs = s.apply_T(z.to(dev), out_dtype=tdt, theta0=[None if t is None else t.to(dev) for t in th])
    refs = O.apply_T("affd", shapes, D, seed, z.numpy().astype(np.float64),
                     theta0=[None if t is None else t.numpy() for t in th])
    for o, r in zip(outs, refs):
        assert rel_err(o.float().cpu().numpy(), r) < (TOL_BF16 if dtype == "bf16" else TOL_F32)
    s.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case,batch", [(i, b) for i in range(len(CASES)) for b in ((1, 2, 3) if i != 4 else (1,))])
def test_affd_few_vectors(case, batch, dtype, dev, monkeypatch):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    D, shapes, flags, ws_mb = CASES[case]
    if ws_mb is not None:
        monkeypatch.setenv("SK_WORKSPACE_MB", str(ws_mb))
    seed = 950 + case
    s = Sketch("affd", shapes, D, seed, device=dev, flags=flags)
    xs = rand_inputs(shapes, batch, seed, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
    ref = O.apply("affd", shapes, D, seed, [oracle_in(x)[0] for x in xs], dtype=dtype)
    xd = [x.to(dev) for x in xs]
    y = s.apply(xd)
    assert rel_err(y.cpu().numpy(), ref) < TOL_F32
    s.apply(xd, out=y, accumulate=True)
    assert rel_err(y.cpu().numpy(), 2 * ref) < TOL_F32
    s.close()


# Intermediates stay near the input's size: 2^112 times z and 2^108 times the vectors (the sum over several slabs adds
# their number) give as many times the results, bit for bit; four unnormalised transforms grow by sqrt(N' D), 2^11 to
# 2^20 here.
@pytest.mark.parametrize("D,shapes", [(16384, [(1, 2 ** 17 + 3), (1, 768), (1, 2 ** 19 - 5), (1, 3 * 2 ** 20 + 1)]),
                                      (1 << 17, [(1, 2 ** 19), (1, 2 ** 20 + 7)]), (2048, [(1, 3), (33, 1023)])])
def test_affd_large_values(D, shapes, dev):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    s = Sketch("affd", shapes, D, 27, device=dev)
    z = torch.randn((5, D), generator=torch.Generator().manual_seed(28)).to(dev)
    for a, b in zip(s.apply_T(z * 2.0 ** 112), s.apply_T(z)):
        assert torch.isfinite(b).all() and torch.equal(a, b * 2.0 ** 112)
    xs = [x.to(dev) for x in rand_inputs(shapes, 2, 29)]
    y = s.apply(xs)
    assert torch.isfinite(y).all() and torch.equal(s.apply([x * 2.0 ** 108 for x in xs]), y * 2.0 ** 108)
    s.close()


# Calls of 4 to 32 vectors: one-slab layers in the grouped passes first, then the several-slab layers and the small ones
# through their own, all in one output; 33 vectors leave the grouped passes.  The small workspace holds some of the
# layers' groups and few slots of G^T.
MIXED = [(1, 768), (33, 1023), (1, 2 ** 17 + 3), (1, 2 ** 19 - 5), (1, 2 ** 20 + 5), (3, 1000), (1, 3 * 2 ** 18 + 1), (1, 100)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D,batch,ws_mb", [(16384, 4, None), (16384, 8, 48), (4096, 32, None), (2048, 33, None),
                                           (65536, 8, None), (65536, 5, 40), (16384, 32, 96)])
def test_affd_mixed_paths(D, batch, ws_mb, dtype, dev, monkeypatch):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    if ws_mb is not None:
        monkeypatch.setenv("SK_WORKSPACE_MB", str(ws_mb))
    seed = 970 + batch
    s = Sketch("affd", MIXED, D, seed, device=dev)
    xs = rand_inputs(MIXED, batch, seed, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
    ref = O.apply("affd", MIXED, D, seed, [oracle_in(x)[0] for x in xs], dtype=dtype)
    xd = [x.to(dev) for x in xs]
    y = s.apply(xd)
    assert rel_err(y.cpu().numpy(), ref) < TOL_F32
    s.apply(xd, out=y, accumulate=True)
    assert rel_err(y.cpu().numpy(), 2 * ref) < TOL_F32
    s.close()


# One-slab column tiles over more vectors than 2048 workgroups take at once: a workgroup goes on to further vectors.
# 40 layers of 512 rows make 1280 tiles, each with all three vectors on one workgroup; 40 of 64 rows make 640 of the
# smaller tiles, eight vectors on three workgroups each.
@pytest.mark.parametrize("n,batch", [(2 ** 19 - 77, 3), (2 ** 16 - 5, 8)])
def test_affd_vector_turns(n, batch, dev):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    shapes, D, seed = [(1, n - 13 * i) for i in range(40)], 2048, 33
    s = Sketch("affd", shapes, D, seed, device=dev)
    xs = rand_inputs(shapes, batch, seed)
    y = s.apply([x.to(dev) for x in xs])
    assert rel_err(y.cpu().numpy(), O.apply("affd", shapes, D, seed, [x.numpy() for x in xs])) < TOL_F32
    z = torch.randn((batch, D), generator=torch.Generator().manual_seed(seed))
    outs = s.apply_T(z.to(dev))
    refs = O.apply_T("affd", shapes, D, seed, z.numpy().astype(np.float64))
    for o, r in zip(outs, refs):
        assert rel_err(o.cpu().numpy(), r) < TOL_F32
    s.close()


# Which calls of up to three vectors take the grouped passes: a lone layer of one slab up to D below 2^20 values, none of
# several, layers of seven slabs with two vectors and not with three, several-slab and small layers side by side.
@pytest.mark.parametrize("D,shapes,batches", [(16384, [(1, 2 ** 21 + 9)], (1, 3)), (1 << 19, [(1, 2 ** 20 - 7)], (1, 2)),
                                              (4096, [(1, 7 * 2 ** 20 - 3), (1, 6 * 2 ** 20 + 1)], (2, 3)),
                                              (1 << 20, [(1, 2 ** 20 - 7), (1, 9)], (1, 2, 3)),
                                              (16384, [(1, 2 ** 22 - 3), (1, 768), (1, 12 * 2 ** 20)], (3,))])
def test_affd_few_vectors_routes(D, shapes, batches, dev):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    s = Sketch("affd", shapes, D, 41, device=dev)
    for batch in batches:
        xs = rand_inputs(shapes, batch, 42)
        ref = O.apply("affd", shapes, D, 41, [x.numpy() for x in xs])
        y = s.apply([x.to(dev) for x in xs])
        assert rel_err(y.cpu().numpy(), ref) < TOL_F32
    s.close()
