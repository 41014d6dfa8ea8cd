"""AFJL forward with 128 to 1024 destination rows: one and several layer groups, ragged
layers, a layer with two fold items per destination row, accumulated and in chunks of a
small workspace, against the fp64 oracle."""
import pytest
import torch

import oracle as O
from test_gpu_parity import TOL_F32, dev, oracle_in, rand_inputs, rel_err  # noqa: F401

pytestmark = pytest.mark.gpu

LAYERS = [(1, 2), (1, 769), (33, 1024), (257, 1024), (3, 100001)]


@pytest.mark.parametrize("lgD,batch,ws_mb,layers", [
    (17, 1, None, LAYERS), (17, 2, None, LAYERS * 4), (17, 9, None, LAYERS), (17, 1, None, [(1, 2 ** 25 + 5)]),
    (18, 1, None, LAYERS * 4), (18, 5, 48, LAYERS), (18, 17, None, LAYERS),
    (19, 1, None, LAYERS), (19, 3, None, LAYERS * 2), (20, 1, None, LAYERS), (20, 9, None, LAYERS[2:]),
])
def test_afjl_tail_rows(lgD, batch, ws_mb, layers, dev, monkeypatch):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    if ws_mb is not None:
        monkeypatch.setenv("SK_WORKSPACE_MB", str(ws_mb))
    D, seed = 1 << lgD, 60 + lgD
    xs = rand_inputs(layers, batch, seed, dtype=torch.float32)
    ref = O.apply("afjl", layers, D, seed, [oracle_in(x)[0] for x in xs], dtype="f32")
    s = Sketch("afjl", layers, D, seed, device=dev)
    xd = [x.to(dev) for x in xs]
    assert rel_err(s.apply(xd).cpu().numpy(), ref) < TOL_F32
    if len(xd) > 2:
        y = s.apply(xd[:2])
        s.apply(xd[2:], out=y, first_layer=2, accumulate=True)
        assert rel_err(y.cpu().numpy(), ref) < TOL_F32
    s.close()
