"""QK in bf16 with many layers per launch: every kernel of the first contraction (one to eight tiles of B, one to
four of A, and its wide form) and of the second mixed in one call, more layers than a launch takes, layers off the
tiling in between, second contractions divided into ranges (K > 1024), accumulated calls over a sub-range, a
workspace that holds a few layers, and one vector (fp64 sums), against the fp64 oracle.

Bound: B (or A) is carried to 16 mantissa bits and sums are fp32 over up to 2048 terms: 1e-4 as in the other bf16
matrix-core tests; one vector and layers off the tiling hold 1e-6."""
import pytest
import torch

import oracle as O
from test_gpu_parity import dev, oracle_in, rand_inputs, rel_err  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = ([(16, 128, 16, 16 * k) for k in range(1, 9)] + [(64, 256, 16 * k, 80) for k in range(1, 5)] +
          [(64, 512, 16, 16), (128, 1024, 32, 16), (33, 70, 5, 7), (2048, 128, 48, 16), (64, 2048, 32, 128)] +
          [(64, 256, 16, 32)] * 20)


@pytest.mark.parametrize("batch,ws_mb", [(1, None), (2, None), (5, None), (40, 16)])
def test_qk_bf16_groups(batch, ws_mb, dev, monkeypatch):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    if ws_mb is not None:
        monkeypatch.setenv("SK_WORKSPACE_MB", str(ws_mb))
    D, seed, f = sum(s[2] * s[3] for s in SHAPES), 23, 9
    s = Sketch("qk", SHAPES, D, seed, device=dev)
    xs = rand_inputs(SHAPES, batch, seed, dtype=torch.bfloat16)
    ref = O.apply("qk", SHAPES, D, seed, [oracle_in(x)[0] for x in xs], dtype="bf16")
    xd = [x.to(dev) for x in xs]
    y = s.apply(xd)
    tol = 1e-6 if batch == 1 else 1e-4
    assert rel_err(y.cpu().numpy(), ref) < tol
    s.apply(xd[f:], out=y, first_layer=f, accumulate=True)
    col = sum(t[2] * t[3] for t in SHAPES[:f])
    ref[:, col:] *= 2
    assert rel_err(y.cpu().numpy(), ref) < tol
    s.close()


# 4 x 4 tiles per block of the second contraction: divided, but whole with 256 and 480 to 512 blocks
@pytest.mark.parametrize("batch", [3, 255, 256, 257, 479, 480])
def test_qk_bf16_whole_blocks(batch, dev):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    shapes, seed = [(2048, 128, 64, 64)], 29
    s = Sketch("qk", shapes, 64 * 64, seed, device=dev)
    xs = rand_inputs(shapes, batch, seed, dtype=torch.bfloat16)
    ref = O.apply("qk", shapes, 64 * 64, seed, [oracle_in(x)[0] for x in xs], dtype="bf16")
    assert rel_err(s.apply([x.to(dev) for x in xs]).cpu().numpy(), ref) < 1e-4
    s.close()


# A workspace of two vectors: the last vector of a call of three is alone in its chunk and still sees B as two bf16
# terms.  With one entry every sum has one product, so that equal vectors agree bit for bit.
def test_qk_bf16_last_chunk(dev, monkeypatch):  # noqa: F811
    from paper_2402_03994_amd import Sketch
    monkeypatch.setenv("SK_WORKSPACE_MB", "16")
    shape = (16384, 128, 16, 128)
    s = Sketch("qk", [shape], 16 * 128, 33, device=dev)
    x = torch.zeros((3, 16384 * 128), dtype=torch.bfloat16, device=dev)
    x[:, 5 * 128 + 7] = 1.0
    y = s.apply([x])
    assert y.abs().max() > 0 and torch.equal(y[0], y[1]) and torch.equal(y[0], y[2])
    s.close()
