"""The persistent form of the strided bounded passes (a workgroup walks several
tiles, the next one's loads in flight during the transform): HP_PERSIST caps its
workgroups so that small problems take it, against one workgroup a tile
(HP_PERSIST=0), bit for bit.  Tiles at the end of a row of tiles that are partly
filled, rows off the cache lines (tiles in XCD order), one-way passes and
sandwiches of every family of types."""
import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu

CASES = [("dirichlet", "staggered", [64, 64, 96]), ("neumann", "staggered", [128, 64, 64]),
         ("dirichlet", "regular", [64, 64, 64]), ("neumann", "regular", [64, 128, 32]),
         ("neumann", "regular", [256, 32, 64]), (["dirichlet", "neumann", "periodic"], "staggered", [64, 256, 37]),
         (["periodic", "dirichlet", "periodic"], "staggered", [64, 32, 75]),
         (["neumann", "periodic", "dirichlet"], "regular", [32, 128, 64])]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("bc,grid,nc", CASES)
def test_persistent_equals_plain(bc, grid, nc, prec, monkeypatch):
    import torch
    from paper_2301_01145_amd import Solver
    print(f"persistent {bc} {grid} {nc} {prec}", flush=True)
    dtype = torch.float32 if prec == "f32" else torch.float64
    s = Solver(bc, grid, nc, kernel="fd2", dtype=dtype)
    f = to_dev(np.random.default_rng(11).normal(size=s.in_shape).astype(np.float32), dtype, torch)
    out = []
    for cap in ("0", "3", "7"):
        monkeypatch.setenv("HP_PERSIST", cap)
        psi = torch.full(s.out_shape, float("nan"), dtype=dtype, device="cuda")
        s.solve(f, psi=psi)
        torch.cuda.synchronize()
        out.append(psi.cpu().numpy())
    s.close()
    assert np.all(np.isfinite(out[0]))
    assert np.array_equal(out[1], out[0]) and np.array_equal(out[2], out[0])
