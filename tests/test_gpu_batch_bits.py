"""A batch has the bits of its problems' single plans where both run the same tile
bodies: FP32 lengths of the wavefront kernels (kernel mode 1), and general
lengths in either precision (mode 0).  The mode of every batch is checked."""
import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu

WAVE = [[32, 48, 64], [64, 32, 128], [96, 64, 48], [128, 96, 32]]
WAVE_REGULAR = [[32, 64, 128], [128, 32, 64], [96, 48, 32]]
GENERAL = [[20, 33, 17], [40, 24, 50], [7, 81, 26], [60, 12, 37]]


@pytest.mark.parametrize("bc,grid,prec,sizes,mode", [
    ("neumann", "staggered", "f32", WAVE, 1), ("dirichlet", "staggered", "f32", WAVE, 1),
    ("neumann", "regular", "f32", WAVE_REGULAR, 1), ("neumann", "staggered", "f32", GENERAL, 0),
    ("dirichlet", "staggered", "f64", GENERAL, 0), ("neumann", "regular", "f64", GENERAL, 0)])
def test_batch_has_the_bits_of_single_plans(bc, grid, prec, sizes, mode):
    import torch
    from paper_2301_01145_amd import Solver
    from paper_2301_01145_amd.batched import BatchedSolver
    dtype = torch.float32 if prec == "f32" else torch.float64
    b = BatchedSolver(bc, grid, [{"nc": nc} for nc in sizes], kernel="fd2", dtype=dtype)
    assert b.kernel_mode() == mode
    rng = np.random.default_rng(41)
    fs = [to_dev(rng.normal(size=s).astype(np.float32), dtype, torch) for s in b.in_shapes]
    psis = b.bind(fs)
    b.run()
    torch.cuda.synchronize()
    for nc, f, p in zip(sizes, fs, psis):
        s = Solver(bc, grid, nc, kernel="fd2", dtype=dtype)
        ref, _ = s.solve(f)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(ref[0]).all()) and torch.equal(p, ref[0]), (nc, float((p - ref[0]).abs().max()))
        s.close()
