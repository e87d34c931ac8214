"""Batched plans as one launch per pass level: batches that mix every transform
length of the wavefront tile bodies, one problem alone, and general lengths
(primes, mixed registers) against single plans bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BATCHES = {
    "one": [(64, 96, 128)],
    "all_lengths": [(32, 48, 64), (96, 128, 32), (48, 32, 96), (128, 64, 48), (64, 96, 128), (32, 32, 32)],
    "general": [(30, 17, 23), (9, 40, 64), (32, 48, 50), (97, 8, 12)],
}


@pytest.mark.parametrize("bc,grid,kernel", [("neumann", "staggered", "ps"), ("neumann", "regular", "fd2"),
                                            ("dirichlet", "staggered", "fd2")])
@pytest.mark.parametrize("name", list(BATCHES))
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_levels_equal_single_plans(bc, grid, kernel, name, prec):
    import torch
    from paper_2301_01145_amd import Solver
    from paper_2301_01145_amd.batched import BatchedSolver
    dtype = torch.float32 if prec == "f32" else torch.float64
    # REGULAR Neumann: lengths 2 (n - 1) of n = N_c + 1 nodes are those of N_c cells
    shapes = BATCHES[name]
    rng = np.random.default_rng(31)
    bs = BatchedSolver(bc, grid, [{"nc": list(s)} for s in shapes], kernel=kernel, dtype=dtype)
    fs = [torch.as_tensor(rng.normal(size=bs.in_shapes[i]), dtype=dtype, device="cuda") for i in range(len(shapes))]
    psis = bs.bind(fs)
    for _ in range(2):
        bs.run()
    torch.cuda.synchronize()
    assert bs.error_flag() == 0
    for i, s in enumerate(shapes):
        one = BatchedSolver(bc, grid, [{"nc": list(s)}], kernel=kernel, dtype=dtype)
        ref = one.bind([fs[i]])
        one.run()
        single = Solver(bc, grid, list(s), kernel=kernel, dtype=dtype)
        psi, _ = single.solve(fs[i])
        torch.cuda.synchronize()
        # alone or beside others: the same tiles; the single plan's kernels may
        # differ (wavefront or general per axis), so to rounding
        if one.kernel_mode() == bs.kernel_mode():
            assert torch.equal(ref[0], psis[i]), (i, s)
        err = float((psi[0] - psis[i]).double().norm() / psi[0].double().norm())
        assert err <= (1e-5 if prec == "f32" else 1e-12), (i, s, err)
        single.close()
        one.close()
    bs.close()
