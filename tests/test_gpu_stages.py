"""The stages of the general kernels against the oracle: every register radix
alone and in products, the primes on both sides of the largest register radix
(7 in FP64, 13 in FP32), single large primes, the longest transforms (both
register budgets) and coupled fields that leave no LDS for a prime's table.
Tolerances: those of the parity tests (a sum of 4096 terms, the longest of a
prime stage, rounds to about 0.3 eps sqrt(4096) = 1e-6 in FP32, 4e-15 in FP64)."""
import pytest

from gpu_util import TOL, case_input, gpu_solve, oracle_solve, rel_l2, rel_max

pytestmark = pytest.mark.gpu

LO = [0.0, -0.5, 1.0]
HI = [1.0, 1.3, 2.5]

# lengths along x: single radices, two and three stages, primes, prime products
LENGTHS = list(range(2, 18)) + [19, 22, 26, 29, 34, 49, 77, 91, 121, 143, 169, 180, 200, 240, 251, 256, 289, 323,
                                374, 506, 2047, 2048]
LONG = {"f32": [4095, 4096, 7680, 8143, 8189, 8190, 8191, 8192], "f64": [2049, 3840, 4088, 4092, 4093, 4095, 4096]}


def check(bc, grid, nc, kernel, diff, prec, ncomp, seed, inhom=False):
    nd = len(nc)
    print(f"stages {bc} {grid} {nc} {diff} {prec}", flush=True)
    f, faces = case_input(bc, grid, nc, ncomp, inhom, prec, seed=seed)
    got, gd = gpu_solve(bc, grid, nc, LO[:nd], HI[:nd], f, kernel, diff, prec, ncomp, faces)
    ref, rd = oracle_solve(bc, grid, nc, LO[:nd], HI[:nd], f, kernel, diff, faces)
    l2, mx = TOL[prec]
    assert len(gd) == len(rd)
    for name, g, r in [("psi", got, ref)] + [(f"deriv {a}", gd[a], rd[a]) for a in range(len(rd))]:
        assert rel_l2(g, r) <= l2 and rel_max(g, r) <= mx, (name, rel_l2(g, r), rel_max(g, r))


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", LENGTHS)
def test_stage_lengths(n, prec):
    # complex pencils (n along x) and half spectra (n along y)
    check("periodic", "staggered", [n, 21], "ps", "grad", prec, 1, seed=n)
    check("periodic", "staggered", [18, n], "fd2", "none", prec, 1, seed=n + 1)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", [6, 11, 13, 17, 23, 38, 46, 75, 99])
@pytest.mark.parametrize("bc,grid", [("dirichlet", "regular"), ("dirichlet", "staggered"), ("neumann", "regular"),
                                     ("neumann", "staggered")])
def test_stage_lengths_bounded(bc, grid, n, prec):
    # strided, contiguous and sandwich passes, pairs with an odd last pencil,
    # boundary terms added after the extension
    check(bc, grid, [n, 9, 14], "fd2", "none", prec, 1, seed=n, inhom=True)
    check(bc, grid, [7, 12, n], "ps", "none", prec, 1, seed=n + 1)


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_longest_transforms(prec):
    for n in LONG[prec]:
        check("periodic", "staggered", [n], "ps", "none", prec, 1, seed=n)


def test_coupled_fields_without_prime_table():
    # x pencils of 2557 (FP64) and 5113 (FP32), both prime: four resident tiles
    # fill LDS
    check("periodic", "staggered", [2557, 3, 4], "ps", "curl", "f64", 3, seed=7)
    check("periodic", "staggered", [5113, 3, 4], "ps", "curl", "f32", 3, seed=6)
