"""The forms a pass takes by size, where they change over, against the oracle and each other.

A pass is compiled in forms chosen by the grid (split halves, whole tiles or bounds-checked
ones, block-to-tile orders, one launch for the middle passes of a small grid, a persistent
fused pass).  All forms of a pass compute the same bits, so forms are compared bitwise; the
transforms themselves are compared with the oracle at the suite's 1e-12 (FFT rounding grows
like eps log2(2n): below 3e-15 of the maximum at these lengths).
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
import paper_1501_04438_amd as gs

TOL = 1e-12
D = ((0.8, 0.4, -0.3), (0.3, 0.9, -0.1))


def cuda(a):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda:0")


def relmax(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


# k_plane runs the middle passes of these grids; a plan whose workspace does not hold every
# plane (slab_planes below n + 1) and single steps run the three passes
@pytest.mark.gpu
@pytest.mark.parametrize("n", [8, 12, 16, 20, 24, 28, 32, 40, 48, 56, 64, 80])
@pytest.mark.parametrize("kernel", ["coulomb3d", "dipolar3d"])
def test_small_grid_forms_same_bits(kernel, n):
    kw = {"dipole": D} if kernel == "dipolar3d" else {}
    rho = cuda(np.random.default_rng(n).standard_normal((n, n, n)))
    plan = gs.Plan(kernel, n=n, L=4.0, **kw)
    slabs = gs.Plan(kernel, n=n, L=4.0, slab_planes=n // 2 + 1, **kw)
    u = plan.eval(rho)
    v = torch.empty_like(rho)
    for i in range(len(plan.steps())):
        plan.eval_step(rho, v, i)
    assert torch.equal(u, v)
    assert torch.equal(u, slabs.eval(rho))
    e, g = plan.energy_and_gradient(rho)
    es, g2 = slabs.energy_and_gradient(rho)
    assert float(e) == float(es) and torch.equal(g, g2)


# every transform length on both axes of a 2D grid: x passes as PN x 16, fused pass as 16 x PN
@pytest.mark.gpu
@pytest.mark.parametrize("n", [20, 28, 40, 56, 80, 96, 112, 160, 192, 224, 320, 384, 640, 768, 1536, 2048])
def test_lengths_on_either_axis(n):
    rng = np.random.default_rng(7 * n)
    for shape in ((n, 16), (16, n)):
        rho = rng.standard_normal(shape)
        plan = gs.Plan("coulomb2d", n=shape, L=5.0)
        ref = oracle.evaluate(oracle.make_plan("coulomb2d", 2, shape, 5.0), rho)
        assert relmax(plan.eval(cuda(rho)).cpu().numpy(), ref) <= TOL


# whole tiles (extents a multiple of the tiles) and ragged ones, split and persistent forms
@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(96, 32, 64), (32, 96, 24), (16, 64, 256), (12, 20, 192), (128, 12, 28), (20, 8, 512),
                                   (8, 384, 16), (320, 16, 8)])
@pytest.mark.parametrize("kernel", ["coulomb3d", "dipolar3d"])
def test_axes_that_differ(kernel, shape):
    kw = {"dipole": D} if kernel == "dipolar3d" else {}
    rho = np.random.default_rng(sum(shape)).standard_normal(shape)
    plan = gs.Plan(kernel, n=shape, L=5.0, **kw)
    ref = oracle.evaluate(oracle.make_plan(kernel, 3, shape, 5.0, **kw), rho)
    x = cuda(rho)
    u = plan.eval(x)
    assert relmax(u.cpu().numpy(), ref) <= TOL
    slabs = gs.Plan(kernel, n=shape, L=5.0, slab_planes=(shape[-1] + 2) // 2, **kw)
    e, g = plan.energy_and_gradient(x)
    es, gslab = slabs.energy_and_gradient(x)
    assert torch.equal(u, slabs.eval(x)) and float(e) == float(es) and torch.equal(g, gslab)


# the cache hints and the slab split (other block counts and orders) leave the bits alone, at
# lengths on both sides of the rules for the block order and the persistent grid
@pytest.mark.gpu
@pytest.mark.parametrize("n", [96, 112, 160, 256, 320, 384])
@pytest.mark.parametrize("kernel", ["coulomb3d", "dipolar3d"])
def test_orders_and_hints_same_bits(kernel, n):
    kw = {"dipole": D} if kernel == "dipolar3d" else {}
    rho = cuda(np.random.default_rng(n).standard_normal((n, n, n)))
    plan = gs.Plan(kernel, n=n, L=4.0, **kw)
    other = gs.Plan(kernel, n=n, L=4.0, slab_planes=n // 3, hint_bits=(27 if n <= 160 else 0), **kw)
    assert torch.equal(plan.eval(rho), other.eval(rho))
    (e, g), (e2, g2) = plan.energy_and_gradient(rho), other.energy_and_gradient(rho)
    assert float(e) == float(e2) and torch.equal(g, g2)


def die_tile(b, nb, run):
    """The block-to-tile order of the kernels: nb tiles in groups of 8 runs, block b on die b % 8."""
    if run == 1 or b >= nb // (8 * run) * (8 * run):
        return b
    return (b // (8 * run) * 8 + b % 8) * run + (b // 8) % run


@pytest.mark.parametrize("run", [1, 2, 4, 5, 16])
@pytest.mark.parametrize("nb", [1, 7, 16, 17, 40, 64, 129, 321])
def test_block_order_is_a_permutation(nb, run):
    assert sorted(die_tile(b, nb, run) for b in range(nb)) == list(range(nb))
