"""The persistent fused pass of grids whose axes differ, looping over pencil groups.

A launch holds at most four rounds of co-resident blocks; with more pencil groups than that
every block works several, reusing its LDS areas, twiddles and energy scratch.  The grids here
have more groups than four rounds at the most waves a SIMD can hold (256 CUs; 128-thread blocks at z =
128, 256 and 512: at most 8 per CU, their registers allow four waves per SIMD at most; one-wave blocks at
192 and 384: at most 12 per CU), against slab plans whose launches have fewer groups than
blocks: the same bits, per pencil and per energy sum."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1501_04438_amd as gs

DIPOLE = ((0.8, 0.4, -0.3), (0.3, 0.9, -0.1))
# (z, y, x), pencils per block, blocks per CU at most.  The dipolar kernel at z = 128 loops beyond 256 MB
# of X2 only
SHAPES = [((128, 256, 256), 4, 8), ((192, 128, 112), 2, 12), ((256, 96, 128), 2, 8), ((384, 96, 80), 1, 12),
          ((512, 64, 80), 1, 8)]


@pytest.mark.gpu
@pytest.mark.parametrize("kernel", ["coulomb3d", "dipolar3d"])
@pytest.mark.parametrize("shape,per_block,per_cu", SHAPES)
def test_looping_blocks_same_bits(kernel, shape, per_block, per_cu):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    z, y, x = shape
    groups = (x + 1) * 2 * y // per_block
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    planes = 4
    assert groups > 4 * per_cu * cus and planes * 2 * y // per_block < 4 * cus
    kw = {"dipole": DIPOLE} if kernel == "dipolar3d" else {}
    rho = torch.from_numpy(np.random.default_rng(z + y + x).standard_normal(shape)).to("cuda:0")
    plan = gs.Plan(kernel, n=shape, L=5.0, **kw)
    slabs = gs.Plan(kernel, n=shape, L=5.0, slab_planes=planes, **kw)
    assert torch.equal(plan.eval(rho), slabs.eval(rho))
    (e, g), (es, gslab) = plan.energy_and_gradient(rho), slabs.energy_and_gradient(rho)
    assert float(e) == float(es) and torch.equal(g, gslab)
