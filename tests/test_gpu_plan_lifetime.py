"""Plans made and closed one after the other: every device buffer of a plan is freed once.

Axes of equal length share one twiddle table, so which tables a plan owns depends on the
pattern of equal axes; a table freed twice leaves an error that the next plan's creation
reports."""

import itertools

import pytest

torch = pytest.importorskip("torch")

import paper_1501_04438_amd as gs


@pytest.mark.gpu
@pytest.mark.parametrize("shape", sorted(set(itertools.product((8, 16), repeat=3)) | set(itertools.permutations((8, 12, 16)))))
def test_close_and_make_again(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = torch.ones(shape, dtype=torch.float64, device="cuda:0")
    first = gs.Plan("coulomb3d", n=shape, L=4.0)
    u = first.eval(x)
    first.close()
    again = gs.Plan("coulomb3d", n=shape, L=4.0)
    assert torch.equal(again.eval(x), u)
    again.close()


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(16, 16), (8, 16), (16, 8)])
def test_close_and_make_again_2d(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = torch.ones(shape, dtype=torch.float64, device="cuda:0")
    first = gs.Plan("coulomb2d", n=shape, L=4.0)
    u = first.eval(x)
    first.close()
    again = gs.Plan("coulomb2d", n=shape, L=4.0)
    assert torch.equal(again.eval(x), u)
    again.close()
