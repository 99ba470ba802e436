"""What the autotuners keep: choices timed on other kernels are not taken over."""

import json
import re

import pytest

torch = pytest.importorskip("torch")

import paper_1501_04438_amd as gs


def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def other_builds(path, out, digest):
    """The entries of a cache file as another build would have left them."""
    entries = {re.sub(r"/src[0-9a-f]+", digest, k): v for k, v in json.loads(path.read_text()).items()}
    lines = ['  "%s": {"schedule": %d, "tiles_per_task": %d, "largest_first": %d, "grid": %d, "ms": %g}'
             % (k, v["schedule"], v["tiles_per_task"], v["largest_first"], v["grid"], v["ms"]) for k, v in entries.items()]
    out.write_text("{\n" + ",\n".join(lines) + "\n}\n")
    return entries


# "": a file of a build whose keys held no digest
@pytest.mark.gpu
@pytest.mark.parametrize("digest", ["", "/src0123456789ab"])
def test_plan_choice_of_other_kernels_is_timed_again(digest, tmp_path, monkeypatch):
    need_gpu()
    new, old = tmp_path / "new.json", tmp_path / "old.json"
    monkeypatch.setenv("GS_AUTOTUNE_CACHE", str(new))
    gs.Plan("coulomb3d", n=24, L=5.0, autotune=True)
    kept = other_builds(new, old, digest)
    monkeypatch.setenv("GS_AUTOTUNE_CACHE", str(old))
    plan = gs.Plan("coulomb3d", n=24, L=5.0, autotune=True)
    assert plan.info["tune_candidates"] > 0
    # the other build's entry stays in the file, beside the new one
    entries = json.loads(old.read_text())
    assert set(kept) < set(entries) and len(entries) == 2


@pytest.mark.gpu
def test_batch_choice_of_other_kernels_is_timed_again(tmp_path, monkeypatch):
    need_gpu()
    new, old = tmp_path / "new.json", tmp_path / "old.json"
    monkeypatch.setenv("GS_AUTOTUNE_CACHE", str(new))
    plans = [gs.Plan("coulomb3d", n=16, L=5.0) for _ in range(4)]
    x = [torch.ones((16,) * 3, dtype=torch.float64, device="cuda:0") for _ in plans]
    gs.Batch(plans, schedule="auto").eval(x)
    other_builds(new, old, "")
    monkeypatch.setenv("GS_AUTOTUNE_CACHE", str(old))
    b = gs.Batch(plans, schedule="auto")
    b.eval(x)
    assert b.info["candidates"] > 0


# cubes up to 64^3 run their middle passes in one launch, which takes no hints: the tuner leaves
# their bits alone (a slab plan runs them one by one and times them)
@pytest.mark.gpu
@pytest.mark.parametrize("n,planes", [(16, 0), (48, 0), (64, 0), (64, 33)])
def test_hints_that_no_launch_takes_are_not_timed(n, planes, tmp_path, monkeypatch):
    need_gpu()
    monkeypatch.setenv("GS_AUTOTUNE_CACHE", str(tmp_path / "tune.json"))
    start = gs.Plan("coulomb3d", n=n, L=5.0, slab_planes=planes).info["hint_bits"]
    tuned = gs.Plan("coulomb3d", n=n, L=5.0, slab_planes=planes, autotune=True).info
    assert tuned["tune_candidates"] == (5 if planes else 3)
    if not planes:
        assert (tuned["hint_bits"] ^ start) & 14 == 0


# the rounds of the persistent fused pass are tried where it is persistent, on unequal axes too
# (fused axis z: 128 plain; dipolar 128 on a grid inside the cache and z = 24 run one block per group)
@pytest.mark.gpu
@pytest.mark.parametrize("kernel,shape,rounds", [("coulomb3d", (128, 16, 32), 2), ("dipolar3d", (128, 16, 32), 0),
                                                 ("dipolar3d", (192, 16, 32), 2), ("coulomb3d", (24, 16, 32), 0)])
def test_rounds_are_timed_on_unequal_axes(kernel, shape, rounds, tmp_path, monkeypatch):
    need_gpu()
    monkeypatch.setenv("GS_AUTOTUNE_CACHE", str(tmp_path / "tune.json"))
    kw = {"dipole": ((0.6, 0.8, 0.0), (0.0, 0.6, 0.8))} if kernel == "dipolar3d" else {}
    x = torch.ones(shape, dtype=torch.float64, device="cuda:0")
    tuned = gs.Plan(kernel, n=shape, L=5.0, autotune=True, **kw)
    assert tuned.info["tune_candidates"] == 5 + rounds
    assert torch.equal(tuned.eval(x), gs.Plan(kernel, n=shape, L=5.0, **kw).eval(x))
