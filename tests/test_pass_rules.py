"""The rules that choose a pass's form, read from the compiled sources by a host program."""

import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    cc = next((c for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")) if c and os.path.exists(c)), None)
    if cc is None:
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("rules") / "pass_rules_driver")
    r = subprocess.run([cc, "-x", "hip", "--cuda-host-only", "--offload-arch=gfx950", "-std=c++20", "-O1",
                        "-Wno-unused-command-line-argument", os.path.join(HERE, "native", "pass_rules_driver.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return [line.split() for line in r.stdout.splitlines()]


def test_fused_loop_of_unequal_axes(rules):
    """The persistent loop of the fused pass where it was measured to gain: at 128 the dipolar
    kernel loses two of its four waves per SIMD to it, so there it starts beyond the cache."""
    loop = {int(n): (p, d) for tag, n, p, d in (r for r in rules if r[0] == "loop_g")}
    assert loop[128] == ("always", "beyond_cache")
    assert loop[192] == loop[256] == ("always", "always")
    assert loop[384] == loop[512] == ("always", "never")
    assert all(v == ("never", "never") for n, v in loop.items() if n not in (128, 192, 256, 384, 512))
    at = {(int(r[1]), int(r[2]), r[3] == "1"): (r[4] == "1", r[5] == "1") for r in rules if r[0] == "persistent_g"}
    for mb, ev, en in ((38, False, False), (168, False, False), (202, False, True), (236, False, True), (269, True, True),
                       (538, True, True)):
        assert at[128, mb, False] == (True, ev) and at[128, mb, True] == (True, en)
    assert at[192, 38, False] == (True, True) and at[512, 538, False] == (True, False)
    assert at[224, 538, True] == (False, False)


def test_two_phase_inverse_at_24_values_is_checked(rules):
    """The two-phase x-inverse tile holds 24 values per thread at 1536 only; its unchecked form
    waits for every pair of loads there."""
    got = {int(r[1]): (r[2] == "1", r[3] == "1") for r in rules if r[0] == "p5_unchecked"}
    assert got[1536] == (False, False)
    assert all(unchecked for n, (_, unchecked) in got.items() if n != 1536)


def test_block_orders_are_permutations(rules):
    """The kernels' own block-to-tile orders, at every length, tile and row they are launched with."""
    got = [r for r in rules if r[0] == "orders"]
    assert len(got) == 6 * sum(r[0] == "runs" for r in rules) and all(r[3:] == ["1", "1", "1"] for r in got)


def test_runs_of_a_die(rules):
    """From 320 a die works a contiguous eighth of a row of tiles, at 256 two tiles, below only the
    tiles that share lines."""
    runs = {int(r[1]): (int(r[2]), int(r[3])) for r in rules if r[0] == "runs"}
    assert runs[320] == (5, 5) and runs[512] == (8, 8) and runs[256] == (2, 2) and runs[128] == (1, 1)


def test_only_kernels_that_are_launched():
    """Padding to B_3 transforms lengths 3 n / 2 at one tile per length; the fused pass's 3D groups of up
    to 8 pencils are always full (every length is a multiple of 4)."""
    lib = os.path.join(os.path.dirname(HERE), "paper_1501_04438_amd", "libgs.so")
    if not os.path.exists(lib):
        pytest.skip("library not built")
    with open(lib, "rb") as f:
        data = f.read()
    emb = {tuple(m) for m in re.findall(rb"k_x_(r2c|c2r)_emb(?:_split)?ILi(\d+)E", data)}
    assert emb and all(int(n) % 3 == 0 for _, n in emb)
    tiles = set(re.findall(rb"k_x_r2c_emb_splitILi(\d+)ELi[01]ELi(\d+)E", data))
    assert tiles and len(tiles) == len({n for n, _ in tiles})
    ragged = {int(n) for n in re.findall(rb"k_fused_gILi(\d+)ELi3ELi[01]ELi[01]ELb[01]ELb0E", data)}
    assert ragged and max(ragged) < 64
