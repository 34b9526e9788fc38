"""CPU tests of the axis passes' host side: the tables, tiles and plane groups
(walked as the kernel walks them, under the sanitizers), which plans take the
passes, and what a device memory bound does to them. No GPU."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

import paper_2406_05577_amd as pk
import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_pass_addresses_under_sanitizers(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = tmp_path / "pass_check"
    csrc = os.path.join(ROOT, "paper_2406_05577_amd", "csrc")
    subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=undefined",
                    os.path.join(ROOT, "tests", "native", "pass_check.cpp"),
                    os.path.join(csrc, "plan.cpp"), os.path.join(csrc, "pass_plan.cpp"),
                    "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stderr
    assert "pass_check OK" in res.stdout


def _log(capfd, dims, nb, dtype="c128", flags=0, tuning=None):
    m, lin = synth.sphere_map(dims, [0.25 * d for d in dims], (0.1, 0.2, -0.3))
    p = pk.Plan(dims, [lin], nb, dtype=dtype, flags=flags | pk.PLAN_HOST_ONLY, tuning=tuning)
    return p, capfd.readouterr().err


def test_which_plans_take_passes(monkeypatch, capfd):
    """Passes: no tiling request, and no band-inner x lines, the forward, or an
    inverse whose class pairs have no whole work; every other direction keeps the
    class-split kernels."""
    monkeypatch.setenv("FFTB_LOG", "1")
    for dtype in ("c128", "c64"):
        p, log = _log(capfd, (60, 50, 45), 7, dtype)
        assert log.count("axis passes") == 2
        p, log = _log(capfd, (60, 50, 45), 7, dtype, tuning=dict(path=1))
        assert "axis passes" not in log and p.info["tuning"]["inv"]["path"] == 1
        p, log = _log(capfd, (60, 50, 45), 7, dtype, tuning=dict(inv_band_chunk=4))
        assert log.count("inverse: axis passes") == 0 and log.count("forward: axis passes") == 1
        # lines longer than any split, and band-inner shapes
        _, log = _log(capfd, (6, 4, 540), 3, dtype)
        assert "axis passes" not in log
        # band-inner shapes: the forward, and the inverse unless its class pairs fill
        # their band chunks (8 bands, complex64 16) and the rounds of 256 tasks
        for dims, nb, pairs in (((96, 96, 96), 64, True), ((96, 96, 96), 63, False),
                                ((96, 96, 96), 72, dtype == "c128"), ((32, 32, 32), 8, False),
                                ((96, 96, 96), 16, False), ((96, 144, 96), 64, False),
                                ((128, 128, 128), 64, True), ((144, 160, 180), 128, False),
                                ((144, 160, 180), 16, dtype == "c128"), ((96, 96, 160), 64, dtype == "c128")):
            p, log = _log(capfd, dims, nb, dtype)
            assert p.info["tuning"]["inv"]["path"] == 3 and "forward: axis passes" in log
            assert ("inverse: axis passes" not in log) == pairs, (dims, nb)
        _, log = _log(capfd, (96, 96, 96), 7, dtype, tuning=dict(path=3))
        assert "axis passes" not in log


def test_pass_scratch_under_a_bound(monkeypatch, capfd):
    """Under FFTB_MAX_DEVICE_BYTES the passes take no more scratch than the
    class-split kernels did, in more groups of planes."""
    monkeypatch.setenv("FFTB_LOG", "1")
    _, log = _log(capfd, (60, 50, 45), 16)
    assert "inverse: axis passes, 1 groups of 45 planes" in log
    monkeypatch.setenv("FFTB_MAX_DEVICE_BYTES", str(1 << 30))
    _, log = _log(capfd, (60, 50, 45), 16)
    groups = int(re.search(r"inverse: axis passes, (\d+) groups", log).group(1))
    assert groups > 1
    scratch = float(re.search(r"scratch ([0-9.]+) GB", log).group(1))
    _, log = _log(capfd, (60, 50, 45), 16, tuning=dict(path=1))
    assert scratch <= float(re.search(r"scratch ([0-9.]+) GB", log).group(1))


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_plane_kernel_plans_hold_no_slab_scratch(dtype, monkeypatch, capfd):
    """Planes in one launch live in LDS: their plans hold the columns alone, are
    in no plane groups and on no second stream, and a device memory bound that
    leaves no room for a slab plane does not keep them from the passes."""
    monkeypatch.setenv("FFTB_LOG", "1")
    nb = 16
    p, log = _log(capfd, (60, 54, 50), nb, "c64")
    assert "planes in one launch" in log and "groups of" not in log and "streams" not in log
    columns = p.info["total_columns"] * nb * 50 * 8
    assert float(re.search(r"scratch ([0-9.]+) GB", log).group(1)) <= (columns + 50 * 128) / 1e9 + 5e-4
    # few columns over many slabs: a slab plane is larger than the columns
    monkeypatch.setenv("FFTB_MAX_DEVICE_BYTES", str(1 << 30))
    lin = np.array([x + 60 * (x % 3) for x in range(0, 60, 2)], dtype=np.int32)
    pk.Plan((60, 60, 1), [lin], 3, dtype=dtype, flags=pk.PLAN_HOST_ONLY)
    assert capfd.readouterr().err.count("planes in one launch") == 2


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_reported_tiling_gives_the_plan_again(dtype, monkeypatch, capfd):
    """A plan made with the tiling that another plan reports runs what that plan
    runs: axis passes where it took them, or a tiling of its own that was asked for."""
    monkeypatch.setenv("FFTB_LOG", "1")
    for dims, nb, asked in (((108, 100, 120), 50, None), ((96, 96, 96), 63, None), ((96, 96, 96), 64, None),
                            ((32, 32, 32), 4, None), ((6, 4, 540), 3, None), ((60, 50, 45), 7, dict(threads=128)),
                            ((96, 96, 96), 64, dict(inv_acc=1)), ((60, 50, 45), 7, dict(fwd_threads=128))):
        p, log = _log(capfd, dims, nb, dtype, tuning=asked)
        again = {f"{d}_{k}": v for d in ("inv", "fwd") for k, v in p.info["tuning"][d].items()}
        q, log2 = _log(capfd, dims, nb, dtype, tuning=again)
        assert log2 == log, (dims, nb, asked)
        assert q.info["tuning"] == p.info["tuning"]
