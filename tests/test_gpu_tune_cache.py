"""GPU tests of the autotuner's cache file beside the axis passes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

AUTOTUNE = 2


def _plan(tuning=None):
    from paper_2406_05577_amd import Plan
    dims = (96, 32, 30)
    lin = np.array([x + 96 * (y + 32 * z) for z in (0, 1, 29) for y in (0, 1, 31) for x in (0, 1, 95)], np.int32)
    return Plan(dims, [lin], 4, dtype="c128", flags=AUTOTUNE, tuning=tuning), lin


def test_entries_older_than_the_passes_are_timed_again(tmp_path, monkeypatch):
    """A cache line whose pick was made before the zero tiling could mean axis
    passes (same tag and layout, the key without them) is not taken."""
    def fnv(*parts):
        h = 1469598103934665603
        for b in b"".join(parts):
            h = (h ^ b) * 1099511628211 % (1 << 64)
        return h

    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("FFTB_TUNE_CACHE", str(cache))
    monkeypatch.setenv("FFTB_TUNE_MAX_CANDIDATES", "1")
    _, lin = _plan()
    fresh = cache.read_text()
    key = fnv(np.array([96, 32, 30], np.int32).tobytes(), np.int32(0).tobytes(), np.uint32(0).tobytes(),
              np.int64(lin.size).tobytes(), np.int32(4).tobytes(), lin.tobytes())
    stale = f"fftb-tune-v2 {key:x} 4 2 1 8 256 1 0 0 0 4 2 1 8 256 1 0 0 0\n"
    cache.write_text(stale)
    p, _ = _plan()
    assert p.info["autotuned"] == 1 and cache.read_text() == stale + fresh
    p.close()
    p, _ = _plan()       # and the new line is taken
    assert p.info["autotuned"] == 2
    p.close()


def test_autotuned_plans_keep_the_fused_potential_step(tmp_path, monkeypatch):
    """The potential step runs as passes with one x pass where the tuner, not the
    caller, chose the inverse's tiling (no plane kernel of the forward is
    launched), with the result of the two directions; a caller's own tiling of
    the inverse keeps the two directions."""
    import torch
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("FFTB_TUNE_CACHE", str(cache))
    monkeypatch.setenv("FFTB_TUNE_MAX_CANDIDATES", "1")
    _plan()
    tag, key = cache.read_text().split()[:2]
    cache.write_text(f"{tag} {key} 4 2 0 0 256 1 0 0 0 0 0 0 0 0 0 0 0 0\n")
    v = torch.rand(96 * 32 * 30, dtype=torch.float64, device="cuda") - 0.5
    out = {}
    for name, asked, fused in (("tuned", None, True), ("asked", dict(inv_path=1), False)):
        p, _ = _plan(asked)
        assert p.info["autotuned"] == 2 and p.info["tuning"]["inv"]["path"] == 1
        sph = torch.linspace(-1, 1, p.info["sphere_elems"], dtype=torch.float64, device="cuda").to(torch.complex128)
        p.set_profiling(True)
        out[name] = p.apply_potential(sph, v)
        n = {k: c for k, (c, _) in p.get_profile().items()}
        assert n["plane_inverse"] == 1 and n["plane_forward"] == (0 if fused else 1), (name, n)
        p.close()
    assert torch.linalg.norm(out["tuned"] - out["asked"]) <= 1e-12 * torch.linalg.norm(out["asked"])
