"""Calls at the ends of their ranges keep their speed: the path that a size or
an input takes is not a multiple slower there than a simple measure of the
same work on the same card.  Every bound has the time of a wrong path well
above it and the right one's well below (both are given), so that noise
decides nothing; results are checked too.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _say(text):
    print("call shape:", text, flush=True)


def _kernel_us(fn, name):
    """Median time of kernel `name` in seven calls of fn."""
    from paper_2503_01074_amd import _lib
    us = []
    fn()
    for _ in range(7):
        _lib.oceansim_trace_enable(True)
        try:
            fn()
            torch.cuda.synchronize()
            us.append(_lib.oceansim_trace_summary()[name][1])
        finally:
            _lib.oceansim_trace_enable(False)
    return sorted(us)[3]


def test_returns_in_one_bin():
    """256 frames of 32768 returns, all in one bin (a wall at normal incidence)
    against scattered: the tiles take 13 times as long; by compare-and-swap of
    that one LDS word 24 times."""
    import paper_2503_01074_amd as osm
    _say("returns in one bin")
    n, frames = 32768, 256
    g = osm.SonarGeometry(r_min=1.0, r_max=65.0, n_range=256, n_azimuth=255, fov_az=2.0, fov_el=0.35,
                          speckle_mode=osm.SPECKLE_OFF)
    gen = torch.Generator(device="cuda").manual_seed(3)
    zero = torch.zeros(n, device="cuda")
    mat = torch.zeros(n, dtype=torch.int32, device="cuda")

    def hits(phi, r):
        return osm.DeviceHits(r * torch.cos(phi), r * torch.sin(phi), zero, -torch.cos(phi), -torch.sin(phi), zero, mat)

    params = osm.sonar_params([dict(alpha=0.0, gain=1.0, sigma_phi=0.2, sigma_sa=0.1, sigma_sm=0.1)])
    refl = torch.ones(1, device="cuda")
    piled = hits(zero, torch.full((n,), 20.1, device="cuda"))
    spread = hits(torch.rand(n, generator=gen, device="cuda") * 1.99 - 0.995,
                  torch.rand(n, generator=gen, device="cuda") * 63.8 + 1.1)
    out = osm.render_sonar([g], [piled], params, refl)[0]["polar"]
    want = torch.zeros_like(out)
    want[int((20.1 - 1.0) / 0.25), 127] = n   # unit intensities: an exact sum
    assert torch.equal(out, want)
    t = {k: _kernel_us(lambda: osm.render_sonar([g] * frames, [h] * frames, params, refl), "k_tile")
         for k, h in (("piled", piled), ("spread", spread))}
    assert t["piled"] < 18.0 * t["spread"], t
