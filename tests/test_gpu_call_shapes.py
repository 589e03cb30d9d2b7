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


def _wall_us(fn):
    """Best of five mean times of 20 calls."""
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    fn()
    best = float("inf")
    for _ in range(5):
        a.record()
        for _ in range(20):
            fn()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 20 * 1e3)
    return best


@pytest.mark.parametrize("ticks, vehicles", [(1, 1 << 20), (8, 1 << 20), (16, 1 << 18)])
def test_dvl_of_few_ticks(ticks, vehicles):
    """A few ticks of very many vehicles against a copy of the same bytes (or
    12 us): 1 to 1.5 times its time; a workgroup's slab of 32 ticks for each 64
    vehicles takes 2.7 to 12 times."""
    import paper_2503_01074_amd as osm
    _say("DVL %d x %d" % (ticks, vehicles))
    gen = torch.Generator(device="cuda").manual_seed(ticks)
    t = torch.arange(ticks, device="cuda", dtype=torch.float64) * 0.02
    r = torch.rand(ticks, vehicles, 4, generator=gen, device="cuda") * 80.0 + 2.0
    v = torch.randn(ticks, vehicles, 3, generator=gen, device="cuda")
    src = torch.zeros(ticks * vehicles * 22, dtype=torch.uint8, device="cuda")
    dst = torch.empty_like(src)
    copy = _wall_us(lambda: dst.copy_(src))
    dvl = _wall_us(lambda: osm.dvl(t, r, v, sigma_v=0.01, seed=(1, 2)))
    assert dvl < 2.0 * max(copy, 12.0), (dvl, copy)


def _hull_over_floor(n=400, radius=3.0):
    """A floor of two triangles and a sphere of 2 n (n - 1) over it."""
    u, w = np.meshgrid(np.linspace(0, 2 * np.pi, n, endpoint=False), np.linspace(0.02, np.pi - 0.02, n), indexing="ij")
    v = np.stack([6.0 + radius * np.sin(w) * np.cos(u), radius * np.sin(w) * np.sin(u),
                  -14.0 + radius * np.cos(w)], -1).reshape(-1, 3)
    i = np.arange(n * n).reshape(n, n)
    a, b, c, d = i[:, :-1], np.roll(i, -1, 0)[:, :-1], np.roll(i, -1, 0)[:, 1:], i[:, 1:]
    t = np.concatenate([np.stack([a, b, c], -1).reshape(-1, 3), np.stack([a, c, d], -1).reshape(-1, 3)]) + 4
    floor = np.array([[-2e3, -2e3, -20], [2e3, -2e3, -20], [2e3, 2e3, -20], [-2e3, 2e3, -20]])
    v = np.concatenate([floor, v]).astype(np.float32)
    t = np.concatenate([[[0, 1, 2], [0, 2, 3]], t]).astype(np.int32)
    return v, t, (np.arange(len(t)) % 61).astype(np.int32)


def test_cast_over_a_dense_object():
    """Four poses in one launch against four launches of one, over an object
    whose triangles are far smaller than the rays' spacing: a third of
    their time; by one traversal for all rays of a wave as long or longer."""
    import paper_2503_01074_amd as osm
    _say("cast over a dense object")
    scene = osm.Scene(*_hull_over_floor())
    pose = (np.array([-24.0, 0.0, -13.0], np.float32), np.eye(3, dtype=np.float32))
    args = (1024, 128, float(np.float32(2.2)), float(np.float32(0.4)), 50.0)
    one = osm.raycast(scene, [pose], *args)
    four = osm.raycast(scene, [pose] * 4, *args)
    for h in four:
        assert torch.equal(h.mat, one[0].mat) and torch.equal(h.x, one[0].x)
    assert (one[0].mat >= 0).any()
    other = 4 * _wall_us(lambda: osm.raycast(scene, [pose], *args, out=one))
    cast = _wall_us(lambda: osm.raycast(scene, [pose] * 4, *args, out=four))
    assert cast < 0.6 * other, (cast, other)
    scene.close()


def test_backward_of_a_dense_fan():
    """A fan with 44 pixels in every polar bin: the operator kernel takes 3.5
    times as long as the forward's fan kernel, with few entries a round 8.4."""
    import paper_2503_01074_amd as osm
    _say("dense fan")
    n = 4000
    g = osm.SonarGeometry(r_min=0.5, r_max=20.0, n_range=256, n_azimuth=256, fov_az=2.2, fov_el=0.4, fan_h=1200,
                          fan_w=2401, speckle_mode=osm.SPECKLE_OFF)
    gen = torch.Generator(device="cuda").manual_seed(5)
    phi = torch.rand(n, generator=gen, device="cuda") * 2.0 - 1.0
    r = torch.rand(n, generator=gen, device="cuda") * 18.0 + 1.0
    zero = torch.zeros(n, device="cuda")
    h = osm.DeviceHits(r * torch.cos(phi), r * torch.sin(phi), zero, -torch.cos(phi), -torch.sin(phi), zero,
                       torch.zeros(n, dtype=torch.int32, device="cuda"))
    plan = osm.Plan([(g, h)] * 12,
                    sonar_params=osm.sonar_params([dict(alpha=0.1, gain=1.0, sigma_phi=0.2, sigma_sa=0.1, sigma_sm=0.1)]),
                    refl=torch.ones(1, device="cuda"), backward=True)
    for o in plan.sonar_out:
        o["grad_fan"].normal_(generator=gen)
    fan = _kernel_us(plan.forward, "k_fan")
    back = _kernel_us(plan.backward, "k_fant_bwd")
    plan.close()
    assert back < 5.5 * fan, (back, fan)
