"""GPU parity of plans whose camera forward is split over the binning and the
fan launch: camera sizes on both sides of the line (1024 blocks of 1024
pixels), fans with more and with fewer workgroups than the share, no fan, and
several camera frames of odd sizes, against the FP64 oracle."""
import pytest

import oracle
from oracle import SonarConfig
import workloads as W
from _tol import assert_image_close

pytestmark = pytest.mark.gpu


# (name, fans [(range, azimuth, fan_h, fan_w)], cameras [(height, width)])
CASES = [
    ("just below the line", [(256, 128, 1024, 1025)], [(1023, 1024)]),
    ("at the line", [(256, 128, 1024, 1025)], [(1024, 1024)]),
    ("few fan workgroups", [(64, 48, 40, 71), (33, 21, 17, 16)], [(1024, 1024)]),
    ("one fan workgroup", [(33, 21, 9, 16)], [(1025, 1023)]),
    ("no fan", [(64, 48, 0, 0)], [(1024, 1024)]),
    ("odd frames", [(128, 96, 301, 517), (300, 201, 700, 901)], [(511, 1023), (3, 5), (1, 1), (767, 1025)]),
]


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("name,fans,images", CASES, ids=[c[0].replace(" ", "_") for c in CASES])
def test_camera_split_over_binning_and_fan(name, fans, images, graph):
    import torch
    import paper_2503_01074_amd as osm
    print("[case] camera split, %s, graph %s" % (name, graph), flush=True)
    st = W.Stream(961, len(images))
    specs = [W.SonarSpec(r_min=0.5, r_max=11.0, sigma_phi=0.3, sigma_sa=0.1, sigma_sm=0.1, seed_lo=7, gamma_k=2,
                         n_range=r, n_azimuth=a, fan_h=h, fan_w=w, alpha=0.08, gain=1.1, frame_id=k,
                         speckle_mode=W.SPECKLE_PAPER) for k, (r, a, h, w) in enumerate(fans)]
    frames = [W.SonarFrame(s, W.make_hits(st, s, 3000, n_materials=5, outside_frac=0.05)) for s in specs]
    refl = frames[0].hits.refl
    for f in frames:
        f.hits.refl = refl
    cams = [W.make_camera(st, h, w, water_row=k % 2) for k, (h, w) in enumerate(images)]
    waters = [W.make_water(st), W.make_water(st)]
    plan = osm.Plan([(osm.SonarGeometry.from_spec(s, param_row=k), osm.DeviceHits.from_host(f.hits))
                     for k, (s, f) in enumerate(zip(specs, frames))],
                    [(torch.as_tensor(c.J).cuda(), torch.as_tensor(c.depth).cuda(), c.water_row) for c in cams],
                    sonar_params=osm.sonar_params([osm.sonar_params_from_spec(s) for s in specs]),
                    refl=torch.as_tensor(refl).cuda(),
                    water=osm.water_params([(w.beta_d, w.beta_b, w.b_inf) for w in waters]), graph=graph)
    sonar = [oracle.sonar_forward(SonarConfig.from_spec(f.spec), f.hits, refl) for f in frames]
    image = [oracle.uw_forward(c.J, c.depth, *(getattr(waters[c.water_row], k) for k in ("beta_d", "beta_b", "b_inf")))
             for c in cams]
    for rep in range(3):
        for o in plan.sonar_out + plan.camera_out:
            for key in ("polar", "fan", "out"):
                if o.get(key) is not None:
                    o[key].fill_(float("nan"))
        plan.forward()
        torch.cuda.synchronize()
        for o in plan.sonar_out + plan.camera_out:
            for key in ("polar", "fan", "out"):
                assert o.get(key) is None or torch.isfinite(o[key]).all()
        for k, (o, want) in enumerate(zip(plan.sonar_out, sonar)):
            assert_image_close(o["polar"].cpu().numpy(), want["out"], "%s polar %d rep %d" % (name, k, rep))
            if specs[k].fan_h:
                assert_image_close(o["fan"].cpu().numpy(), want["fan"], "%s fan %d rep %d" % (name, k, rep),
                                   mask=~want["ambiguous"])
        for k, (o, want) in enumerate(zip(plan.camera_out, image)):
            got = o["out"].cpu().numpy()
            assert_image_close(got, want, "%s camera %d rep %d" % (name, k, rep))
    plan.close()


@pytest.mark.parametrize("side,split", [(600, True), (480, False)])
def test_large_cameras_ride_in_the_binning_alone(side, split):
    """A camera frame of 1200 x 1200 pixels (1407 workgroups) is split over
    the binning and the fan launch only if the fan has a quarter of its
    pixels: 600 x 610, but not 480 x 610."""
    import torch
    import paper_2503_01074_amd as osm
    from paper_2503_01074_amd import _lib
    print("[case] camera split, fan side %d" % side, flush=True)
    st = W.Stream(962, side)
    spec = W.SonarSpec(r_min=0.5, r_max=11.0, n_range=64, n_azimuth=48, fan_h=side, fan_w=610,
                       speckle_mode=W.SPECKLE_OFF)
    hits = W.make_hits(st, spec, 3000, n_materials=5)
    cam = W.make_camera(st, 1200, 1200)
    water = W.make_water(st)
    plan = osm.Plan([(osm.SonarGeometry.from_spec(spec), osm.DeviceHits.from_host(hits))],
                    [(torch.as_tensor(cam.J).cuda(), torch.as_tensor(cam.depth).cuda(), 0)],
                    sonar_params=osm.sonar_params([osm.sonar_params_from_spec(spec)]),
                    refl=torch.as_tensor(hits.refl).cuda(),
                    water=osm.water_params([(water.beta_d, water.beta_b, water.b_inf)]))
    _lib.oceansim_trace_enable(True)
    try:
        plan.forward()
        torch.cuda.synchronize()
        names = set(_lib.oceansim_trace_summary())
    finally:
        _lib.oceansim_trace_enable(False)
    assert "k_bin_uw" in names and ("k_fan_uw" if split else "k_fan") in names
    assert ("k_fan" if split else "k_fan_uw") not in names
    want = oracle.sonar_forward(SonarConfig.from_spec(spec), hits, hits.refl)
    o = plan.sonar_out[0]
    assert_image_close(o["polar"].cpu().numpy(), want["out"], "polar")
    assert_image_close(o["fan"].cpu().numpy(), want["fan"], "fan", mask=~want["ambiguous"])
    image = oracle.uw_forward(cam.J, cam.depth, water.beta_d, water.beta_b, water.b_inf)
    assert_image_close(plan.camera_out[0]["out"].cpu().numpy(), image, "camera")
    plan.close()
