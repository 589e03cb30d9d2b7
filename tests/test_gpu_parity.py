"""GPU parity: the HIP path (through the C ABI) against the FP64 oracle.

Bins are compared bit-exactly; images element by element to 1e-5 relative
(floor 1e-3 of the peak); gradients to 1e-5 of the oracle's analytic FP64
gradient and 1e-3 of FP64 central differences of the oracle's forward pass.
"""
import copy
import math
import sys

import numpy as np
import pytest

import oracle
from oracle import SonarConfig
import workloads as W
from _cases import build_hits, hit_at, tiny_golden
from _tol import (GRAD_RTOL_FD, GRAD_RTOL_ORACLE, assert_grad_cond, assert_image_close)

pytestmark = pytest.mark.gpu


def _osm():
    import torch  # noqa: F401
    import paper_2503_01074_amd as osm
    return osm


def _say(msg):
    print("[case] " + msg, flush=True)
    sys.stdout.flush()


def merged(frames):
    """Frames sharing one reflectivity table: per-frame tables concatenated,
    material ids offset (misses stay negative)."""
    out, tables, base = [], [], 0
    for f in frames:
        h = copy.copy(f.hits)
        h.mat = np.where(f.hits.mat >= 0, f.hits.mat + base, f.hits.mat).astype(np.int32)
        tables.append(f.hits.refl)
        base += f.hits.refl.shape[0]
        out.append(W.SonarFrame(f.spec, h))
    refl = np.concatenate(tables).astype(np.float32)
    for f in out:
        f.hits.refl = refl
    return out, refl


def gpu_forward(frames, refl, fan=True, bins=True):
    import torch
    osm = _osm()
    geoms = [osm.SonarGeometry.from_spec(f.spec, param_row=i) for i, f in enumerate(frames)]
    hits = [osm.DeviceHits.from_host(f.hits) for f in frames]
    params = osm.sonar_params([osm.sonar_params_from_spec(f.spec) for f in frames])
    refl_d = torch.as_tensor(refl).cuda()
    outs = osm.render_sonar(geoms, hits, params, refl_d, polar=True, fan=fan, bins=bins)
    torch.cuda.synchronize()
    return [{k: v.cpu().numpy() for k, v in o.items()} for o in outs]


def oracle_forward(frame, refl):
    return oracle.sonar_forward(SonarConfig.from_spec(frame.spec), frame.hits, refl)


def check_frame(got, want, what, fan=True):
    np.testing.assert_array_equal(got["bins"], want["bins"], err_msg=what + " bins")
    assert_image_close(got["polar"], want["out"], what + " polar")
    if fan and "fan" in want:
        assert_image_close(got["fan"], want["fan"], what + " fan", mask=~want["ambiguous"])


# --------------------------------------------------------------------------- #
# forward                                                                     #
# --------------------------------------------------------------------------- #
def test_tiny_golden():
    _say("tiny golden frame")
    spec, hits, bins, expected = tiny_golden()
    got = gpu_forward([W.SonarFrame(spec, hits)], hits.refl, fan=False)[0]
    np.testing.assert_array_equal(got["bins"], bins)
    np.testing.assert_allclose(got["polar"], expected, rtol=1e-6, atol=1e-7)


@pytest.mark.parametrize("name", ["c1", "c2"])
def test_workload_forward(name):
    frames = W.sonar_c1() if name == "c1" else W.sonar_c2()
    f = frames[0]
    _say("%s forward: %d returns, %dx%d bins, fan %dx%d" % (name, f.hits.n, f.spec.n_range,
                                                          f.spec.n_azimuth, f.spec.fan_h, f.spec.fan_w))
    got = gpu_forward(frames, f.hits.refl)[0]
    want = oracle_forward(f, f.hits.refl)
    check_frame(got, want, name)
    assert want["ambiguous"].sum() == 0


SMALL_SHAPES = [
    # (n_range, n_azimuth, fan_h, fan_w, n_returns)
    (37, 29, 41, 83, 3000),      # ragged everything, several tiles, odd fan width
    (1, 17, 8, 16, 200),         # single range row
    (23, 1, 9, 9, 200),          # single azimuth column
    (300, 4096, 64, 128, 20000),  # one row per tile (widest supported grid)
    (4100, 2, 16, 16, 5000),     # more range rows than the tile height many times over
]


@pytest.mark.parametrize("shape", SMALL_SHAPES)
@pytest.mark.parametrize("mode", [W.SPECKLE_OFF, W.SPECKLE_PAPER, W.SPECKLE_GAMMA])
def test_shapes_and_modes(shape, mode):
    Nr, Np, H, Wd, n = shape
    _say("shape %s mode %d" % (shape, mode))
    st = W.Stream(1234, Nr * 7 + Np + mode)
    spec = W.SonarSpec(r_min=0.7, r_max=13.0, n_range=Nr, n_azimuth=Np, fan_h=H, fan_w=Wd,
                       speckle_mode=mode, gamma_k=3, sigma_sm=0.15, sigma_sa=0.12, sigma_phi=0.3,
                       alpha=0.09, gain=1.3, seed_lo=77, seed_hi=5, frame_id=9)
    hits = W.make_hits(st, spec, n, n_materials=5, outside_frac=0.1)
    frame = W.SonarFrame(spec, hits)
    got = gpu_forward([frame], hits.refl)[0]
    want = oracle_forward(frame, hits.refl)
    check_frame(got, want, "shape %s mode %d" % (shape, mode))


@pytest.mark.parametrize("k", [1, 2, 4, 5, 8])
def test_gamma_shapes(k):
    _say("gamma k=%d" % k)
    st = W.Stream(55, k)
    spec = W.SonarSpec(r_min=0.5, r_max=20.0, n_range=128, n_azimuth=96, fan_h=64, fan_w=128,
                       speckle_mode=W.SPECKLE_GAMMA, gamma_k=k, seed_lo=k, frame_id=3)
    hits = W.make_hits(st, spec, 5000)
    f = W.SonarFrame(spec, hits)
    check_frame(gpu_forward([f], hits.refl)[0], oracle_forward(f, hits.refl), "gamma k=%d" % k)


def test_empty_and_all_miss():
    _say("empty and all-miss frames")
    spec = W.SonarSpec(r_min=0.5, r_max=20.0, n_range=64, n_azimuth=64, fan_h=32, fan_w=64,
                       speckle_mode=W.SPECKLE_GAMMA, seed_lo=3)
    empty = build_hits([], refl=[1.0])
    st = W.Stream(8, 8)
    misses = W.make_hits(st, spec, 1000, miss_frac=1.0)
    for hits, what in [(empty, "empty"), (misses, "all misses")]:
        f = W.SonarFrame(spec, hits)
        got = gpu_forward([f], hits.refl)[0]
        want = oracle_forward(f, hits.refl)
        check_frame(got, want, what)
        assert np.all(want["P"] == 0)


def test_kappa_one_and_material_ids():
    _say("path factor 1 and out-of-table material ids")
    st = W.Stream(9, 9)
    spec = W.SonarSpec(r_min=0.5, r_max=20.0, n_range=100, n_azimuth=80, kappa=1.0,
                       speckle_mode=W.SPECKLE_OFF)
    hits = W.make_hits(st, spec, 4000, n_materials=10)
    hits.mat[::7] = 10          # one past the table: a miss
    hits.mat[::11] = 1 << 30    # far outside the table: a miss
    f = W.SonarFrame(spec, hits)
    check_frame(gpu_forward([f], hits.refl, fan=False)[0], oracle_forward(f, hits.refl), "kappa 1", fan=False)


def test_dense_collisions():
    """Many returns per bin (the dense shape of the paper's qualitative figure:
    3000 x 460 rays on 350 x 220 bins, here at a tenth of the rays)."""
    _say("dense collisions")
    st = W.Stream(10, 10)
    spec = W.SonarSpec(r_min=0.5, r_max=20.0, n_range=350, n_azimuth=220, fan_h=350, fan_w=700,
                       speckle_mode=W.SPECKLE_GAMMA, seed_lo=1)
    hits = W.make_hits(st, spec, 138000)
    f = W.SonarFrame(spec, hits)
    check_frame(gpu_forward([f], hits.refl)[0], oracle_forward(f, hits.refl), "dense")


@pytest.mark.parametrize("n_hot", [1, 2, 7, 64])
@pytest.mark.parametrize("n_az", [15, 129])
def test_returns_piled_up_in_few_bins(n_hot, n_az):
    """Returns on the x axis at n_hot ranges, all facing the sensor without
    attenuation: intensities are the reflectivities 1 and 1/2 exactly, so the
    sums of lanes that change the same histogram word at once are exact."""
    spec = W.SonarSpec(r_min=1.0, r_max=65.0, n_range=64, n_azimuth=n_az, speckle_mode=W.SPECKLE_OFF, alpha=0.0)
    n = 40001
    st = W.Stream(15, n_hot)
    row = st.integers(0, n_hot - 1, n)
    x = (1.5 + row).astype(np.float32)
    z = np.zeros(n, np.float32)
    mat = st.integers(0, 1, n).astype(np.int32)
    hits = W.SonarHits(x=x, y=z, z=z.copy(), nx=np.full(n, -1, np.float32), ny=z.copy(), nz=z.copy(), mat=mat,
                       refl=np.array([1.0, 0.5], np.float32))
    want = np.zeros((64, n_az))
    np.add.at(want, (row, n_az // 2), hits.refl[mat])
    got = gpu_forward([W.SonarFrame(spec, hits)], hits.refl, fan=False)[0]
    np.testing.assert_array_equal(got["polar"], want.astype(np.float32))


def test_batched_equals_plain_and_oracle():
    _say("batched uneven frames")
    frames = W.sonar_c3(n_frames=6)
    frames, refl = merged(frames)
    batched = gpu_forward(frames, refl)
    for i, f in enumerate(frames):
        plain = gpu_forward([f], refl)[0]
        want = oracle_forward(f, refl)
        check_frame(batched[i], want, "batched frame %d" % i)
        np.testing.assert_array_equal(batched[i]["bins"], plain["bins"])
        assert_image_close(batched[i]["polar"], plain["polar"], "batched vs plain %d" % i, rtol=1e-6)
        assert_image_close(batched[i]["fan"], plain["fan"], "batched vs plain fan %d" % i, rtol=1e-6)


# --------------------------------------------------------------------------- #
# backward                                                                    #
# --------------------------------------------------------------------------- #
def gpu_backward(frames, refl, gpol, gfan, saved=False):
    """GPU gradients; with ``saved`` the forward pass runs first and saves the
    fan stencils that the backward pass then reads."""
    import torch
    osm = _osm()
    geoms = [osm.SonarGeometry.from_spec(f.spec, param_row=0) for f in frames]
    hits = [osm.DeviceHits.from_host(f.hits) for f in frames]
    params = osm.sonar_params([osm.sonar_params_from_spec(frames[0].spec)])
    refl_d = torch.as_tensor(refl).cuda()
    gp = [None if g is None else torch.as_tensor(g, dtype=torch.float32).cuda() for g in gpol]
    gf = [None if g is None else torch.as_tensor(g, dtype=torch.float32).cuda() for g in gfan]
    stencils = None
    if saved:
        outs = osm.render_sonar(geoms, hits, params, refl_d, save_stencil=True)
        stencils = [o.get("stencil") for o in outs]
    g_refl, g_par = osm.render_sonar_backward(geoms, hits, params, refl_d, gp, gf, stencils)
    torch.cuda.synchronize()
    return g_refl.cpu().numpy().astype(np.float64), g_par.cpu().numpy().astype(np.float64)


def oracle_backward(frames, refl, gpol, gfan):
    """Summed oracle gradients and their conditions (sums of term magnitudes)."""
    g_refl = np.zeros(refl.shape[0])
    g_par = np.zeros(5)
    a_refl = np.zeros(refl.shape[0])
    a_par = np.zeros(5)
    for f, gp, gf in zip(frames, gpol, gfan):
        a, b, _, ca, cb = oracle.sonar_backward(SonarConfig.from_spec(f.spec), f.hits, refl, gp, gf,
                                                with_abs=True)
        g_refl += a
        g_par += b
        a_refl += ca
        a_par += cb
    return g_refl, g_par, a_refl, a_par


def _bwd_case(mode, n_mat, n_frames=1, fan=True, polar=True, seed=0):
    st = W.Stream(4321 + seed, mode * 10 + n_frames)
    frames = []
    for k in range(n_frames):
        spec = W.SonarSpec(r_min=0.5, r_max=10.0, n_range=48 + 8 * k, n_azimuth=40 + 4 * k,
                           fan_h=(40 if fan else 0), fan_w=(72 + 2 * k if fan else 0),
                           alpha=0.11, gain=1.2, sigma_phi=0.3, sigma_sa=0.15, sigma_sm=0.1,
                           speckle_mode=mode, gamma_k=4, seed_lo=17, frame_id=k)
        frames.append(W.SonarFrame(spec, W.make_hits(st, spec, 3000, n_materials=n_mat)))
    frames, refl = merged(frames) if n_mat is None else (frames, frames[0].hits.refl)
    if n_mat is not None:
        for f in frames:
            f.hits.refl = refl
    gpol = [W.loss_weights((7, 2 * k), (f.spec.n_range, f.spec.n_azimuth)) if polar else None
            for k, f in enumerate(frames)]
    gfan = [W.loss_weights((7, 2 * k + 1), (f.spec.fan_h, f.spec.fan_w)) if fan else None
            for k, f in enumerate(frames)]
    return frames, refl, gpol, gfan


def _oracle_loss(frames, refl, gpol, gfan, **over):
    L = 0.0
    for f, gp, gf in zip(frames, gpol, gfan):
        res = oracle.sonar_forward(SonarConfig.from_spec(f.spec, **over), f.hits, refl)
        if gp is not None:
            L += float((gp.astype(np.float64) * res["out"]).sum())
        if gf is not None:
            L += float((gf.astype(np.float64) * res["fan"]).sum())
    return L


@pytest.mark.parametrize("saved", [False, True])
@pytest.mark.parametrize("mode", [W.SPECKLE_OFF, W.SPECKLE_PAPER, W.SPECKLE_GAMMA])
@pytest.mark.parametrize("n_mat", [6, 64])
def test_sonar_backward_vs_oracle_and_fd(mode, n_mat, saved):
    _say("sonar backward mode %d n_mat %d saved stencils %s" % (mode, n_mat, saved))
    frames, refl, gpol, gfan = _bwd_case(mode, n_mat, n_frames=2)
    g_refl, g_par = gpu_backward(frames, refl, gpol, gfan, saved)
    o_refl, o_par, c_refl, c_par = oracle_backward(frames, refl, gpol, gfan)
    assert_grad_cond(g_refl, o_refl, c_refl, what="refl vs oracle")
    assert_grad_cond(g_par[0, :5], o_par, c_par, what="params vs oracle")
    assert np.all(g_par[0, 5:] == 0)
    # FP64 central differences of the oracle's forward pass, one parameter at a time
    for k, name in enumerate(["alpha", "gain", "sigma_phi", "sigma_sa", "sigma_sm"]):
        x0 = float(getattr(frames[0].spec, name))
        h = 1e-6 * max(1.0, abs(x0))
        fd = (_oracle_loss(frames, refl, gpol, gfan, **{name: x0 + h}) -
              _oracle_loss(frames, refl, gpol, gfan, **{name: x0 - h})) / (2 * h)
        if abs(fd) < 1e-9 and abs(g_par[0, k]) < 1e-9:
            continue
        assert abs(g_par[0, k] - fd) <= GRAD_RTOL_FD * max(abs(fd), 1e-6), (name, g_par[0, k], fd)


def test_sonar_backward_many_materials_and_polar_only():
    _say("sonar backward, per-return reflectivity (atomic path), polar-only loss")
    frames, refl, gpol, gfan = _bwd_case(W.SPECKLE_GAMMA, None, n_frames=3, fan=False)
    g_refl, g_par = gpu_backward(frames, refl, gpol, gfan)
    o_refl, o_par, c_refl, c_par = oracle_backward(frames, refl, gpol, gfan)
    assert refl.shape[0] > 64
    assert_grad_cond(g_refl, o_refl, c_refl, what="refl vs oracle")
    assert_grad_cond(g_par[0, :5], o_par, c_par, what="params vs oracle")


def test_sonar_backward_fan_only_and_bitwise_repeat():
    _say("sonar backward, fan-only loss, five repeats")
    frames, refl, gpol, gfan = _bwd_case(W.SPECKLE_PAPER, 64, n_frames=2, polar=False)
    runs = [gpu_backward(frames, refl, gpol, gfan) for _ in range(5)]
    for a, b in runs[1:]:
        np.testing.assert_array_equal(a, runs[0][0])
        np.testing.assert_array_equal(b, runs[0][1])
    o_refl, o_par, c_refl, c_par = oracle_backward(frames, refl, gpol, gfan)
    assert_grad_cond(runs[0][0], o_refl, c_refl, what="refl vs oracle")
    assert_grad_cond(runs[0][1][0, :5], o_par, c_par, what="params vs oracle")


# --------------------------------------------------------------------------- #
# camera                                                                      #
# --------------------------------------------------------------------------- #
def _gpu_uw(cams, waters):
    import torch
    osm = _osm()
    Js = [torch.as_tensor(c.J).cuda() for c in cams]
    ds = [torch.as_tensor(c.depth).cuda() for c in cams]
    water = osm.water_params([(w.beta_d, w.beta_b, w.b_inf) for w in waters])
    outs = osm.uw_form(Js, ds, water, [c.water_row for c in cams])
    torch.cuda.synchronize()
    return [o.cpu().numpy() for o in outs]


def test_uw_forward_c2():
    _say("uw_form 1920x1080")
    cams, waters = W.camera_c2()
    got = _gpu_uw(cams, waters)[0]
    w = waters[0]
    want = oracle.uw_forward(cams[0].J, cams[0].depth, w.beta_d, w.beta_b, w.b_inf)
    assert_image_close(got, want, "uw 1080p")


def test_uw_special_cases_and_ragged_batch():
    _say("uw_form special cases, ragged batch")
    st = W.Stream(12, 12)
    shapes = [(7, 13), (32, 32), (1, 1), (5, 3), (64, 33)]
    cams = [W.make_camera(st, h, w, water_row=k % 2) for k, (h, w) in enumerate(shapes)]
    cams[2].depth[:] = np.inf
    cams[3].depth[:] = 0.0
    waters = [W.make_water(st), W.WaterSpec(beta_d=np.zeros(3, np.float32), beta_b=np.zeros(3, np.float32),
                                            b_inf=np.array([0.1, 0.2, 0.3], np.float32))]
    got = _gpu_uw(cams, waters)
    for c, g in zip(cams, got):
        w = waters[c.water_row]
        want = oracle.uw_forward(c.J, c.depth, w.beta_d, w.beta_b, w.b_inf)
        assert_image_close(g, want, "uw %s" % (c.depth.shape,))
        if c.water_row == 1:
            np.testing.assert_array_equal(g, c.J)   # no water: the clear image, bit for bit


@pytest.mark.parametrize("shapes", [[(1, 1)], [(1, 3)], [(1, 5)], [(7, 37)], [(1, 1023)], [(1, 1025)], [(3, 683)],
                                    [(1, 2047)], [(1, 2050)], [(541, 963)],
                                    [(1, 4097), (5, 410), (1, 2), (541, 963), (64, 64)]])
def test_uw_images_of_any_size(shapes):
    """Pixel counts of every remainder by four (planes that start unaligned
    to 16 bytes) and around the kernels' blocks of 1024 and 2048 pixels, alone
    and in one batch: forward, parameter and image gradients; guard pixels
    around every output stay as they were."""
    import torch
    osm = _osm()
    st = W.Stream(14, sum(h * w for h, w in shapes))
    cams = [W.make_camera(st, h, w) for h, w in shapes]
    water = W.make_water(st)
    gos = [W.loss_weights((14, k), c.J.shape) for k, c in enumerate(cams)]
    wt = osm.water_params([(water.beta_d, water.beta_b, water.b_inf)])
    Js = [torch.as_tensor(c.J).cuda() for c in cams]
    ds = [torch.as_tensor(c.depth).cuda() for c in cams]

    def guarded(shape):   # a view 16-byte aligned inside a larger buffer of a marker value
        n = int(np.prod(shape))
        buf = torch.full((n + 64,), 7.0, device="cuda")
        return buf, buf[32:32 + n].view(shape)

    from paper_2503_01074_amd import _lib, api
    bufs = [[guarded(c.J.shape), guarded(c.J.shape), guarded(c.depth.shape)] for c in cams]
    frames = [api._uw_struct(J, d, b[0][1], 0, torch.as_tensor(g).cuda(), b[1][1], b[2][1])
              for J, d, g, b in zip(Js, ds, gos, bufs)]
    keep = [torch.as_tensor(g).cuda() for g in gos]
    for f, g in zip(frames, keep):
        f.grad_out = g.data_ptr()
    ws = torch.empty(max(256, _lib.oceansim_uw_workspace_size(frames, True)), dtype=torch.uint8, device="cuda")
    g_w = torch.empty(1, 9, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    _lib.oceansim_uw_form(frames, wt.data_ptr(), 1, ws.data_ptr(), ws.numel(), s)
    _lib.oceansim_uw_form_backward(frames, wt.data_ptr(), 1, g_w.data_ptr(), ws.data_ptr(), ws.numel(), s)
    torch.cuda.synchronize()
    o_par, c_par = np.zeros(9), np.zeros(9)
    bd, bb, bi = (x.astype(np.float64) for x in (water.beta_d, water.beta_b, water.b_inf))
    for k, (c, b) in enumerate(zip(cams, bufs)):
        for buf, _ in b:
            assert bool((buf[:32] == 7.0).all()) and bool((buf[-32:] == 7.0).all())
        assert_image_close(b[0][1].cpu().numpy(), oracle.uw_forward(c.J, c.depth, bd, bb, bi), "uw %d" % k)
        p, oj, od, cp = oracle.uw_backward(c.J, c.depth, bd, bb, bi, gos[k], with_abs=True)
        o_par += p
        c_par += cp
        assert_image_close(b[1][1].cpu().numpy(), oj, "grad J %d" % k)
        d = c.depth.astype(np.float64)[None]
        T, S = np.exp(-bd[:, None, None] * d), np.exp(-bb[:, None, None] * d)
        cond = (np.abs(gos[k]) * (bd[:, None, None] * np.abs(c.J) * T + bi[:, None, None] * bb[:, None, None] * S)).sum(0)
        assert np.all(np.abs(b[2][1].cpu().numpy().astype(np.float64) - od) <= 1e-5 * cond + 1e-30), "grad depth %d" % k
    assert_grad_cond(g_w.cpu().numpy()[0], o_par, c_par, what="water params vs oracle")


def test_uw_backward():
    _say("uw_form backward")
    import torch
    osm = _osm()
    st = W.Stream(13, 13)
    cams = [W.make_camera(st, 96, 64), W.make_camera(st, 540, 960), W.make_camera(st, 3, 5)]
    water = W.make_water(st)
    gos = [W.loss_weights((13, k), c.J.shape) for k, c in enumerate(cams)]
    Js = [torch.as_tensor(c.J).cuda() for c in cams]
    ds = [torch.as_tensor(c.depth).cuda() for c in cams]
    wt = osm.water_params([(water.beta_d, water.beta_b, water.b_inf)])
    g_w, gJ, gd = osm.uw_form_backward(Js, ds, wt, [torch.as_tensor(g).cuda() for g in gos])
    torch.cuda.synchronize()
    o_par = np.zeros(9)
    c_par = np.zeros(9)
    bd, bb, bi = (x.astype(np.float64) for x in (water.beta_d, water.beta_b, water.b_inf))
    for k, c in enumerate(cams):
        p, oj, od, cp = oracle.uw_backward(c.J, c.depth, bd, bb, bi, gos[k], with_abs=True)
        o_par += p
        c_par += cp
        assert_image_close(gJ[k].cpu().numpy(), oj, "grad J %d" % k)
        # dL/dd sums terms of both signs over the channels: bound its error by
        # 1e-5 of the sum of the magnitudes of those terms (its condition)
        d = c.depth.astype(np.float64)[None]
        J = c.J.astype(np.float64)
        T = np.exp(-bd[:, None, None] * d)
        S = np.exp(-bb[:, None, None] * d)
        cond = (np.abs(gos[k]) * (bd[:, None, None] * np.abs(J) * T + bi[:, None, None] * bb[:, None, None] * S)).sum(0)
        err = np.abs(gd[k].cpu().numpy().astype(np.float64) - od)
        assert np.all(err <= 1e-5 * cond + 1e-30), "grad depth %d: worst %.3e" % (k, (err / np.maximum(cond, 1e-300)).max())
    assert_grad_cond(g_w.cpu().numpy()[0], o_par, c_par, what="water params vs oracle")
    params = np.concatenate([bd, bb, bi])
    for k in range(9):
        h = 1e-6 * max(1.0, abs(params[k]))
        p1, p2 = params.copy(), params.copy()
        p1[k] += h
        p2[k] -= h
        L = lambda p: sum(float((g * oracle.uw_forward(c.J, c.depth, p[:3], p[3:6], p[6:])).sum())
                          for c, g in zip(cams, gos))
        fd = (L(p1) - L(p2)) / (2 * h)
        assert abs(g_w.cpu().numpy()[0, k] - fd) <= GRAD_RTOL_FD * abs(fd), (k, fd)


@pytest.mark.parametrize("saved", [False, True])
def test_sonar_backward_tall_fan_rescale(saved):
    """A fan taller than one row batch with many candidates per tile and a
    gradient whose magnitude grows down the image (the fixed-point scale of a
    tile grows between batches)."""
    _say("sonar backward, 1400 x 2800 fan, growing gradient magnitude, saved %s" % saved)
    st = W.Stream(77, 1)
    spec = W.SonarSpec(r_min=0.5, r_max=30.0, n_range=300, n_azimuth=200, fan_h=1400, fan_w=2800,
                       alpha=0.08, gain=1.1, sigma_phi=0.3, sigma_sa=0.15, speckle_mode=W.SPECKLE_GAMMA,
                       seed_lo=5, frame_id=1)
    frames = [W.SonarFrame(spec, W.make_hits(st, spec, 20000, n_materials=16))]
    refl = frames[0].hits.refl
    ramp = np.logspace(-6, 3, spec.fan_h)[:, None]
    gfan = [(W.loss_weights((77, 2), (spec.fan_h, spec.fan_w)) * ramp).astype(np.float32)]
    gpol = [W.loss_weights((77, 3), (spec.n_range, spec.n_azimuth))]
    g_refl, g_par = gpu_backward(frames, refl, gpol, gfan, saved)
    o_refl, o_par, c_refl, c_par = oracle_backward(frames, refl, gpol, gfan)
    assert_grad_cond(g_refl, o_refl, c_refl, what="refl vs oracle")
    assert_grad_cond(g_par[0, :5], o_par, c_par, what="params vs oracle")


@pytest.mark.parametrize("saved", [False, True])
def test_sonar_backward_nonfinite_gradient(saved):
    _say("sonar backward, a NaN in the fan gradient, saved %s" % saved)
    frames, refl, gpol, gfan = _bwd_case(W.SPECKLE_GAMMA, 6, n_frames=1)
    gfan = [g.copy() for g in gfan]
    gfan[0][20, 30] = np.nan
    g_refl, g_par = gpu_backward(frames, refl, gpol, gfan, saved)
    o_refl, o_par, _, _ = oracle_backward(frames, refl, gpol, gfan)
    np.testing.assert_array_equal(np.isnan(g_refl), np.isnan(o_refl))
    np.testing.assert_array_equal(np.isnan(g_par[0, :5]), np.isnan(o_par))
    assert np.isnan(o_par).any()


def test_negative_reflectivities():
    """Sums that cancel to zero inside a bin (only possible with signed
    reflectivities) still get the multiplicative speckle exactly once."""
    _say("signed reflectivities")
    st = W.Stream(78, 1)
    spec = W.SonarSpec(r_min=0.5, r_max=10.0, n_range=64, n_azimuth=48, fan_h=32, fan_w=64,
                       speckle_mode=W.SPECKLE_GAMMA, seed_lo=8)
    hits = W.make_hits(st, spec, 30000, n_materials=3)
    hits.refl = np.array([0.5, -0.5, 0.25], np.float32)
    # put pairs of opposite returns on the same point so that some bins cancel exactly
    hits.x[1::2], hits.y[1::2], hits.z[1::2] = hits.x[0::2], hits.y[0::2], hits.z[0::2]
    hits.nx[1::2], hits.ny[1::2], hits.nz[1::2] = hits.nx[0::2], hits.ny[0::2], hits.nz[0::2]
    hits.mat[0::4] = 0
    hits.mat[1::4] = 1
    f = W.SonarFrame(spec, hits)
    want = oracle_forward(f, hits.refl)
    got = gpu_forward([f], hits.refl)[0]
    np.testing.assert_array_equal(got["bins"], want["bins"])
    # bin sums of signed terms: float32 rounding is relative to the sum of the
    # magnitudes of the terms (cond), not to the cancelled result
    ok = want["bins"] >= 0
    cond = np.bincount(want["bins"][ok], weights=np.abs(want["intensity"][ok]),
                       minlength=spec.n_range * spec.n_azimuth).reshape(spec.n_range, spec.n_azimuth)
    _, mul = oracle.speckle_fields(SonarConfig.from_spec(spec))
    o = want["out"]
    bound = 1e-5 * np.maximum(np.abs(o), 1e-3 * np.abs(o).max()) + 1e-6 * float(spec.gain) * mul * cond
    assert (np.abs(got["polar"] - o) <= bound).all()
    assert ((want["P"] == 0) & (cond > 0)).sum() > 0       # some bins cancel exactly


@pytest.mark.parametrize("shape", [(37, 29, 41, 83), (1, 17, 8, 16), (23, 1, 9, 9), (60, 40, 33, 64)])
def test_sonar_backward_saved_matches_recomputed(shape):
    """Saved-stencil and recomputed-geometry backward passes agree, on odd and
    degenerate grids (one range row, one azimuth column, odd fan width)."""
    Nr, Np, H, Wd = shape
    _say("saved vs recomputed stencils %s" % (shape,))
    st = W.Stream(79, Nr + Np)
    spec = W.SonarSpec(r_min=0.7, r_max=13.0, n_range=Nr, n_azimuth=Np, fan_h=H, fan_w=Wd,
                       speckle_mode=W.SPECKLE_PAPER, seed_lo=3, frame_id=2)
    frames = [W.SonarFrame(spec, W.make_hits(st, spec, 3000, n_materials=5))]
    refl = frames[0].hits.refl
    gpol = [W.loss_weights((79, 1), (Nr, Np))]
    gfan = [W.loss_weights((79, 2), (H, Wd))]
    a = gpu_backward(frames, refl, gpol, gfan, False)
    b = gpu_backward(frames, refl, gpol, gfan, True)
    o_refl, o_par, c_refl, c_par = oracle_backward(frames, refl, gpol, gfan)
    for g_refl, g_par in (a, b):
        assert_grad_cond(g_refl, o_refl, c_refl, what="refl vs oracle")
        assert_grad_cond(g_par[0, :5], o_par, c_par, what="params vs oracle")


@pytest.mark.parametrize("per_return_refl", [False, True])
def test_sonar_backward_many_frames_and_rows(per_return_refl):
    """Seven uneven frames in one backward call, sharing four parameter rows
    (frames 0, 3 on row 0; 1, 4 on row 1; 2, 5 on row 2; 6 on row 3), every
    speckle mode, a shared 20-material table or per-return reflectivity:
    each row's gradient is the sum over its frames, the reflectivity gradient
    the sum over all."""
    import torch
    osm = _osm()
    _say("sonar backward, 7 frames on 4 parameter rows, per-return reflectivity %s" % per_return_refl)
    st = W.Stream(4400, 7 + per_return_refl)
    rows = [0, 1, 2, 0, 1, 2, 3]
    modes = [W.SPECKLE_GAMMA, W.SPECKLE_PAPER, W.SPECKLE_OFF, W.SPECKLE_GAMMA, W.SPECKLE_PAPER, W.SPECKLE_OFF,
             W.SPECKLE_GAMMA]
    frames = []
    for k, (r, mode) in enumerate(zip(rows, modes)):
        spec = W.SonarSpec(r_min=0.5, r_max=8.0 + k, n_range=30 + 7 * k, n_azimuth=24 + 5 * k, fan_h=20 + 3 * k,
                           fan_w=41 + 6 * k, alpha=0.05 + 0.02 * r, gain=0.8 + 0.2 * r, sigma_phi=0.2 + 0.05 * r,
                           sigma_sa=0.1 + 0.02 * r, sigma_sm=0.1 + 0.03 * r, speckle_mode=mode, gamma_k=3,
                           seed_lo=5, frame_id=k)
        frames.append(W.SonarFrame(spec, W.make_hits(st, spec, 900 + 300 * k, n_materials=20)))
    if per_return_refl:
        frames, refl = merged(frames)            # one reflectivity per return (ids offset per frame)
    else:
        refl = frames[0].hits.refl
        for f in frames:
            f.hits.refl = refl
    gpol = [W.loss_weights((4401, k), (f.spec.n_range, f.spec.n_azimuth)) for k, f in enumerate(frames)]
    gfan = [W.loss_weights((4402, k), (f.spec.fan_h, f.spec.fan_w)) for k, f in enumerate(frames)]
    geoms = [osm.SonarGeometry.from_spec(f.spec, param_row=r) for f, r in zip(frames, rows)]
    hits = [osm.DeviceHits.from_host(f.hits) for f in frames]
    row_spec = {r: f.spec for f, r in zip(frames, rows)}
    params = osm.sonar_params([osm.sonar_params_from_spec(row_spec[r]) for r in range(4)])
    refl_d = torch.as_tensor(refl).cuda()
    outs = osm.render_sonar(geoms, hits, params, refl_d, save_stencil=True)
    g_refl, g_par = osm.render_sonar_backward(
        geoms, hits, params, refl_d, [torch.as_tensor(g).cuda() for g in gpol],
        [torch.as_tensor(g).cuda() for g in gfan], [o.get("stencil") for o in outs])
    torch.cuda.synchronize()
    g_refl = g_refl.cpu().numpy().astype(np.float64)
    g_par = g_par.cpu().numpy().astype(np.float64)
    o_refl, c_refl = np.zeros(refl.shape[0]), np.zeros(refl.shape[0])
    o_par, c_par = np.zeros((4, 5)), np.zeros((4, 5))
    for f, r, gp, gf in zip(frames, rows, gpol, gfan):
        a, b, _, ca, cb = oracle.sonar_backward(SonarConfig.from_spec(f.spec), f.hits, refl, gp, gf, with_abs=True)
        o_refl += a
        c_refl += ca
        o_par[r] += b
        c_par[r] += cb
    assert_grad_cond(g_refl, o_refl, c_refl, what="refl")
    for r in range(4):
        assert_grad_cond(g_par[r, :5], o_par[r], c_par[r], what="row %d" % r)
    assert np.all(g_par[:, 5:] == 0)


@pytest.mark.parametrize("n_az", [1, 2, 3, 4, 5, 7, 8, 12, 62, 64, 100, 252, 255, 256, 257, 1000, 1001, 1022, 2047, 4095])
def test_groups_of_four_bins_and_range_rows(n_az):
    """The additive term is drawn for groups of four bins: rows whose length is
    a multiple of four (a group lies in one row) and lengths around it (groups
    over two or more rows), in frames without and with returns."""
    n_range = max(3, 6000 // n_az)
    st = W.Stream(1450, n_az)
    specs = [W.SonarSpec(r_min=0.5, r_max=10.0, n_range=n_range, n_azimuth=n_az, speckle_mode=mode, sigma_sa=0.3,
                         sigma_phi=0.4, sigma_sm=0.1, gamma_k=2, seed_lo=n_az, frame_id=k, alpha=0.05)
             for k, mode in enumerate((W.SPECKLE_PAPER, W.SPECKLE_GAMMA))]
    frames, refl = merged([W.SonarFrame(s, W.make_hits(st, s, n, n_materials=4)) for s, n in zip(specs, (1, 3000))])
    got = gpu_forward(frames, refl, fan=False)
    for k, f in enumerate(frames):
        check_frame(got[k], oracle_forward(f, refl), "n_az %d frame %d" % (n_az, k), fan=False)
    gpol = [W.loss_weights((1451, k), (n_range, n_az)) for k in range(2)]
    g_refl, g_par = gpu_backward(frames, refl, gpol, [None, None])
    o_refl, o_par, c_refl, c_par = oracle_backward(frames, refl, gpol, [None, None])
    assert_grad_cond(g_refl, o_refl, c_refl, what="refl")
    assert_grad_cond(g_par[0, :5], o_par, c_par, what="params")


@pytest.mark.parametrize("blocks", [1, 2, 15, 16, 17, 255, 256, 257, 511, 3839, 3840, 3841, 4095, 4096, 4097, 4352])
def test_water_gradient_sums_of_any_number_of_partials(blocks):
    """Constant images of `blocks` workgroups of 2048 pixels, on two parameter
    rows: every partial sum is the same, so a partial missed or taken twice by
    the reduction shows as 1 / blocks of the result (the pixels' FP32 terms are
    within 1e-6 of theirs)."""
    import torch
    osm = _osm()
    bd, bb, bi = (0.125, 0.25, 0.5), (0.0625, 0.25, 0.375), (0.5, 0.25, 0.75)
    wt = osm.water_params([(bd, bb, bi), (bb, bd, bi)])
    J = torch.full((3, blocks, 2048), 0.5, device="cuda")
    d = torch.full((blocks, 2048), 2.0, device="cuda")
    J1, d1 = torch.full((3, 1, 5), 0.5, device="cuda"), torch.full((1, 5), 2.0, device="cuda")
    g_w, _, _ = osm.uw_form_backward([J, J1], [d, d1], wt, [torch.ones_like(J), torch.ones_like(J1)], rows=[0, 1],
                                     want_image_grads=False)
    got = g_w.cpu().numpy().astype(np.float64)
    for row, n, (a, b) in ((0, blocks * 2048, (bd, bb)), (1, 5, (bb, bd))):
        a, b, i = np.array(a), np.array(b), np.array(bi)
        want = n * np.concatenate([-0.5 * 2.0 * np.exp(-2.0 * a), i * 2.0 * np.exp(-2.0 * b), 1.0 - np.exp(-2.0 * b)])
        assert np.all(np.abs(got[row] - want) <= 2e-6 * np.abs(want)), (got[row], want)


@pytest.mark.parametrize("n_az", [2, 64, 511, 1024, 2047, 2048, 2857, 2858, 4096])
@pytest.mark.parametrize("fov", [0.05, 2.0943951, 3.1415925])
def test_returns_at_azimuth_edges(n_az, fov):
    """Returns from 1e-9 to 1e-2 cells off the azimuth edges, inside and outside
    the distance below which the FP32 azimuth is redone in FP64 (7e-7 n_az
    cells): the oracle's bins, exactly."""
    st = W.Stream(1470, n_az)
    n = 60000
    spec = W.SonarSpec(r_min=0.5, r_max=40.0, n_range=16, n_azimuth=n_az, fov_az=fov, fov_el=0.5,
                       speckle_mode=W.SPECKLE_OFF, alpha=0.02)
    half, scale = 0.5 * np.float64(np.float32(fov)), n_az / np.float64(np.float32(fov))
    edge = st.integers(0, n_az, n)
    off = 10.0 ** st.uniform(-9.0, -2.0, n) * np.where(st.integers(0, 1, n) == 1, 1.0, -1.0)
    phi, r = (edge + off) / scale - half, st.uniform(0.6, 39.0, n)
    el = st.uniform(-0.2, 0.2, n)
    x, y, z = r * np.cos(el) * np.cos(phi), r * np.cos(el) * np.sin(phi), r * np.sin(el)
    nrm = np.stack([st.uniform(-1.0, 1.0, n) for _ in range(3)])
    nrm[:, ::7] *= 1e-15   # normals of any length
    nrm[:, 1::7] *= 1e15
    nrm[:, 2::97] = 0.0
    f32 = lambda a: np.asarray(a, np.float32)
    hits = W.SonarHits(x=f32(x), y=f32(y), z=f32(z), nx=f32(nrm[0]), ny=f32(nrm[1]), nz=f32(nrm[2]),
                       mat=st.integers(0, 3, n).astype(np.int32), refl=f32([0.2, 0.5, 0.8, 1.0]))
    got = gpu_forward([W.SonarFrame(spec, hits)], hits.refl, fan=False)[0]
    check_frame(got, oracle_forward(W.SonarFrame(spec, hits), hits.refl), "n_az %d fov %g" % (n_az, fov), fan=False)
