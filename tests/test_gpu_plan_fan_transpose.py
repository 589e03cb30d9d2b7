"""GPU parity of a backward plan's transposed fan operators (built once at
plan creation from the fan kernel's stencils; the backward gathers each polar
bin's fan gradient through them), against the FP64 oracle, on odd and
degenerate grids, mixed frames, growing gradient magnitudes and a NaN.
"""
import sys

import numpy as np
import pytest

import oracle
from oracle import SonarConfig
import workloads as W
from _tol import assert_grad_cond

pytestmark = pytest.mark.gpu


def _say(msg):
    print("[case] " + msg, flush=True)
    sys.stdout.flush()


def _plan_backward(frames, refl, gpol, gfan, rows=None, graph=False):
    """Plan forward + backward; gradients as float64 numpy arrays."""
    import torch
    import paper_2503_01074_amd as osm
    rows = rows or [0] * len(frames)
    geoms = [osm.SonarGeometry.from_spec(f.spec, param_row=r) for f, r in zip(frames, rows)]
    hits = [osm.DeviceHits.from_host(f.hits) for f in frames]
    row_spec = {r: f.spec for f, r in zip(frames, rows)}
    params = osm.sonar_params([osm.sonar_params_from_spec(row_spec[r]) for r in range(max(rows) + 1)])
    plan = osm.Plan(list(zip(geoms, hits)), sonar_params=params, refl=torch.as_tensor(refl).cuda(),
                    backward=True, graph=graph)
    assert plan.shape()["bwd_block_bins"] in (256, 512, 1024)
    for o, gp, gf in zip(plan.sonar_out, gpol, gfan):
        if "grad_polar" in o:
            o["grad_polar"].copy_(torch.as_tensor(gp))
        if "grad_fan" in o:
            o["grad_fan"].copy_(torch.as_tensor(gf) if gf is not None else torch.zeros_like(o["grad_fan"]))
    plan.forward()
    plan.backward()
    torch.cuda.synchronize()
    g_refl = plan.grad_refl.cpu().numpy().astype(np.float64)
    g_par = plan.grad_sonar_params.cpu().numpy().astype(np.float64)
    plan.close()
    return g_refl, g_par


def _oracle(frames, refl, gpol, gfan, rows=None):
    rows = rows or [0] * len(frames)
    n_rows = max(rows) + 1
    o_refl, c_refl = np.zeros(refl.shape[0]), np.zeros(refl.shape[0])
    o_par, c_par = np.zeros((n_rows, 5)), np.zeros((n_rows, 5))
    for f, r, gp, gf in zip(frames, rows, gpol, gfan):
        a, b, _, ca, cb = oracle.sonar_backward(SonarConfig.from_spec(f.spec), f.hits, refl, gp, gf, with_abs=True)
        o_refl += a
        c_refl += ca
        o_par[r] += b
        c_par[r] += cb
    return o_refl, o_par, c_refl, c_par


def _frame(st, Nr, Np, H, Wd, n, mode=W.SPECKLE_PAPER, frame_id=0, r_max=13.0):
    spec = W.SonarSpec(r_min=0.7, r_max=r_max, n_range=Nr, n_azimuth=Np, fan_h=H, fan_w=Wd, speckle_mode=mode,
                       gamma_k=3, sigma_sm=0.12, sigma_sa=0.15, sigma_phi=0.3, alpha=0.09, gain=1.2, seed_lo=3,
                       frame_id=frame_id)
    return W.SonarFrame(spec, W.make_hits(st, spec, n, n_materials=5))


@pytest.mark.parametrize("shape", [(37, 29, 41, 83), (1, 17, 8, 16), (23, 1, 9, 9), (60, 40, 33, 64),
                                   (300, 700, 64, 128), (24, 1, 10, 20), (2, 2, 12, 30)])
@pytest.mark.parametrize("graph", [False, True])
def test_plan_fan_transpose_vs_oracle(shape, graph):
    """Odd fan width (a centre column that is its own mirror: plain operator
    rows), even widths (mirrored rows) with an odd azimuth count (a middle
    column that is its own mirror), one range row, one or two azimuth columns,
    more bins than fan pixels."""
    Nr, Np, H, Wd = shape
    _say("plan fan transpose %s graph %s" % (shape, graph))
    st = W.Stream(8100, Nr + Np)
    frames = [_frame(st, Nr, Np, H, Wd, 3000)]
    refl = frames[0].hits.refl
    gpol = [W.loss_weights((8101, 1), (Nr, Np))]
    gfan = [W.loss_weights((8101, 2), (H, Wd))]
    g_refl, g_par = _plan_backward(frames, refl, gpol, gfan, graph=graph)
    o_refl, o_par, c_refl, c_par = _oracle(frames, refl, gpol, gfan)
    assert_grad_cond(g_refl, o_refl, c_refl, what="refl")
    assert_grad_cond(g_par[0, :5], o_par[0], c_par[0], what="params")
    assert np.all(g_par[0, 5:] == 0)


def test_plan_fan_transpose_mixed_frames_and_rows():
    """Frames with a fan, without one, and with a fan whose gradient is zero,
    on three parameter rows and all speckle modes, in one plan."""
    _say("plan fan transpose: mixed frames on three rows")
    st = W.Stream(8200, 1)
    frames = [
        _frame(st, 48, 40, 40, 72, 3000, W.SPECKLE_GAMMA, 0),
        _frame(st, 30, 24, 0, 0, 1500, W.SPECKLE_PAPER, 1),
        _frame(st, 61, 53, 51, 91, 4000, W.SPECKLE_OFF, 2, r_max=9.0),
        _frame(st, 20, 300, 64, 129, 2500, W.SPECKLE_GAMMA, 3),
    ]
    rows = [0, 1, 2, 0]
    refl = frames[0].hits.refl
    for f in frames:
        f.hits.refl = refl
    gpol = [W.loss_weights((8201, k), (f.spec.n_range, f.spec.n_azimuth)) for k, f in enumerate(frames)]
    gfan = [W.loss_weights((8202, k), (f.spec.fan_h, f.spec.fan_w)) if f.spec.fan_h else None
            for k, f in enumerate(frames)]
    gfan[2] = np.zeros((frames[2].spec.fan_h, frames[2].spec.fan_w), np.float32)
    g_refl, g_par = _plan_backward(frames, refl, gpol, gfan, rows)
    o_refl, o_par, c_refl, c_par = _oracle(frames, refl, gpol, gfan, rows)
    assert_grad_cond(g_refl, o_refl, c_refl, what="refl")
    for r in range(3):
        assert_grad_cond(g_par[r, :5], o_par[r], c_par[r], what="row %d" % r)


def test_plan_fan_transpose_growing_magnitudes():
    """A tall fan whose gradient magnitude spans nine decades down the image:
    each bin's FP64 sum keeps the small terms."""
    _say("plan fan transpose: 1400 x 2800 fan, growing gradient magnitude")
    st = W.Stream(8300, 1)
    spec = W.SonarSpec(r_min=0.5, r_max=30.0, n_range=300, n_azimuth=200, fan_h=1400, fan_w=2800,
                       alpha=0.08, gain=1.1, sigma_phi=0.3, sigma_sa=0.15, speckle_mode=W.SPECKLE_GAMMA,
                       seed_lo=5, frame_id=1)
    frames = [W.SonarFrame(spec, W.make_hits(st, spec, 20000, n_materials=16))]
    refl = frames[0].hits.refl
    ramp = np.logspace(-6, 3, spec.fan_h)[:, None]
    gfan = [(W.loss_weights((8301, 2), (spec.fan_h, spec.fan_w)) * ramp).astype(np.float32)]
    gpol = [W.loss_weights((8301, 3), (spec.n_range, spec.n_azimuth))]
    g_refl, g_par = _plan_backward(frames, refl, gpol, gfan)
    o_refl, o_par, c_refl, c_par = _oracle(frames, refl, gpol, gfan)
    assert_grad_cond(g_refl, o_refl, c_refl, what="refl")
    assert_grad_cond(g_par[0, :5], o_par[0], c_par[0], what="params")


def test_plan_fan_transpose_nan_gradient():
    """A NaN in the fan gradient reaches the same outputs as in the oracle."""
    _say("plan fan transpose: a NaN in the fan gradient")
    st = W.Stream(8400, 1)
    frames = [_frame(st, 48, 40, 40, 72, 3000, W.SPECKLE_GAMMA)]
    refl = frames[0].hits.refl
    gpol = [W.loss_weights((8401, 1), (48, 40))]
    gfan = [W.loss_weights((8401, 2), (40, 72)).copy()]
    gfan[0][20, 30] = np.nan
    g_refl, g_par = _plan_backward(frames, refl, gpol, gfan)
    o_refl, o_par, _, _ = _oracle(frames, refl, gpol, gfan)
    np.testing.assert_array_equal(np.isnan(g_refl), np.isnan(o_refl))
    np.testing.assert_array_equal(np.isnan(g_par[0, :5]), np.isnan(o_par[0]))
    assert np.isnan(o_par).any()


@pytest.mark.parametrize("n_frames,n_bins,block_bins,mixed,odd_az", [(3, 1024, 512, True, False),
                                                                      (4, 2048, 1024, True, False),
                                                                      (3, 1024, 512, False, False),
                                                                      (4, 2048, 1024, False, False),
                                                                      (3, 1024, 512, True, True),
                                                                      (4, 2048, 1024, True, True)])
def test_plan_fan_transpose_large_batches(n_frames, n_bins, block_bins, mixed, odd_az):
    """Batches of many polar bins take two or four rows per thread (the
    workgroup's wave spans then cover 128 or 256 rows and several chunks);
    even and odd fan widths alternate (mirrored and plain operator rows in one
    launch), or all widths are odd (plain rows only: the kernel without
    mirror outputs); with odd azimuth counts a thread's mirrored rows wrap
    from one range row to the next around a middle column that is its own
    mirror."""
    import paper_2503_01074_amd as osm
    _say("plan fan transpose: %d frames of %d x %d bins, mixed layouts %s, odd azimuth counts %s"
         % (n_frames, n_bins, n_bins, mixed, odd_az))
    st = W.Stream(8500 + n_bins, n_frames)
    frames = []
    for k in range(n_frames):
        spec = W.SonarSpec(r_min=0.5, r_max=12.0 + k, n_range=n_bins, n_azimuth=n_bins + 8 * k + (1 if odd_az else 0), fan_h=150 + 10 * k,
                           fan_w=300 + 21 * k if mixed else 301 + 20 * k, alpha=0.09, gain=1.2, sigma_phi=0.3, sigma_sa=0.15, sigma_sm=0.12,
                           speckle_mode=(W.SPECKLE_GAMMA, W.SPECKLE_PAPER, W.SPECKLE_OFF)[k % 3], gamma_k=3,
                           seed_lo=3, frame_id=k)
        frames.append(W.SonarFrame(spec, W.make_hits(st, spec, 3000, n_materials=5)))
    refl = frames[0].hits.refl
    for f in frames:
        f.hits.refl = refl
    gpol = [W.loss_weights((8501, k), (f.spec.n_range, f.spec.n_azimuth)) for k, f in enumerate(frames)]
    gfan = [W.loss_weights((8502, k), (f.spec.fan_h, f.spec.fan_w)) for k, f in enumerate(frames)]
    import torch
    geoms = [osm.SonarGeometry.from_spec(f.spec) for f in frames]
    hits = [osm.DeviceHits.from_host(f.hits) for f in frames]
    params = osm.sonar_params([osm.sonar_params_from_spec(frames[0].spec)])
    plan = osm.Plan(list(zip(geoms, hits)), sonar_params=params, refl=torch.as_tensor(refl).cuda(), backward=True)
    assert plan.shape()["bwd_block_bins"] == block_bins
    for o, gp, gf in zip(plan.sonar_out, gpol, gfan):
        o["grad_polar"].copy_(torch.as_tensor(gp))
        o["grad_fan"].copy_(torch.as_tensor(gf))
    plan.forward()
    plan.backward()
    torch.cuda.synchronize()
    g_refl = plan.grad_refl.cpu().numpy().astype(np.float64)
    g_par = plan.grad_sonar_params.cpu().numpy().astype(np.float64)
    plan.close()
    o_refl, o_par, c_refl, c_par = _oracle(frames, refl, gpol, gfan)
    assert_grad_cond(g_refl, o_refl, c_refl, what="refl")
    assert_grad_cond(g_par[0, :5], o_par[0], c_par[0], what="params")


@pytest.mark.parametrize("fan", [(96, 200), (96, 201)])
def test_frames_of_one_geometry_share_an_operator(fan):
    """Frames of the same fan geometry read one operator; one that differs in
    a single field (range, grid or fan) has its own."""
    st = W.Stream(8600 + fan[1], 0)
    H, Wd = fan
    frames = [_frame(st, 60, 50, H, Wd, 2000, frame_id=0), _frame(st, 60, 50, H, Wd, 1500, frame_id=1, mode=W.SPECKLE_GAMMA),
              _frame(st, 60, 50, H, Wd, 1000, frame_id=2, r_max=14.0), _frame(st, 60, 50, H + 1, Wd, 1000, frame_id=3),
              _frame(st, 60, 51, H, Wd, 1000, frame_id=4), _frame(st, 60, 50, H, Wd, 700, frame_id=5),
              _frame(st, 60, 50, H, Wd + 1, 900, frame_id=6)]
    refl = frames[0].hits.refl
    for f in frames:
        f.hits.refl = refl
    gpol = [W.loss_weights((8601, k), (f.spec.n_range, f.spec.n_azimuth)) for k, f in enumerate(frames)]
    gfan = [W.loss_weights((8602, k), (f.spec.fan_h, f.spec.fan_w)) for k, f in enumerate(frames)]
    g_refl, g_par = _plan_backward(frames, refl, gpol, gfan)
    o_refl, o_par, c_refl, c_par = _oracle(frames, refl, gpol, gfan)
    assert_grad_cond(g_refl, o_refl, c_refl, what="refl")
    assert_grad_cond(g_par[0, :5], o_par[0], c_par[0], what="params")


@pytest.mark.parametrize("n_bins,side,block_bins", [(1024, 300, 512), (1024, 800, 256), (2048, 400, 1024),
                                                    (2048, 900, 512), (2048, 1100, 256)])
def test_operator_rows_per_thread_follow_the_fan_density(n_bins, side, block_bins):
    """Large batches take several operator rows per thread only where the
    fan has few pixels per polar bin."""
    import torch
    import paper_2503_01074_amd as osm
    st = W.Stream(8700 + n_bins, side)
    n = 4
    spec = W.SonarSpec(r_min=0.5, r_max=12.0, n_range=n_bins, n_azimuth=n_bins, fan_h=side, fan_w=2 * side,
                       speckle_mode=W.SPECKLE_OFF, alpha=0.09)
    hits = W.make_hits(st, spec, 2000, n_materials=5)
    g, h = osm.SonarGeometry.from_spec(spec), osm.DeviceHits.from_host(hits)
    gpol = W.loss_weights((8701, side), (n_bins, n_bins))
    gfan = W.loss_weights((8702, side), (side, 2 * side))
    params = osm.sonar_params([osm.sonar_params_from_spec(spec)])
    plan = osm.Plan([(g, h)] * n, sonar_params=params, refl=torch.as_tensor(hits.refl).cuda(), backward=True)
    assert plan.shape()["bwd_block_bins"] == block_bins
    for o in plan.sonar_out:
        o["grad_polar"].copy_(torch.as_tensor(gpol))
        o["grad_fan"].copy_(torch.as_tensor(gfan))
    plan.forward()
    plan.backward()
    torch.cuda.synchronize()
    g_refl = plan.grad_refl.cpu().numpy().astype(np.float64) / n
    plan.close()
    o_refl, _, c_refl, _ = _oracle([W.SonarFrame(spec, hits)], hits.refl, [gpol], [gfan])
    assert_grad_cond(g_refl, o_refl, c_refl, what="refl")


@pytest.mark.parametrize("n_range,n_az", [(3, 62), (5, 63), (5, 64), (4, 65), (3, 124), (4, 125), (5, 126), (4, 127),
                                          (5, 128), (2, 253), (3, 504), (7, 505), (64, 3), (90, 2)])
@pytest.mark.parametrize("fan", [(50, 120), (50, 121), (7, 10)])
def test_cells_at_wave_and_workgroup_edges(n_range, n_az, fan):
    """A wave takes 63 operator rows and the cell before them: range rows (and
    mirrored halves of them) of just under, exactly and just over that many
    rows, ends of waves and workgroups within a range row and between two, and
    fans with many and with hardly any pixels per bin."""
    st = W.Stream(8800 + n_az, n_range)
    H, Wd = fan
    frames = [_frame(st, n_range, n_az, H, Wd, 1500), _frame(st, n_range, n_az, H + 3, Wd, 900, frame_id=1,
                                                            mode=W.SPECKLE_GAMMA, r_max=11.0)]
    refl = frames[0].hits.refl
    for f in frames:
        f.hits.refl = refl
    gpol = [W.loss_weights((8801, k), (n_range, n_az)) for k in range(2)]
    gfan = [W.loss_weights((8802, k), (f.spec.fan_h, f.spec.fan_w)) for k, f in enumerate(frames)]
    g_refl, g_par = _plan_backward(frames, refl, gpol, gfan)
    o_refl, o_par, c_refl, c_par = _oracle(frames, refl, gpol, gfan)
    assert_grad_cond(g_refl, o_refl, c_refl, what="refl")
    assert_grad_cond(g_par[0, :5], o_par[0], c_par[0], what="params")


def test_unused_fan_gradient_stays_in_its_cell():
    """A fan pixel's gradient reaches its own bins alone, also where the next
    lane, wave or range row sums beside it: bins that no fan pixel of a NaN
    gradient reads keep their gradient exactly."""
    import torch
    import paper_2503_01074_amd as osm
    st = W.Stream(8900, 1)
    for n_range, n_az, Wd in ((6, 126, 140), (6, 126, 141), (5, 64, 90), (40, 3, 30)):
        f = _frame(st, n_range, n_az, 40, Wd, 4000, mode=W.SPECKLE_OFF)
        # every return its own material: the gradient of a reflectivity is its bin's
        f.hits.mat[:] = np.arange(len(f.hits.mat))
        refl = np.full((len(f.hits.mat),), 0.5, np.float32)
        gfan = W.loss_weights((8901, n_az), (40, Wd))
        got = []
        for v, u in ((None, None), (20, 3), (20, Wd - 4), (33, Wd // 2), (12, Wd // 4)):
            g = gfan.copy()
            if v is not None:
                g[v, u] = np.nan
            plan = osm.Plan([(osm.SonarGeometry.from_spec(f.spec), osm.DeviceHits.from_host(f.hits))],
                            sonar_params=osm.sonar_params([osm.sonar_params_from_spec(f.spec)]),
                            refl=torch.as_tensor(refl).cuda(), backward=True, bins=True)
            plan.sonar_out[0]["grad_polar"].zero_()
            plan.sonar_out[0]["grad_fan"].copy_(torch.as_tensor(g))
            plan.forward()
            plan.backward()
            torch.cuda.synchronize()
            got.append((plan.grad_refl.cpu().numpy(), plan.sonar_out[0]["bins"].cpu().numpy()))
            plan.close()
        base, bins = got[0]
        assert np.isfinite(base).all()
        for g, _ in got[1:]:
            bad = ~np.isfinite(g)
            hit = np.unique(bins[bad])
            # one pixel's stencil: two neighbouring columns of two range rows
            assert len(hit) <= 4 and (len(hit) == 0 or (hit % n_az).max() - (hit % n_az).min() <= 1)
            assert (np.unique(hit // n_az).size <= 2)
            np.testing.assert_array_equal(g[~bad], base[~bad])


@pytest.mark.parametrize("n_range,n_az,Wd", [(6, 126, 140), (6, 127, 141), (5, 64, 90), (9, 31, 77), (40, 3, 30),
                                             (40, 126, 140), (30, 127, 141)])
def test_fan_gradient_reaches_exactly_its_stencil(n_range, n_az, Wd):
    """One return in the middle of every bin, each its own material: a NaN in
    one fan pixel's gradient makes exactly the reflectivity gradients of the
    bins of its stencil non-finite (those that the oracle's adjoint of that
    pixel alone fills; bins of weight zero may join them) and changes no other.
    Pixels of cells in all columns, at both ends of a wave's 63 operator rows,
    at the mirrored half's last columns, and outside the sector."""
    import torch
    import paper_2503_01074_amd as osm
    H = 100
    spec = W.SonarSpec(r_min=1.0, r_max=9.0, n_range=n_range, n_azimuth=n_az, fan_h=H, fan_w=Wd,
                       speckle_mode=W.SPECKLE_OFF)
    cfg = SonarConfig.from_spec(spec)
    b = np.arange(n_range * n_az)
    r = spec.r_min + (b // n_az + 0.5) * (spec.r_max - spec.r_min) / n_range
    phi = ((b % n_az + 0.5) / n_az - 0.5) * spec.fov_az
    x, y, z = (r * np.cos(phi)).astype(np.float32), (r * np.sin(phi)).astype(np.float32), np.zeros(len(b), np.float32)
    hits = W.SonarHits(x=x, y=y, z=z, nx=-x, ny=-y, nz=z.copy(), mat=b.astype(np.int32),
                       refl=np.full(len(b), 0.5, np.float32))
    plan = osm.Plan([(osm.SonarGeometry.from_spec(spec), osm.DeviceHits.from_host(hits))],
                    sonar_params=osm.sonar_params([osm.sonar_params_from_spec(spec)]),
                    refl=torch.as_tensor(hits.refl).cuda(), backward=True, bins=True)
    plan.sonar_out[0]["grad_polar"].zero_()
    g = torch.as_tensor(W.loss_weights((8911, n_az), (H, Wd))).cuda()
    grad_fan = plan.sonar_out[0]["grad_fan"]

    def gradient():
        plan.backward()
        torch.cuda.synchronize()
        return plan.grad_refl.cpu().numpy()

    grad_fan.copy_(g)
    plan.forward()
    base = gradient()
    np.testing.assert_array_equal(plan.sonar_out[0]["bins"].cpu().numpy(), b)
    assert np.isfinite(base).all()
    # cells of the fan's pixels: first range row and column, from images of the row and column index
    ones, _ = oracle.fan_forward(cfg, np.ones((n_range, n_az)))
    inside = ones > 0.5
    i0, j0 = (np.floor(oracle.fan_forward(cfg, im)[0] + 1e-9).astype(int) for im in
              (np.repeat(np.arange(n_range), n_az).reshape(n_range, n_az), np.tile(np.arange(n_az), (n_range, 1))))
    ncol = (n_az + 1) // 2 if Wd % 2 == 0 else n_az
    row = np.where(inside & (j0 < ncol), i0 * ncol + j0, -1)
    pixels = [np.argwhere(inside & (j0 == j)) for j in range(n_az)]                # every column
    pixels += [np.argwhere((row >= 0) & (row % 63 == k)) for k in (0, 1, 61, 62)]   # around the ends of a wave
    pixels += [np.argwhere(inside & (i0 == i) & (j0 >= ncol - 2) & (j0 <= ncol)) for i in range(n_range)]
    pixels += [np.argwhere(~inside)]
    assert len(pixels[0]) and len(pixels[max(n_az - 2, 0)]) and (n_range * ncol < 63 or all(map(len, pixels[n_az:n_az + 4])))
    for v, u in np.unique(np.concatenate([q[[0, len(q) // 2, -1]] for q in pixels if len(q)]), axis=0):
        delta = np.zeros((H, Wd), np.float32)
        delta[v, u] = 1.0
        want = np.flatnonzero(oracle.fan_adjoint(cfg, delta).reshape(-1))
        grad_fan[v, u] = float("nan")
        got = gradient()
        grad_fan[v, u] = g[v, u]
        bad = np.flatnonzero(~np.isfinite(got))
        assert np.isin(want, bad).all(), (v, u)
        if len(want) == 0:
            assert len(bad) == 0, (v, u)
            continue
        assert len(bad) <= 4, (v, u)
        for near, have in ((want // n_az, bad // n_az), (want % n_az, bad % n_az)):
            assert have.min() >= near.max() - 1 and have.max() <= near.min() + 1, (v, u)
        fine = np.setdiff1d(b, bad)
        np.testing.assert_array_equal(got[fine], base[fine])
    plan.close()
