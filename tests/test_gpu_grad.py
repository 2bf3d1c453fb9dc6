"""GPU parity of the adjoint (d/dmap, the transposed gather) and of the knot
gradient (hat-basis gather) against the FP64 oracle's gradients, whose own
correctness is pinned by exact central differences in the CPU suite."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import REL_RMS_TOL, assert_tie_free, log, rel_rms, to_dev, to_host

pytestmark = pytest.mark.gpu


def _A():
    import paper_1211_3556_amd as A
    return A


def _sync():
    import torch
    torch.cuda.synchronize()


@pytest.mark.parametrize("nside,nb,tc_deg,nk", [(32, 3, 10.3, 64), (24, 1, 40.3, 200),
                                                 (16, 8, 99.3, 33)])
def test_gradients_full_maps(nside, nb, tc_deg, nk):
    tc = np.radians(tc_deg)
    assert_tie_free(nside, tc)
    knots = W.gaussian_profile_knots(tc / 3, tc, nk)
    x = W.white_noise(nside, 600, nbatch=nb)
    g = W.white_noise(nside, 700, nbatch=nb)
    A = _A()
    plan = A.Plan(nside, tc, ntab=nk, max_batch=nb, learnable=True)
    plan.set_knots(to_dev(knots))
    log("gradients Nside %d batch %d" % (nside, nb))
    gx, gk = plan.backward(to_dev(g), to_dev(x), want_map=True, want_knots=True)
    _sync()
    gx, gk = to_host(gx), to_host(gk)
    gk_ref = sum(O.knot_grad(nside, tc, nk, x[b], g[b]) for b in range(nb))
    for b in range(nb):
        assert rel_rms(gx[b], O.map_grad(nside, tc, knots, g[b])) <= REL_RMS_TOL
    assert np.max(np.abs(gk - gk_ref)) <= 1e-5 * np.abs(gk_ref).max()
    assert rel_rms(gk, gk_ref) <= 1e-6
    # knot gradient alone, and map gradient alone, agree with the fused call
    _, gk2 = plan.backward(to_dev(g), to_dev(x), want_map=False, want_knots=True)
    gx2, _ = plan.backward(to_dev(g), None, want_map=True, want_knots=False)
    _sync()
    assert rel_rms(to_host(gk2), gk_ref) <= 1e-6
    assert np.array_equal(to_host(gx2), gx)


@pytest.mark.parametrize("nside,tc_deg,nk", [(16, 74.7, 33), (40, 7.0, 257), (100, 3.31, 64),
                                             (16, 0.5, 16)])
def test_knot_gradient_map_groups(nside, tc_deg, nk):
    """The knot gradient of plans for 1, 2 and 6 maps (groups of one, two and four,
    the last one partial, and the tiles' chunks split between workgroups) called
    with every number of maps up to their limit."""
    A = _A()
    tc = np.radians(tc_deg)
    assert_tie_free(nside, tc)
    x = W.white_noise(nside, 610, nbatch=6)
    g = W.white_noise(nside, 710, nbatch=6)
    each = np.stack([O.knot_grad(nside, tc, nk, x[b], g[b]) for b in range(6)])
    for mb in (1, 2, 6):
        plan = A.Plan(nside, tc, ntab=nk, max_batch=mb, learnable=True)
        plan.set_knots(to_dev(W.gaussian_profile_knots(tc / 3, tc, nk)))
        for nb in range(1, mb + 1):
            _, gk = plan.backward(to_dev(g[:nb]), to_dev(x[:nb]), want_map=False,
                                  want_knots=True)
            _sync()
            ref = each[:nb].sum(axis=0)
            assert np.max(np.abs(to_host(gk) - ref)) <= 1e-5 * np.abs(ref).max(), (mb, nb)
            assert rel_rms(to_host(gk), ref) <= 1e-6, (mb, nb)


def test_learnable_plan_of_any_batch_limit():
    """Creating a learnable plan does not take longer with max_batch: the knot
    gradient's partial rows are bounded by the device, not counted map by map."""
    import time
    A = _A()
    log("learnable plan max_batch 700000000")
    A.Plan(1, 1.0, ntab=16, learnable=True)
    t = time.perf_counter()
    A.Plan(1, 1.0, ntab=16, max_batch=700_000_000, learnable=True)
    assert time.perf_counter() - t < 0.2


@pytest.mark.parametrize("nside,tc_deg,nb", [(64, 22.1, 3), (64, 22.1, 4), (64, 22.1, 5)])
def test_knot_gradient_on_both_sides_of_the_map_group_line(nside, tc_deg, nb):
    """Calls with little work sum the maps one by one, others in groups (the line
    lies between these): the gradient of several maps is that of the maps' sum."""
    A = _A()
    tc = np.radians(tc_deg)
    nk = 129
    assert_tie_free(nside, tc)
    x = W.white_noise(nside, 611, nbatch=nb)
    g = W.white_noise(nside, 711, nbatch=nb)
    plan = A.Plan(nside, tc, ntab=nk, max_batch=nb, learnable=True)
    plan.set_knots(to_dev(W.gaussian_profile_knots(tc / 3, tc, nk)))
    log("knot gradient map groups Nside %d %d maps" % (nside, nb))
    _, gk = plan.backward(to_dev(g), to_dev(x), want_map=False, want_knots=True)
    _sync()
    ref = sum(O.knot_grad(nside, tc, nk, x[b], g[b]) for b in range(nb))
    assert np.max(np.abs(to_host(gk) - ref)) <= 1e-5 * np.abs(ref).max()
    assert rel_rms(to_host(gk), ref) <= 1e-6


@pytest.mark.parametrize("nside,tc_deg,nb,nk,kw", [
    (200, 5.6, 3, 64, {}), (200, 5.6, 7, 257, dict(biased=True)),   # 200 / 2 pixels, two groups
    (256, 5.6, 4, 1700, dict(rings=(3, 300))),                      # three maps a group, a ring range
    (100, 12.0, 6, 33, dict(rings=(20, 171))), (100, 12.0, 8, 300, {}),
    (64, 30.0, 4, 65, {}), (64, 60.0, 3, 129, {}), (64, 91.0, 5, 64, {})])   # whole rings
def test_knot_gradient_of_map_groups_equals_single_maps(nside, tc_deg, nb, nk, kw):
    """Calls with enough work for the several-map form, over its angle series, tile
    shapes and group sizes: the sum of the single-map calls (the per-map form), whose
    FP32 results round to half an ulp each."""
    A = _A()
    tc = np.radians(tc_deg)
    x = to_dev(W.white_noise(nside, 612, nbatch=nb))
    g = to_dev(W.white_noise(nside, 712, nbatch=nb))
    plan = A.Plan(nside, tc, ntab=nk, max_batch=nb, learnable=True, **kw)
    plan.set_knots(to_dev(W.gaussian_profile_knots(tc / 3, tc, nk)))
    log("knot gradient of map groups Nside %d, %g deg, %d maps" % (nside, tc_deg, nb))
    _, gk = plan.backward(g, x, want_map=False, want_knots=True)
    each = [to_host(plan.backward(g[b], x[b], want_map=False, want_knots=True)[1])
            for b in range(nb)]
    assert rel_rms(to_host(gk), np.sum(each, axis=0)) <= 1e-6


def test_autograd_function_and_loss():
    """The torch.autograd.Function path on the c5 loss L = sum (conv(x) - t)^2 at
    a reduced Nside: gradients match the oracle's."""
    import torch
    A = _A()
    spec = W.C5
    nside, nb = 128, 2
    tc = spec.theta_cut * 8     # same number of pixels per disc radius as at Nside 1024
    knots = W.gaussian_profile_knots(spec.fwhm * 8, tc, spec.nknots)
    target_knots = W.gaussian_profile_knots(spec.target_fwhm * 8, tc, spec.nknots)
    x = W.white_noise(nside, spec.seed0, nbatch=nb)
    t = np.stack([O.convolve(nside, tc, target_knots, x[b]) for b in range(nb)])
    y_ref = np.stack([O.convolve(nside, tc, knots, x[b]) for b in range(nb)])
    g_ref = 2.0 * (y_ref - t)
    gx_ref = np.stack([O.map_grad(nside, tc, knots, g_ref[b]) for b in range(nb)])
    gk_ref = sum(O.knot_grad(nside, tc, spec.nknots, x[b], g_ref[b]) for b in range(nb))

    plan = A.Plan(nside, tc, ntab=spec.nknots, max_batch=nb, learnable=True)
    xd = to_dev(x).requires_grad_(True)
    kd = to_dev(knots).requires_grad_(True)
    log("autograd loss")
    y = A.conv(xd, plan, kd)
    loss = torch.sum((y.double() - torch.from_numpy(t).cuda()) ** 2)
    loss.backward()
    _sync()
    assert rel_rms(to_host(y), y_ref) <= REL_RMS_TOL
    # g = 2 (y - t) carries the FP32 forward error into both gradients
    assert rel_rms(to_host(xd.grad), gx_ref) <= 1e-5
    assert np.max(np.abs(to_host(kd.grad) - gk_ref)) <= 1e-4 * np.abs(gk_ref).max()


def test_c5_full_size_sampled_and_identities():
    """Nside 1024, 8 maps, 256 learnable knots, theta_cut 30 arcmin, in the
    benchmark's launch configuration: the adjoint at sampled pixels against
    the oracle, and the Euler identities <K, dL/dK> = <g, y> = <x, A g>,
    which hold at any size, for the knot gradient."""
    spec = W.C5
    A = _A()
    knots = W.gaussian_profile_knots(spec.fwhm, spec.theta_cut, spec.nknots)
    x = W.white_noise(spec.nside, spec.seed0, nbatch=spec.nbatch)
    g = W.white_noise(spec.nside, spec.seed0 + 50, nbatch=spec.nbatch)
    plan = A.Plan(spec.nside, spec.theta_cut, ntab=spec.nknots, max_batch=spec.nbatch,
                  learnable=True)
    plan.set_knots(to_dev(knots))
    log("c5 full size backward")
    xd, gd = to_dev(x), to_dev(g)
    y = plan.convolve(xd)
    gx, gk = plan.backward(gd, xd, want_map=True, want_knots=True)
    _sync()
    pix = W.eval_pixels(spec.nside, 512, spec.seed0, max_strata_ring_pixels=128)
    for b in (0, spec.nbatch - 1):
        # (A^T g)_q = (A g)_q: the operator is symmetric, so the oracle's direct
        # sum of g at the sampled pixels is the adjoint there
        ref = O.convolve(spec.nside, spec.theta_cut, knots, g[b], pixels=pix)
        assert rel_rms(to_host(gx[b])[pix], ref) <= REL_RMS_TOL
    gy = float(np.sum(to_host(gd) * to_host(y)))
    kg = float(np.dot(knots, to_host(gk)))
    xg = float(np.sum(to_host(xd) * to_host(gx)))
    scale = float(np.sqrt(np.sum(to_host(gd) ** 2) * np.sum(to_host(y) ** 2)))
    assert abs(kg - gy) <= 1e-5 * scale
    assert abs(xg - gy) <= 1e-5 * scale


def _sparse_maps(spec, size, seed):
    """Per map b: a pixel sample S_b (uniform draws plus strata rings) and a
    map that is white noise on S_b and zero elsewhere."""
    out = np.zeros((spec.nbatch, spec.npix))
    sets = []
    for b in range(spec.nbatch):
        pix = W.eval_pixels(spec.nside, size, seed + b, max_strata_ring_pixels=128)
        out[b, pix] = np.random.default_rng(seed + 100 + b).standard_normal(pix.size)
        sets.append(pix)
    return out, sets


def test_c5_full_size_knot_gradient_per_knot():
    """Nside 1024, 8 maps, 256 knots, theta_cut 30 arcmin, in the benchmark's
    launch configuration, with g = dL/dy nonzero on a pixel sample of every
    map (uniform plus the polar, cap/belt and equatorial strata): the knot
    gradient matches the FP64 oracle's knot by knot to 1e-5 max|grad|, and
    the map gradient matches it at the sampled pixels and their neighbours."""
    spec = W.C5
    A = _A()
    knots = W.gaussian_profile_knots(spec.fwhm, spec.theta_cut, spec.nknots)
    x = W.white_noise(spec.nside, spec.seed0, nbatch=spec.nbatch)
    x = x.astype(np.float32).astype(np.float64)
    g, sets = _sparse_maps(spec, 2048, spec.seed0 + 70)
    g = g.astype(np.float32).astype(np.float64)
    plan = A.Plan(spec.nside, spec.theta_cut, ntab=spec.nknots, max_batch=spec.nbatch,
                  learnable=True)
    plan.set_knots(to_dev(knots))
    log("c5 full size knot gradient, sampled g")
    gx, gk = plan.backward(to_dev(g), to_dev(x), want_map=True, want_knots=True)
    _sync()
    gk = to_host(gk)
    gk_ref = sum(O.knot_grad(spec.nside, spec.theta_cut, spec.nknots, x[b], g[b])
                 for b in range(spec.nbatch))
    err = np.max(np.abs(gk - gk_ref)) / np.abs(gk_ref).max()
    log("c5 knot gradient max error %.3e of max|grad|, rel rms %.3e"
        % (err, rel_rms(gk, gk_ref)))
    assert err <= 1e-5
    gxh = to_host(gx)
    for b in (0, spec.nbatch - 1):
        pix = np.unique(np.concatenate([sets[b], np.minimum(sets[b] + 1, spec.npix - 1)]))
        ref = O.convolve(spec.nside, spec.theta_cut, knots, g[b], pixels=pix)
        assert rel_rms(gxh[b][pix], ref) <= REL_RMS_TOL


def test_c5_loss_full_size_autograd():
    """The c5 loss at full size through the autograd Function: L = sum over a
    pixel sample of every map of (conv(x) - t)^2, with t the FP64 oracle's
    convolution by the 9 arcmin profile on the same 256-knot grid.  The
    forward, the knot gradient (knot by knot) and the map gradient match the
    oracle's for the same g = 2 (y - t)."""
    import torch
    spec = W.C5
    A = _A()
    knots = W.gaussian_profile_knots(spec.fwhm, spec.theta_cut, spec.nknots)
    target_knots = W.gaussian_profile_knots(spec.target_fwhm, spec.theta_cut, spec.nknots)
    x = W.white_noise(spec.nside, spec.seed0, nbatch=spec.nbatch)
    x = x.astype(np.float32).astype(np.float64)
    _, sets = _sparse_maps(spec, 1024, spec.seed0 + 90)
    t = [O.convolve(spec.nside, spec.theta_cut, target_knots, x[b], pixels=sets[b])
         for b in range(spec.nbatch)]
    plan = A.Plan(spec.nside, spec.theta_cut, ntab=spec.nknots, max_batch=spec.nbatch,
                  learnable=True)
    xd = to_dev(x).requires_grad_(True)
    kd = to_dev(knots).requires_grad_(True)
    log("c5 loss at full size through autograd")
    y = A.conv(xd, plan, kd)
    loss = 0.0
    for b in range(spec.nbatch):
        idx = torch.from_numpy(sets[b]).cuda()
        loss = loss + torch.sum((y[b].index_select(0, idx).double()
                                 - torch.from_numpy(t[b]).cuda()) ** 2)
    loss.backward()
    _sync()
    yh = to_host(y)
    g = np.zeros((spec.nbatch, spec.npix))
    for b in range(spec.nbatch):
        ref = O.convolve(spec.nside, spec.theta_cut, knots, x[b], pixels=sets[b])
        assert rel_rms(yh[b][sets[b]], ref) <= REL_RMS_TOL
        # the gradient the Function received, as FP32 values
        g[b, sets[b]] = np.float32(2.0 * (yh[b][sets[b]] - t[b]))
    gk_ref = sum(O.knot_grad(spec.nside, spec.theta_cut, spec.nknots, x[b], g[b])
                 for b in range(spec.nbatch))
    gk = to_host(kd.grad)
    err = np.max(np.abs(gk - gk_ref)) / np.abs(gk_ref).max()
    log("c5 loss knot gradient max error %.3e of max|grad|" % err)
    assert err <= 1e-5
    gx = to_host(xd.grad)
    for b in (0, spec.nbatch - 1):
        ref = O.convolve(spec.nside, spec.theta_cut, knots, g[b], pixels=sets[b])
        assert rel_rms(gx[b][sets[b]], ref) <= REL_RMS_TOL


@pytest.mark.parametrize("case", ["small", "c5"])
def test_backward_bitwise_reproducible(case):
    """Two backward calls on the same inputs give bit-identical map and knot
    gradients (no float atomics race: static work assignment, one histogram
    per wave, fixed-order merges)."""
    A = _A()
    if case == "small":
        nside, nb, tc, nk = 32, 3, np.radians(10.3), 64
        knots = W.gaussian_profile_knots(tc / 3, tc, nk)
    else:
        spec = W.C5
        nside, nb, tc, nk = spec.nside, spec.nbatch, spec.theta_cut, spec.nknots
        knots = W.gaussian_profile_knots(spec.fwhm, tc, nk)
    x = to_dev(W.white_noise(nside, 610, nbatch=nb))
    g = to_dev(W.white_noise(nside, 710, nbatch=nb))
    plan = A.Plan(nside, tc, ntab=nk, max_batch=nb, learnable=True)
    plan.set_knots(to_dev(knots))
    log("backward twice: %s" % case)
    gx1, gk1 = plan.backward(g, x, want_map=True, want_knots=True)
    gx2, gk2 = plan.backward(g, x, want_map=True, want_knots=True)
    _sync()
    assert np.array_equal(to_host(gk1), to_host(gk2))
    assert np.array_equal(to_host(gx1), to_host(gx2))


def test_knot_gradient_limits():
    import torch
    A = _A()
    plan = A.Plan(8, 0.3, ntab=A.MAX_GRAD_NTAB + 1, learnable=True)
    plan.set_knots(torch.ones(A.MAX_GRAD_NTAB + 1, device="cuda"))
    z = torch.zeros(768, device="cuda")
    with pytest.raises(A.ArkcosError) as e:
        plan.backward(z, z.clone(), want_map=False, want_knots=True)
    assert e.value.status == -4
    gx, _ = plan.backward(z, None, want_map=True)
    _sync()
    assert float(gx.abs().max()) == 0.0
