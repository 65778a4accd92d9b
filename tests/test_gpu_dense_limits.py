"""GPU tests of densities without bound: an opaque voxel (infinite density, or
one so large that the depths around it vanish beside it) ends its rays, and
everything before it keeps its share of the colour."""
import numpy as np
import pytest
import torch

import synth
from oracle import oracle as O
from paper_2112_05131_amd import binding as B
from tests.gpu_util import RGB_ATOL, assert_grads_close, assert_touched_equal, grad_mass, make_pair, say
from tests.test_gpu_march import _pose, _render, _view

pytestmark = pytest.mark.gpu


def _opaque_pair(sh_dtype, value):
    """A dense grid with some opaque voxels, the same on both sides; none next
    to the hull, where a sample may lie on a cell's face (weight 0)."""
    reso = (23, 19, 26)
    sv = synth.dense_random(reso, seed=91, ho_scale=0.2)
    og, gg = make_pair(sv, sh_dtype)
    inner = np.zeros(reso, bool)
    inner[3:-3, 3:-3, 3:-3] = True
    ids = np.flatnonzero(inner)[::61]
    og.density[ids] = value
    words = gg.data if sh_dtype == B.PLX_F32 else gg.data.view(torch.float32)
    words[torch.from_numpy(ids).cuda(), B.SLOT_SIGMA if sh_dtype == B.PLX_F32 else 14] = value
    return og, gg


def check_training(bins, gg, oc, dc, tgt, rgb, check, ref):
    n, m = oc.shape[0], gg.n_vox
    grad = torch.zeros(m, 32, device="cuda")
    touched = torch.zeros(m, dtype=torch.uint8, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    B.plx_render_train(gg.desc(), oc, dc, tgt, 1.0 / n, grad, touched, loss, rgb, bins=bins)
    assert np.abs(rgb.cpu().double().numpy()[check] - ref).max() <= RGB_ATOL
    want = ((rgb.double() - tgt.double()) ** 2).sum().item() / n
    assert abs(loss.item() - want) <= 1e-5 * want
    assert torch.isfinite(grad).all()


@pytest.mark.parametrize("sh_dtype", [B.PLX_F32, B.PLX_F16])
@pytest.mark.parametrize("value", [float("inf"), 1e30])
@pytest.mark.parametrize("n", [700, 98400])
def test_opaque_voxels_match_oracle(sh_dtype, value, n):
    """Colours, depths, losses and finite gradients of the march, with a wave
    per ray and with 16 lanes per ray.  Tolerance: the stated RGB bound; the
    loss's is relative to that of the call's own colours."""
    say("opaque voxels", sh_dtype, value, n)
    og, gg = _opaque_pair(sh_dtype, value)
    o, d = synth.random_rays(n, seed=92)
    check = np.arange(n)[:: max(1, n // 4000)]
    ref, tau_ref = O.render_fwd(og, o.numpy()[check], d.numpy()[check])[:2]
    assert np.isfinite(ref).all() and (tau_ref > 1e20).sum() > 50
    oc, dc, desc = o.cuda(), d.cuda(), gg.desc()
    rgb, tau = torch.empty(n, 3, device="cuda"), torch.empty(n, device="cuda")
    B.plx_render_fwd_rays(desc, oc, dc, rgb, tau)
    assert np.abs(rgb.cpu().double().numpy()[check] - ref).max() <= RGB_ATOL
    got = tau.cpu().double().numpy()[check]
    assert np.array_equal(np.isinf(got), np.isinf(tau_ref))
    fin = np.isfinite(tau_ref)
    assert np.all(np.abs(got[fin] - tau_ref[fin]) <= 1e-5 * (1.0 + tau_ref[fin]))
    tgt = synth.targets_uniform(n, seed=93).cuda()
    check_training(B.make_ray_work(n), gg, oc, dc, tgt, rgb, check, ref)


@pytest.mark.parametrize("sh_dtype", [B.PLX_F32, B.PLX_F16])
@pytest.mark.parametrize("value", [float("inf"), 1e30])
@pytest.mark.parametrize("n,samples", [(200, True), (700, True), (700, False), (9000, True)])
def test_opaque_voxels_in_lists(sh_dtype, value, n, samples):
    """The same over segment lists: replay, and the recorded backward below
    and above 40 segments a brick (runs of a segment composed apart)."""
    say("opaque voxels: lists", sh_dtype, value, n, samples)
    og, gg = _opaque_pair(sh_dtype, value)
    o, d = synth.random_rays(n, seed=94)
    check = np.arange(n)[:: max(1, n // 4000)]
    ref = O.render_fwd(og, o.numpy()[check], d.numpy()[check])[0]
    oc, dc = o.cuda(), d.cuda()
    bins = B.make_bins(gg.desc(), oc, dc, samples=samples)
    assert (bins.n_seg >= 40 * bins.n_brick) == (n > 200)
    check_training(bins, gg, oc, dc, synth.targets_uniform(n, seed=95).cuda(), torch.empty(n, 3, device="cuda"), check, ref)


@pytest.mark.parametrize("w,h", [(30, 20), (300, 250), (1030, 770)])
@pytest.mark.parametrize("value", [float("inf"), 1e30])
def test_views_of_opaque_voxels_match_oracle(value, w, h):
    """The same for views, with each of their cuts (4, 8 and 16 lanes a ray)."""
    say("opaque voxels: view", value, w, h)
    og, gg = _opaque_pair(B.PLX_F32, value)
    c2w, focal = _pose(12), 1.9 * w
    got = _render(gg, [_view(c2w, focal, w, h)], w * h)
    o, d = O.camera_rays(c2w, focal, w, h)
    sel = np.sort(np.random.default_rng(6).choice(w * h, min(3000, w * h), replace=False))
    ref = O.render_fwd(og, o[sel], d[sel])[0]
    assert np.abs(got[torch.from_numpy(sel).cuda()].cpu().double().numpy() - ref).max() <= RGB_ATOL


@pytest.mark.parametrize("sh_dtype", [B.PLX_F32, B.PLX_F16])
@pytest.mark.parametrize("value", [float("inf"), 1e30, 1e12])
@pytest.mark.parametrize("n,cap", [(700, 512), (700, 5), (98400, 512)])
def test_gradients_before_opaque_voxels(sh_dtype, value, n, cap):
    """In ray order: the gradients are those of the same grid with densities
    of 1e12, beyond which nothing changes (no light passes either); the samples
    before an opaque one keep their transmittance.  With the stated bounds;
    with per-ray depths and the beta prior's factor unchanged as well."""
    say("opaque voxels: gradients", sh_dtype, value, n, cap)
    og, gg = _opaque_pair(sh_dtype, value)
    og.density[og.density >= 1e12] = 1e12
    o, d = synth.random_rays(n, seed=96)
    on, dn = o.numpy(), d.numpy()
    oc, dc, desc, m = o.cuda(), d.cuda(), gg.desc(), gg.n_vox
    G = np.random.default_rng(97).normal(size=(n, 3)) * 1e-2
    Gc = torch.from_numpy(G).float().cuda()
    Gd = Gc.cpu().double().numpy()
    ref, tau_ref = O.render_fwd(og, on, dn)[:2]
    work = B.make_ray_work(n, cap=cap)
    rgb, tau = torch.empty(n, 3, device="cuda"), torch.empty(n, device="cuda")
    B.plx_render_fwd_rays(desc, oc, dc, rgb, tau, work)
    assert np.abs(rgb.cpu().double().numpy() - ref).max() <= RGB_ATOL
    plain = torch.empty(n, device="cuda")
    B.plx_render_fwd_rays(desc, oc, dc, rgb, plain)
    assert torch.equal(tau > 1e9, plain > 1e9) and torch.equal(torch.isinf(tau), torch.isinf(plain))
    fin = torch.isfinite(plain)
    assert torch.all((tau[fin] - plain[fin]).abs() <= 1e-6 * (1.0 + plain[fin]))
    gd, gs, t_ref = O.render_bwd(og, on, dn, Gd)
    mass = grad_mass(og, on, dn, Gd)
    grad = torch.zeros(m, 32, device="cuda")
    touched = torch.zeros(m, dtype=torch.uint8, device="cuda")
    pl = torch.zeros(2, dtype=torch.float64, device="cuda")
    B.plx_render_bwd_rays(desc, oc, dc, Gc, work, grad, touched)
    assert_touched_equal(touched, t_ref, "opaque")
    assert_grads_close(grad, gd, gs, "opaque", mass)
    # the beta prior alone: an opaque ray has the largest loss and no gradient
    grad.zero_()
    B.plx_render_bwd_rays(desc, oc, dc, torch.zeros_like(Gc), work, grad, touched, priors=B.Priors(0.0, 0.05, 1e-3, pl))
    _, lb_ref, gd_p, _ = O.regularisers(og, on, dn, 0.0, 0.05, 1e-3)
    assert abs(pl[1].item() - lb_ref) <= 1e-6 * abs(lb_ref) + 1e-9
    assert np.all(np.isfinite(gd_p)) and torch.isfinite(grad).all()
