"""GPU tests of plx_render_fwd with segment lists on both sides of the rules by
which it renders over them or marches the rays, against the FP64 oracle
(colours and optical depths).  Which of the two ran shows in the last bits:
the march gives those of plx_render_fwd_rays."""
import numpy as np
import pytest
import torch

import synth
from oracle import oracle as O
from paper_2112_05131_amd import binding as B
from tests.gpu_util import RGB_ATOL, make_pair, say

pytestmark = pytest.mark.gpu


def check(sv, sh_dtype, n, lists, samples=True, step=0.5, check_rays=2500):
    og, gg = make_pair(sv, sh_dtype, step_voxels=step)
    o, d = synth.random_rays(n, seed=142)
    o[5::11] += 5.0  # misses
    oc, dc, desc = o.cuda(), d.cuda(), gg.desc()
    bgc = torch.rand(n, 3, generator=torch.Generator(device="cuda").manual_seed(143), device="cuda")
    bins = B.make_bins(desc, oc, dc, samples=samples)
    say(f"  {bins.n_seg} segments, {bins.n_brick} bricks, {bins.n_samp} sample slots")
    rgb, tau = torch.empty(n, 3, device="cuda"), torch.empty(n, device="cuda")
    B.plx_render_fwd(desc, oc, dc, rgb, tau, bgc, bins=bins)
    B.plx_bins_verify(desc, bins)
    rays, tau_r = torch.empty_like(rgb), torch.empty_like(tau)
    B.plx_render_fwd_rays(desc, oc, dc, rays, tau_r, None, bgc)
    assert torch.equal(rgb, rays) == (not lists)
    sel = np.sort(np.random.default_rng(144).choice(n, min(n, check_rays), replace=False))
    at = torch.from_numpy(sel).cuda()
    ref, tau_ref = O.render_fwd(og, o.numpy()[sel], d.numpy()[sel], bgc[at].cpu().double().numpy())[:2]
    for got, t in ((rgb, tau), (rays, tau_r)):
        assert np.abs(got[at].cpu().double().numpy() - ref).max() <= RGB_ATOL
        assert np.all(np.abs(t[at].cpu().double().numpy() - tau_ref) <= 1e-5 * (1.0 + tau_ref))
    return bins


@pytest.mark.parametrize("sh_dtype", [B.PLX_F32, B.PLX_BF16, B.PLX_F16])
@pytest.mark.parametrize("n", [786431, 786432, 786450])
def test_large_batches_are_rendered_over_lists(sh_dtype, n):
    say("list forward", sh_dtype, n)
    sv = synth.dense_random((21, 18, 25), seed=141, occupancy=0.5, ho_scale=0.2)
    check(sv, sh_dtype, n, n >= 786432, samples=n != 786450)


@pytest.mark.parametrize("sh_dtype", [B.PLX_BF16, B.PLX_F16])
@pytest.mark.parametrize("reso,n,lists", [((105, 100, 112), 20000, False), ((105, 100, 112), 60000, True),
                                          ((100, 92, 104), 60000, False)])
def test_16_bit_lists_by_samples_a_brick(sh_dtype, reso, n, lists):
    """2,000 samples a brick, from 2,048 bricks on."""
    say("list forward", sh_dtype, reso, n)
    sv = synth.dense_random(reso, seed=145, occupancy=0.8, ho_scale=0.2)
    bins = check(sv, sh_dtype, n, lists, samples=False)
    assert (bins.n_brick >= 2048 and bins.n_samp >= 2000 * bins.n_brick) == lists


@pytest.mark.parametrize("reso,n,lists", [((170, 165, 172), 98303, False), ((170, 165, 172), 98304, True),
                                          ((150, 152, 160), 98304, False)])
def test_fp32_lists_by_bricks(reso, n, lists):
    """8,192 bricks, from 98,304 rays on."""
    say("list forward", reso, n)
    sv = synth.dense_random(reso, seed=146, occupancy=0.2, ho_scale=0.2)
    bins = check(sv, B.PLX_F32, n, lists, samples=False, check_rays=1000)
    assert (bins.n_brick >= 8192 and n >= 98304) == lists


@pytest.mark.parametrize("sh_dtype", [B.PLX_F32, B.PLX_F16])
def test_lists_of_a_batch_serve_their_passes(sh_dtype):
    """One set of lists, read by the forward, serves the backward and the
    fused call as lists made afresh do."""
    say("list forward: one set of lists", sh_dtype)
    sv = synth.dense_random((21, 18, 25), seed=147, occupancy=0.5, ho_scale=0.2)
    og, gg = make_pair(sv, sh_dtype)
    n, m = 786432, gg.n_vox
    o, d = (x.cuda() for x in synth.random_rays(n, seed=148))
    desc = gg.desc()
    rgb, tau = torch.empty(n, 3, device="cuda"), torch.empty(n, device="cuda")
    G = torch.randn(n, 3, generator=torch.Generator(device="cuda").manual_seed(149), device="cuda")
    grads = []
    for fresh in (False, True):
        bins = B.make_bins(desc, o, d)
        B.plx_render_fwd(desc, o, d, rgb, tau, bins=bins)
        grad = torch.zeros(m, 32, device="cuda")
        touched = torch.zeros(m, dtype=torch.uint8, device="cuda")
        B.plx_render_bwd(desc, o, d, G, tau, grad, touched, bins=B.make_bins(desc, o, d) if fresh else bins)
        grads.append((grad, touched))
    assert torch.equal(grads[0][1], grads[1][1])
    scale = grads[1][0].abs().amax(0)
    assert torch.all((grads[0][0] - grads[1][0]).abs() <= 1e-4 * scale)
