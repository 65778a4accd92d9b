"""GPU test of grids whose records take more than 4 GiB (64-bit addresses in
the march) against a pass that shares no record access with it: the fused call
over segment lists."""
import math

import pytest
import torch

import synth
from oracle import oracle as O
from paper_2112_05131_amd import binding as B
from paper_2112_05131_amd.grid import Grid
from tests.gpu_util import RGB_ATOL, say
from tests.test_gpu_march import _pose, _render, _view

pytestmark = pytest.mark.gpu

CASES = [(B.PLX_F32, (336, 320, 320)), (B.PLX_F16, (420, 416, 400))]


def _wide(sh_dtype, reso):
    n = reso[0] * reso[1] * reso[2]
    assert n * B.plx_record_bytes(sh_dtype) > 1 << 32
    rec = torch.zeros(n, 32, dtype=torch.float32, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(1)
    for s in range(27):
        rec[:, s] = torch.rand(n, generator=g, device="cuda") * 0.2 - 0.1 + (2.0 if s % 9 == 0 else 0.0)
    rec[:, 28] = torch.rand(n, generator=g, device="cuda") * 20 - 5
    index = torch.arange(n, dtype=torch.int32, device="cuda")
    # holes, so that NULL corners are read too: their records stay in the table
    index[5::37] = -1
    if sh_dtype != B.PLX_F32:
        r16 = torch.empty(n, 32, dtype=torch.int16, device="cuda")
        B.plx_records_convert(B.PLX_F32, rec, sh_dtype, r16, n)
        rec = r16
    return Grid(reso, index, rec, sh_dtype)


def _train(grid, o, d, tgt, bins):
    n, m = o.shape[0], grid.n_vox
    grad = torch.zeros(m, 32, device="cuda")
    touched = torch.zeros(m, dtype=torch.uint8, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    rgb = torch.empty(n, 3, device="cuda")
    B.plx_render_train(grid.desc(), o, d, tgt, 1.0 / n, grad, touched, loss, rgb, bins=bins)
    return grad, touched, loss.item(), rgb


@pytest.mark.parametrize("sh_dtype,reso", CASES)
def test_march_of_wide_tables_matches_the_lists(sh_dtype, reso):
    """Views, forward, and training with records that are full after three
    samples (the rest is evaluated again) or never.  Two FP32 evaluations of
    the same samples: colours within twice the stated RGB bound, gradients
    within 1e-4 of a slot's largest."""
    say("wide tables", sh_dtype)
    grid = _wide(sh_dtype, reso)
    c2w, w, h = _pose(21), 120, 90
    focal = 0.5 * w / math.tan(0.3)
    o, d = (torch.from_numpy(x).float().cuda().contiguous() for x in O.camera_rays(c2w, focal, w, h))
    n = w * h
    tgt = synth.targets_uniform(n, seed=151).cuda()
    ref = _train(grid, o, d, tgt, B.make_bins(grid.desc(), o, d, samples=False))  # seg_fwd and the replay
    assert (ref[3].max(0).values - ref[3].min(0).values).min() > 0.1  # the grid is seen
    assert (_render(grid, [_view(c2w, focal, w, h)], n) - ref[3]).abs().max().item() <= 2 * RGB_ATOL
    fwd = torch.empty(n, 3, device="cuda")
    B.plx_render_fwd_rays(grid.desc(), o, d, fwd)
    assert (fwd - ref[3]).abs().max().item() <= 2 * RGB_ATOL
    scale = ref[0].abs().amax(0)
    for cap in (3, 512):
        got = _train(grid, o, d, tgt, B.make_ray_work(n, cap=cap))
        assert torch.equal(got[1], ref[1])
        assert abs(got[2] - ref[2]) <= 1e-4 * ref[2]
        assert (got[3] - ref[3]).abs().max().item() <= 2 * RGB_ATOL
        assert torch.all((got[0] - ref[0]).abs().amax(0) <= 1e-4 * scale)
        del got
    del grid, ref
    torch.cuda.empty_cache()
