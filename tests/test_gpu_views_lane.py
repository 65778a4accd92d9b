"""GPU tests of the views that take one lane per ray (from 131,072 pixels on,
where the pixels lie closer than 0.2 voxel, 0.1 with 16-bit records) and of
the large ones beside them that do not, against the FP64 oracle; a view has
the same bits in every launch."""
import numpy as np
import pytest
import torch

import synth
from oracle import oracle as O
from paper_2112_05131_amd import binding as B
from tests.gpu_util import RGB_ATOL, make_pair, say
from tests.test_gpu_march import _pose, _render, _view

pytestmark = pytest.mark.gpu

RESO = (23, 31, 18)


def _focal(pitch, radius):
    """Focal length (pixels) at which a pixel is `pitch` voxels wide at the
    grid's centre (or at half its extent, from inside) of a unit box."""
    return max(_depth(radius), 0.5 * max(RESO)) / pitch


def _depth(radius, seed=11):
    c = _pose(seed, radius).reshape(3, 4)[:, 3] * np.array(RESO)
    return float(np.sqrt((c ** 2).sum()))


def _check(og, got, c2w, focal, w, h, n=3000):
    """Sampled pixels that see the grid, and the last row and column."""
    o, d = O.camera_rays(c2w, focal, w, h)
    rng = np.random.default_rng(8)
    # the box's middle in the image, as far as half its diagonal reaches
    r = min(0.5 * w, 0.9 * focal / 2.0)
    px = np.clip(rng.uniform(0.5 * w - r, 0.5 * w + r, n), 0, w - 1).astype(int)
    py = np.clip(rng.uniform(0.5 * h - r, 0.5 * h + r, n), 0, h - 1).astype(int)
    sel = np.unique(np.concatenate([py * w + px, np.arange(0, w, 7) + (h - 1) * w, np.arange(0, h, 7) * w + w - 1]))
    ref = O.render_fwd(og, o[sel], d[sel])[0]
    err = np.abs(got[torch.from_numpy(sel).cuda()].cpu().double().numpy() - ref).max()
    assert err <= RGB_ATOL, err
    assert np.any(np.abs(ref - 1.0) > 0.05) and torch.all(got >= 0)  # grid seen, every pixel written


@pytest.mark.parametrize("sh_dtype", [B.PLX_F32, B.PLX_BF16, B.PLX_F16])
@pytest.mark.parametrize("w,h", [(512, 256), (509, 263), (1025, 768), (2001, 64)])
@pytest.mark.parametrize("pitch,radius", [(0.03, 0.5), (0.09, 2.0), (0.11, 2.0), (0.19, 2.0), (0.21, 2.0)])
def test_large_views_match_oracle(sh_dtype, w, h, pitch, radius):
    """Both sides of both lines, with 8 and with 4 lanes a ray, sizes that do
    not fill their tiles, and a camera inside the grid.  Tolerance: the
    stated RGB bound."""
    say("large view", sh_dtype, w, h, pitch, radius)
    sv = synth.dense_random(RESO, seed=7, occupancy=0.35)
    og, gg = make_pair(sv, sh_dtype=sh_dtype)
    c2w, focal = _pose(11, radius), _focal(pitch, radius)
    _check(og, _render(gg, [_view(c2w, focal, w, h)], w * h), c2w, focal, w, h)


def test_a_launch_of_more_tiles_than_workgroups():
    """4200x4200 pixels, 1.1M tiles of 2^20 workgroups, too far apart for a
    lane per ray."""
    say("large view: strided tiles")
    sv = synth.blob_scene((40, 40, 40), n_blobs=5, occupancy=0.2, seed=8)
    og, gg = make_pair(sv)
    w = h = 4200
    c2w, focal = _pose(3, 60.0), 60.0 * 40 / 0.25
    got = _render(gg, [_view(c2w, focal, w, h)], w * h)
    o, d = O.camera_rays(c2w, focal, w, h)
    rng = np.random.default_rng(6)
    sel = np.concatenate([(rng.integers(2000, 2200, 3000) * w + rng.integers(2000, 2200, 3000)), w * h - 1 - rng.choice(4 * w, 500)])
    ref = O.render_fwd(og, o[sel], d[sel])[0]
    assert np.abs(got[torch.from_numpy(sel).cuda()].cpu().double().numpy() - ref).max() <= RGB_ATOL
    assert torch.all(got >= 0) and np.any(np.abs(ref - 1.0) > 0.05)


@pytest.mark.parametrize("sh_dtype", [B.PLX_F32, B.PLX_F16])
def test_same_bits_in_every_launch(sh_dtype):
    """Small views, large ones of both kinds and of two scenes, 27 of them
    (two launches), on one queue and repeated: each has the bits of its own
    launch."""
    say("large views in one list", sh_dtype)
    grids = [make_pair(synth.dense_random(RESO, seed=s, occupancy=0.4), sh_dtype=sh_dtype)[1] for s in (1, 2)]
    sizes = [(40, 30), (512, 256), (700, 300), (300, 290)]
    views, off = [], 0
    for i in range(27):
        w, h = sizes[i % 4]
        focal = _focal((0.05, 0.3)[i // 4 % 2], 2.0)
        views.append(_view(_pose(30 + i), focal, w, h, scene=i % 2, off=off))
        off += w * h
    table, q = B.SceneTable(grids), B.views_queue()
    out = torch.full((3 * off,), -1.0, device="cuda")
    for _ in range(2):
        out.fill_(-1.0)
        B.plx_render_views(table, views, out, q)
        B.plx_render_views_status(q)
        assert torch.all(out >= 0)
    for v in views:
        n = v.width * v.height
        alone = torch.full((3 * n,), -1.0, device="cuda")
        one = B.PlxView.from_buffer_copy(v)
        one.out_offset = 0
        B.plx_render_views(table, [one], alone, q)
        assert torch.equal(alone, out[3 * v.out_offset:3 * (v.out_offset + n)])


def test_views_of_unknown_tables_render_nothing():
    """A large view given a table of another storage type: refused by the
    status word, no pixel written."""
    say("large view: wrong table")
    _, gg = make_pair(synth.dense_random(RESO, seed=3, occupancy=0.4))
    table, q = B.SceneTable([gg]), B.views_queue()
    out = torch.full((3 * 512 * 300,), -1.0, device="cuda")
    v = _view(_pose(5), _focal(0.05, 2.0), 512, 300)
    table.sh_dtype = B.PLX_F16
    B.plx_render_views(table, [v], out, q)
    with pytest.raises(B.PlxError):
        B.plx_render_views_status(q)
    assert torch.all(out == -1.0)
