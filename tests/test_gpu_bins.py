"""GPU tests of the segment lists made by several lanes a ray: every maximal
run of a ray's samples in an occupied brick is listed once, in ray order,
whatever part of the ray it begins in, and the lists of a batch of any size
add up."""
import numpy as np
import pytest
import torch

import synth
from oracle import oracle as O
from paper_2112_05131_amd import binding as B
from tests.gpu_util import make_pair, say

pytestmark = pytest.mark.gpu


def _segments(og, occ_bricks, o, d):
    """(ray, brick, first sample, last sample) of every segment."""
    out = []
    for i in range(o.shape[0]):
        tr = O.trace_ray(og, o[i], d[i])
        cell = np.asarray(tr["cell"] if isinstance(tr, dict) else tr[0]).reshape(-1, 3)
        b = cell // 8
        k = 0
        while k < len(b):
            e = k
            while e + 1 < len(b) and np.array_equal(b[e + 1], b[k]):
                e += 1
            if occ_bricks[tuple(b[k])]:
                out.append((i, *b[k], k, e))
            k = e + 1
    return out


@pytest.mark.parametrize("reso,occ,n", [((9, 9, 9), 1.0, 1), ((17, 40, 33), 0.02, 63), ((70, 66, 90), 0.002, 257),
                                        ((70, 66, 90), 1.0, 64), ((128, 16, 16), 0.01, 300)])
def test_segments_are_the_runs_of_occupied_bricks(reso, occ, n):
    say("bins", reso, occ, n)
    sv = synth.dense_random(reso, seed=91, occupancy=occ)
    og, gg = make_pair(sv)
    o, d = synth.random_rays(n, seed=92)
    b = B.make_bins(gg.desc(), o.cuda(), d.cuda())
    idx = og.index.reshape(reso) >= 0
    cells = np.zeros(reso, bool)
    for x in (0, 1):
        for y in (0, 1):
            for z in (0, 1):
                cells[:-1, :-1, :-1] |= idx[x:reso[0] - 1 + x, y:reso[1] - 1 + y, z:reso[2] - 1 + z]
    nb = [-(-(r - 1) // 8) for r in reso]
    full = np.zeros([8 * m for m in nb], bool)
    c = cells[tuple(slice(0, 8 * m) for m in nb)]
    full[tuple(slice(0, s) for s in c.shape)] = c
    bricks = full.reshape(nb[0], 8, nb[1], 8, nb[2], 8).any(axis=(1, 3, 5))
    ref = _segments(og, bricks, o.numpy(), d.numpy())
    assert b.n_seg == len(ref)
    assert b.n_samp == sum(e - k + 1 for *_, k, e in ref)
    assert b.n_brick == len({r[1:4] for r in ref})
    if not ref:
        return
    seg = b.seg_buf[:16 * b.n_seg].view(torch.int32).view(-1, 4).cpu().numpy()
    assert sorted(map(tuple, seg[:, :3].tolist())) == sorted((r[0], r[4], r[5]) for r in ref)
    # slots are in ray order, and along a ray in the order of its samples
    by_slot = seg[np.argsort(seg[:, 3])]
    assert np.array_equal(by_slot[:, 3], np.arange(b.n_seg))
    assert [tuple(r) for r in by_slot[:, :3].tolist()] == [(r[0], r[4], r[5]) for r in ref]
    B.plx_bins_verify(gg.desc(), b)
