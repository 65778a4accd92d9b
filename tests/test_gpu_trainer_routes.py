"""GPU tests of Trainer.run by the order its batches are rendered in: scratch
in ray order, segment lists with the replay, and lists with the recorded
backward, each with the next batch prepared on a second stream and without.
The sets of buffers that alternate are kept and reused, also by a trainer that
changes from one order to the other."""
import numpy as np
import pytest
import torch

import synth
from paper_2112_05131_amd import binding as B
from paper_2112_05131_amd.grid import Grid
from paper_2112_05131_amd.train import RECORDED_MIN_RAYS, RaySampler, TrainConfig, Trainer
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def _pool(gt, n_cam, size, seed):
    poses = synth.sphere_poses(n_cam, seed=seed)
    o, d = (x.cuda() for x in synth.all_camera_rays(poses, size, size))
    g = Grid.from_mask(gt.mask.cuda(), gt.reso, gt.density.cuda(), gt.sh.cuda())
    tgt = torch.empty(o.shape[0], 3, device="cuda")
    B.plx_render_fwd(g.desc(), o, d, tgt)
    return o, d, tgt


def _run(init, pool, batch, overlap, steps):
    g = Grid.from_mask(init.mask, init.reso, init.density, init.sh)
    tr = Trainer(g, TrainConfig(), seed=5)
    sampler = RaySampler(*pool, batch, seed=7)
    losses = []
    for _ in range(steps):
        tr.loss_sum.zero_()
        tr.run(sampler, 1, overlap=overlap)
        torch.cuda.synchronize()
        losses.append(tr.loss_sum.item())
    tr.loss_sum.zero_()
    tr.run(sampler, 5, overlap=overlap)
    torch.cuda.synchronize()
    losses.append(tr.loss_sum.item())
    return tr, losses


@pytest.mark.parametrize("reso,occ,batch,route", [((48, 48, 48), 0.2, 5000, "rays"), ((48, 48, 48), 0.5, 30000, "replay"),
                                                  ((40, 44, 52), 1.0, RECORDED_MIN_RAYS + 1000, "recorded")])
def test_overlapped_preparation_matches_sequential(reso, occ, batch, route):
    """The losses of every step equal those of the plain loop over the same
    batches (up to the order of FP32 atomics)."""
    say("trainer routes", route)
    gt = synth.blob_scene(reso, n_blobs=6, occupancy=occ, seed=311)
    pool = _pool(gt, 10, 100, 311)
    init = synth.perturbed(gt, seed=312, device="cuda")
    desc = Grid.from_mask(init.mask, init.reso, init.density, init.sh).desc()
    assert B.ray_order(desc, batch) == (route == "rays")
    losses = {}
    for overlap in (False, True):
        tr, losses[overlap] = _run(init, pool, batch, overlap, 4)
        bufs = tr._run_bufs
        assert all(b is not None for b in bufs[0][:2]) and all(b is not None for b in bufs[1][:2])
        assert (bufs[0][2] is not None) == (route == "recorded")
        # further batches of the scene fit the buffers and their slack
        ptrs = [[x.data_ptr() if x is not None else None for x in s] for s in bufs]
        tr.run(RaySampler(*pool, batch, seed=8), 4, overlap=overlap)
        torch.cuda.synchronize()
        assert ptrs == [[x.data_ptr() if x is not None else None for x in s] for s in tr._run_bufs]
    say(f"  losses {losses[True]}")
    np.testing.assert_allclose(losses[True], losses[False], rtol=1e-4)
    assert all(x > 0 for x in losses[True])


def test_a_trainer_that_changes_its_order():
    """Batches in ray order, over lists, and in ray order again on one
    trainer, whose buffers then serve either: the losses with overlap are
    those without."""
    say("trainer changes order")
    gt = synth.blob_scene((48, 48, 48), n_blobs=6, occupancy=0.5, seed=321)
    pool = _pool(gt, 8, 100, 321)
    init = synth.perturbed(gt, seed=322, device="cuda")
    got = {}
    for overlap in (False, True):
        g = Grid.from_mask(init.mask, init.reso, init.density, init.sh)
        tr = Trainer(g, TrainConfig(), seed=5)
        got[overlap] = []
        for i, batch in enumerate((2000, 70000, 2000, 30000, 3000)):
            tr.loss_sum.zero_()
            tr.run(RaySampler(*pool, batch, seed=20 + i), 3, overlap=overlap)
            torch.cuda.synchronize()
            got[overlap].append(tr.loss_sum.item())
    np.testing.assert_allclose(got[True], got[False], rtol=1e-4)
    assert all(np.isfinite(got[True])) and all(x > 0 for x in got[True])
