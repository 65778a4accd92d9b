"""GPU test of the per-brick weight pass at the edges of its bricks and lists:
grids of one cell, one brick and a cell more, more segments in a brick than a
workgroup has lanes, and densities that vanish or saturate."""
import numpy as np
import pytest

import synth
from oracle import oracle as O
from paper_2112_05131_amd import binding as B
from tests.gpu_util import make_pair, say
from tests.test_gpu_prune_weight import check_wmax, gpu_max_weight

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sh_dtype", [B.PLX_F32, B.PLX_F16])
@pytest.mark.parametrize("reso,occ,nrays,hi", [((2, 2, 2), 1.0, 700, 30.0), ((9, 9, 9), 1.0, 3000, 30.0),
                                               ((10, 9, 17), 0.5, 1500, 30.0), ((9, 9, 9), 0.2, 600, 4e3),
                                               ((17, 33, 8), 0.3, 257, 0.0)])
def test_max_weight_brick_edges(reso, occ, nrays, hi, sh_dtype):
    """The bound is that of the other tests of the weight pass."""
    say("weight edges", reso, occ, nrays, hi, sh_dtype)
    sv = synth.dense_random(reso, seed=71, occupancy=occ, sigma_lo=-5.0, sigma_hi=hi)
    og, gg = make_pair(sv, sh_dtype=sh_dtype)
    o, d = synth.random_rays(nrays, seed=72)
    ref = O.max_weight(og, o.numpy(), d.numpy())
    assert (ref.max() > 0) == (hi > 0)
    check_wmax(gpu_max_weight(gg, o, d), ref, "edges")
    assert np.isfinite(ref).all()


@pytest.mark.parametrize("sh_dtype", [B.PLX_F32, B.PLX_BF16])
@pytest.mark.parametrize("reso,occ,nrays,sparse", [((100, 90, 99), 0.6, 700, True), ((97, 97, 97), 1.0, 2500, True),
                                                   ((73, 121, 82), 0.4, 9000, False), ((65, 65, 66), 1.0, 900, False)])
def test_max_weight_with_few_segments_a_brick(reso, occ, nrays, sparse, sh_dtype):
    """Both sides of the rule for marking the corners first (1,024 bricks with
    fewer than 32 segments each), partial bricks among them, in one call and
    in two.  The bound is that of the other tests of the weight pass."""
    say("weight: few segments", reso, occ, nrays, sh_dtype)
    sv = synth.dense_random(reso, seed=73, occupancy=occ, sigma_lo=-5.0, sigma_hi=30.0)
    og, gg = make_pair(sv, sh_dtype=sh_dtype)
    o, d = synth.random_rays(nrays, seed=74)
    bins = B.make_bins(gg.desc(), o.cuda(), d.cuda(), samples=False)
    assert (bins.n_brick >= 1024 and bins.n_seg < 32 * bins.n_brick) == sparse
    ref = O.max_weight(og, o.numpy(), d.numpy())
    assert ref.max() > 0
    check_wmax(gpu_max_weight(gg, o, d), ref, "one call")
    check_wmax(gpu_max_weight(gg, o, d, batches=2), ref, "two calls")
