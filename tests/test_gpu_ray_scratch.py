"""GPU tests of what render() in ray order keeps between forward and backward."""
import numpy as np
import pytest
import torch

import synth
from oracle import oracle as O
from paper_2112_05131_amd import binding as B
from paper_2112_05131_amd.autograd import render
from tests.gpu_util import assert_grads_close, grad_mass, make_pair, say

pytestmark = pytest.mark.gpu


def test_render_keeps_a_bounded_number_of_bytes():
    """60,000 rays with about 100 occupied samples each: fewer are kept than
    most rays have, and the gradient is still the oracle's."""
    say("ray order: kept bytes")
    sv = synth.dense_random((80, 72, 76), seed=101, occupancy=0.22, ho_scale=0.2)
    og, gg = make_pair(sv)
    n = 60000
    assert B.ray_order_grad(gg.desc(), n)
    o, d = synth.random_rays(n, seed=102)
    G = torch.from_numpy(np.random.default_rng(103).normal(size=(n, 3))).float()
    oc, dc, Gc = o.cuda(), d.cuda(), G.cuda()
    params = gg.param_records().requires_grad_()
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    rgb = render(gg, oc, dc)
    assert torch.cuda.max_memory_allocated() - before <= B.RAY_SAMP_BYTES + 100 * n
    assert B.ray_cap(n, gg.desc()) < 120
    (rgb * Gc).sum().backward()
    gd, gs, _ = O.render_bwd(og, o.numpy(), d.numpy(), G.double().numpy())
    assert_grads_close(params.grad, gd, gs, "render", grad_mass(og, o.numpy(), d.numpy(), G.double().numpy()))
