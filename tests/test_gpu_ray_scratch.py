"""GPU tests of what render() in ray order keeps between forward and backward."""
import numpy as np
import pytest
import torch

import synth
from oracle import oracle as O
from paper_2112_05131_amd import binding as B
from paper_2112_05131_amd.autograd import RenderFn, render
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


@pytest.mark.parametrize("how", ["no_grad", "inference_mode", "frozen"])
def test_nothing_is_kept_where_no_backward_follows(how):
    """Under no_grad or inference mode, or with parameters that need no
    gradient, render() allocates the image and little more, and returns the
    same bits; RenderFn.apply with five arguments still records."""
    say("render without backward", how)
    _, gg = make_pair(synth.dense_random((40, 36, 44), seed=111, occupancy=0.3, ho_scale=0.2))
    n = 5000
    assert B.ray_order_grad(gg.desc(), n)
    o, d = (x.cuda() for x in synth.random_rays(n, seed=112))
    params = gg.param_records().requires_grad_()
    full = render(gg, o, d)
    assert full.requires_grad
    five = RenderFn.apply(params, gg, o, d, (1.0, 1.0, 1.0))
    five.sum().backward()
    assert torch.equal(five, full) and params.grad.abs().sum() > 0
    del five
    params.requires_grad_(how != "frozen")
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    with {"no_grad": torch.no_grad, "inference_mode": torch.inference_mode, "frozen": torch.enable_grad}[how]():
        rgb = render(gg, o, d)
    assert torch.cuda.max_memory_allocated() - before <= 12 * n + 4096
    assert not rgb.requires_grad and torch.equal(rgb, full.detach())


def test_saved_tensor_hooks_may_hand_back_unaligned_memory():
    """Hooks that keep the saved tensors in one buffer at odd offsets (and
    the rays at offsets of 4 bytes): the gradient is that without hooks."""
    say("saved-tensor hooks")
    _, gg = make_pair(synth.dense_random((20, 24, 22), seed=121, occupancy=0.5, ho_scale=0.2))
    n = 3000
    assert B.ray_order_grad(gg.desc(), n)
    o, d = (x.cuda() for x in synth.random_rays(n, seed=122))
    params = gg.param_records().requires_grad_()

    def pack(t):
        pool = torch.empty(t.numel() + 64, dtype=t.dtype, device=t.device)
        off = 1 if t.dtype == torch.float32 else 12
        pool[off:off + t.numel()] = t.reshape(-1)
        return pool[off:off + t.numel()].view(t.shape)

    grads = []
    for hooks in (False, True):
        params.grad = None
        with torch.autograd.graph.saved_tensors_hooks(pack if hooks else lambda t: t, lambda t: t):
            rgb = render(gg, o, d)
        rgb.square().sum().backward()
        grads.append(params.grad.clone())
    scale = grads[0].abs().max().item()
    assert scale > 0 and (grads[0] - grads[1]).abs().max().item() <= 1e-5 * scale
