"""GPU tests of the optimiser's lists, zero halves and streamed accesses: the
edges of a workgroup's voxels, large grids with most and with few voxels
touched, records of which one half has no gradient, and zero gradients that
must not be skipped (NaN state, infinite rate, no eps)."""
import math

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2112_05131_amd import binding as B
from paper_2112_05131_amd.grid import Grid
from tests.gpu_util import say, split_records

pytestmark = pytest.mark.gpu


def _grid(n, sh_dtype):
    reso = (3, 3, -(-n // 9) + 1)
    mask = torch.zeros(reso[0] * reso[1] * reso[2], dtype=torch.uint8)
    mask[:n] = 1
    gen = torch.Generator().manual_seed(n)
    dens = torch.rand(n, generator=gen) + 0.5
    sh = torch.randn(n, 27, generator=gen)
    return Grid.from_mask(mask.cuda(), reso, dens.cuda(), sh.cuda(), sh_dtype=sh_dtype), dens, sh


# one voxel; a list's edge; a grid large enough for streamed accesses, with
# most voxels touched, with half of each list and with few
@pytest.mark.parametrize("sh_dtype", [B.PLX_F32, B.PLX_F16])
@pytest.mark.parametrize("n,share", [(1, 1.0), (63, 1.0), (64, 1.0), (65, 1.0), (129, 0.5),
                                     (700001, 1.0), (700001, 0.5), (700001, 0.1)])
def test_rmsprop_lists(n, share, sh_dtype):
    """Three steps: gradients in all slots, in the upper half of the record
    only, and none.  The bounds are those of the other RMSProp test."""
    say("rmsprop lists", n, share, sh_dtype)
    gg, dens, sh = _grid(n, sh_dtype)
    gen = torch.Generator().manual_seed(7)
    act = (torch.rand(n, generator=gen) < share).to(torch.uint8)
    on = act.bool()
    d, s = dens.double().numpy().copy(), sh.double().numpy().copy()
    vd, vs = np.zeros(n), np.zeros((n, 27))
    vstate = torch.zeros(n, 32, device="cuda")
    lr_s, lr_h, beta, eps = 3.0, 0.01, 0.95, 1e-8
    for it in range(3):
        grad = torch.randn(n, 32, generator=gen)
        grad[:, 27], grad[:, 29:] = 0.0, 0.0
        if it == 1:
            grad[:, :16] = 0.0
        if it == 2:
            grad[:] = 0.0
        keep = grad.clone()
        before = gg.param_records().clone(), vstate.clone()
        grad, touched = grad.cuda(), act.cuda()
        B.plx_rmsprop_step(gg.desc(), gg.master, vstate, grad, touched, lr_s, lr_h, beta, eps)
        torch.cuda.synchronize()
        assert int(touched.sum()) == 0
        assert torch.equal(grad.cpu(), torch.where(on[:, None], torch.zeros(()), keep))
        assert torch.equal(gg.param_records()[~on.cuda()], before[0][~on.cuda()])
        assert torch.equal(vstate[~on.cuda()], before[1][~on.cuda()])
        if it == 2:  # nothing but the decay
            assert torch.equal(gg.param_records(), before[0])
            assert torch.equal(vstate[on.cuda()], before[1][on.cuda()] * torch.tensor(beta, device="cuda"))
        gd, gs = keep[:, 28].double().numpy().copy(), keep[:, :27].double().numpy().copy()
        O.rmsprop(act.numpy(), d, s, vd, vs, gd, gs, lr_s, lr_h, beta, eps)
    pd, ps = split_records(gg.param_records())
    for got, ref, p0, lr in ((pd, d, dens.double().numpy(), lr_s), (ps, s, sh.double().numpy(), lr_h)):
        assert np.all(np.abs(got - ref) <= 4e-7 * (np.abs(p0) + np.abs(ref) + 3 * lr / math.sqrt(1 - beta)))
    vdg, vsg = split_records(vstate)
    np.testing.assert_allclose(vdg, vd, rtol=2e-6, atol=1e-30)
    np.testing.assert_allclose(vsg, vs, rtol=2e-6, atol=1e-30)


@pytest.mark.parametrize("lr,eps,v0", [(math.inf, 1e-8, 1.0), (0.1, 0.0, 0.0), (0.1, 1e-8, math.nan),
                                       (0.1, 1e-8, -1.0), (0.1, 1e-8, math.inf), (-0.1, 1e-8, 1.0)])
def test_rmsprop_zero_gradient_that_counts(lr, eps, v0):
    """A zero gradient times an infinite rate, or over a zero, negative or
    NaN root, is NaN in the parameter as by the formula; over an infinite one
    or with a negative rate it changes nothing."""
    say("rmsprop zero gradient", lr, eps, v0)
    gg, dens, sh = _grid(70, B.PLX_F32)
    vstate = torch.full((70, 32), v0, device="cuda")
    grad, touched = torch.zeros(70, 32, device="cuda"), torch.ones(70, dtype=torch.uint8, device="cuda")
    before = gg.data.clone()
    B.plx_rmsprop_step(gg.desc(), None, vstate, grad, touched, lr, lr, 0.5, eps)
    ref = before - lr * torch.zeros_like(before) / (torch.sqrt(torch.full_like(before, 0.5 * v0)) + eps)
    used = [*range(27), 28]
    assert torch.equal(torch.isnan(gg.data[:, used]), torch.isnan(ref[:, used]))
    assert torch.equal(torch.nan_to_num(gg.data[:, used]), torch.nan_to_num(ref[:, used]))
