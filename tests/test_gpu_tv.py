"""GPU tests of the total-variation kernel at the edges of its workgroups'
shares: one cell, a share and its neighbours, as many shares as workgroups and
one more, and both sides of the line above which shares are 256 cells."""
import pytest
import torch

from oracle import oracle as O
from paper_2112_05131_amd import binding as B
import synth
from tests.gpu_util import assert_grads_close, assert_touched_equal, make_pair, say
from tests.test_gpu_background import bg_pair

pytestmark = pytest.mark.gpu

COUNTS = [1, 127, 128, 129, 65536, 65537, 131072, 131073, 131329, 200000]


@pytest.mark.parametrize("bg", [False, True])
@pytest.mark.parametrize("count", COUNTS)
def test_tv_segment_lengths(count, bg):
    """Segments that start near the grid's end, so that all but the shortest
    wrap; the bounds are those of the other TV tests."""
    say("tv segment", count, bg)
    og, gg = (bg_pair((50, 64, 65), 171, occupancy=0.3) if bg
              else make_pair(synth.dense_random((50, 64, 65), seed=172, occupancy=0.3)))
    start = 50 * 64 * 65 - 1000
    grad = torch.zeros(gg.n_vox, 32, device="cuda")
    touched = torch.zeros(gg.n_vox, dtype=torch.uint8, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    dev, ref = (B.plx_bg_tv_grad, O.bg_tv) if bg else (B.plx_tv_grad, O.tv)
    dev(gg.desc(), start, count, 0.9, 1.3, 1e-9, grad, touched, loss)
    torch.cuda.synchronize()
    l_ref, gd, gs, t_ref = ref(og, start, count, 0.9, 1.3, 1e-9)
    assert abs(loss.item() - l_ref) <= 1e-5 * abs(l_ref)
    assert_touched_equal(touched, t_ref, "tv")
    assert_grads_close(grad, gd, gs, "tv")


@pytest.mark.parametrize("bg", [False, True])
@pytest.mark.parametrize("with_loss", [False, True])
@pytest.mark.parametrize("count", [65536, 524288, 524289, 700001])
def test_tv_with_and_without_a_loss(count, with_loss, bg):
    """Without a loss, segments above 524,288 cells get a workgroup for every
    1024; the gradient and the touched set are the same sums."""
    say("tv loss", count, with_loss, bg)
    reso = (80, 96, 91)
    og, gg = (bg_pair(reso, 173, occupancy=0.3) if bg else make_pair(synth.dense_random(reso, seed=174, occupancy=0.3)))
    start = 80 * 96 * 91 - 5000
    grad = torch.zeros(gg.n_vox, 32, device="cuda")
    touched = torch.zeros(gg.n_vox, dtype=torch.uint8, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda") if with_loss else None
    dev, ref = (B.plx_bg_tv_grad, O.bg_tv) if bg else (B.plx_tv_grad, O.tv)
    dev(gg.desc(), start, count, 0.9, 1.3, 1e-9, grad, touched, loss)
    torch.cuda.synchronize()
    l_ref, gd, gs, t_ref = ref(og, start, count, 0.9, 1.3, 1e-9)
    assert loss is None or abs(loss.item() - l_ref) <= 1e-5 * abs(l_ref)
    assert_touched_equal(touched, t_ref, "tv")
    assert_grads_close(grad, gd, gs, "tv")
