"""The scratch of batches in ray order is bounded: by bytes, and by the samples
that a ray of the grid can have (host arithmetic; no GPU)."""
import pytest

from paper_2112_05131_amd import binding as B


def _grid(reso, n_vox=0, step_voxels=0.5, size=1.0):
    g = B.PlxGrid()
    g.reso[:] = reso
    g.scale[:] = [r / size for r in reso]
    g.step = step_voxels * size / max(reso)
    g.n_vox = n_vox
    return g


@pytest.mark.parametrize("n", [0, 1, 5000, 13107, 16000, 65537, 300000, 1600000, 8 << 20])
def test_kept_samples_are_bounded_by_bytes(n):
    cap = B.ray_cap(n, _grid((512, 512, 512)))
    assert 1 <= cap <= B.RAY_CAP and cap == B.ray_cap(n)
    # one sample a ray at least; indices and values are each padded to 256 bytes
    assert B.plx_rays_samp_bytes(n, cap) <= max(B.RAY_SAMP_BYTES, 20 * n) + 512
    assert (cap == B.RAY_CAP) == (n <= B.RAY_SAMP_BYTES // (20 * B.RAY_CAP))
    assert B.plx_rays_ray_bytes(n) <= 52 * n + 512


def test_a_large_batch_on_an_almost_empty_grid():
    """Few voxels send a batch of any size to ray order: its scratch is then
    about what its segment lists' per-ray part is."""
    g = _grid((512, 512, 512), n_vox=100)
    n = 8 << 20
    assert B.ray_order(g, n)
    total = B.plx_rays_ray_bytes(n) + B.plx_rays_samp_bytes(n, B.ray_cap(n, g))
    assert total < 1 << 30


@pytest.mark.parametrize("reso,step,size", [((64, 64, 64), 0.5, 1.0), ((33, 17, 128), 0.5, 2.0), ((64, 64, 64), 0.1, 1.0)])
def test_kept_samples_are_bounded_by_the_diagonal(reso, step, size):
    g = _grid(reso, step_voxels=step, size=size)
    diag = sum(((r - 1) * size / r) ** 2 for r in reso) ** 0.5
    most = int(diag / (step * size / max(reso))) + 2  # samples of a ray along it
    assert B.ray_cap(100, g) == min(B.RAY_CAP, most)


def test_grids_that_the_calls_refuse_still_get_a_cap():
    for g in (_grid((8, 8, 8), step_voxels=0.0), B.PlxGrid()):
        assert B.ray_cap(10, g) == B.RAY_CAP
