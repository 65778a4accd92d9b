"""GPU test of the march of a list of rays on both sides of the lines between a
wave per ray and 16 lanes per ray, which depend on the storage type."""
import pytest

from paper_2112_05131_amd import binding as B
from tests.test_gpu_march import test_ray_order_gradients_match_oracle as ray_order_gradients

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sh_dtype,n,cap,priors", [(B.PLX_F32, 98303, 20, False), (B.PLX_F32, 98309, 512, True),
                                                   (B.PLX_F32, 98304, 20, False), (B.PLX_F16, 49151, 512, False),
                                                   (B.PLX_F16, 49153, 20, True), (B.PLX_BF16, 49157, 512, False)])
def test_ray_order_gradients_at_the_lines(sh_dtype, n, cap, priors):
    ray_order_gradients(sh_dtype, n, cap, 0.5, priors)
