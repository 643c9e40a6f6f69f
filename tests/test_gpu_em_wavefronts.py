"""The patch classification where its launch changes from four wavefronts to eight
and to sixteen, and where a lane's last round of patches is partly empty, against
the FP64 oracle: the check and the bar of test_gpu_em_sizes."""
import pytest

from test_gpu_em_sizes import test_weights as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(300,), (512, 5), (1153, 1), (1279,), (1280, 300), (1281,), (2047, 1),
                                   (2049,), (4095,), (4096, 64)])
def test_weights_where_the_launch_changes(sizes):
    check(sizes)
