"""The light gradient on both sides of the number of vertex workgroups up to which
the vertex gather finishes it (64), a workgroup a scene."""
import pytest

from test_gpu_light_sums import test_scenes_on_both_sides_of_the_rule as _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('n', [63, 64, 65])
def test_scenes_at_the_rule(n):
    _check(n)
