"""Statistics that the workgroups put together themselves, counted in groups of 16 partial pairs: layers on both sides of a full
group, of 16 groups, and of the most groups a layer has (320 pairs), which is the line in pairs (5/4 workgroups per CU) as well;
beside layers of one pair."""
import pytest

import test_gpu_stats_fold as fold

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_layer", [[15], [16], [17], [16, 17, 1, 31, 32, 33], [255], [256], [257], [320], [321], [256, 64], [256, 65], [160, 1, 159],
                                       [20] * 16, [1] * 320, [1] * 321])
def test_groups(oracle, per_layer):
    fold.test_both_sides_of_the_line(oracle, per_layer)
