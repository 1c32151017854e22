"""Feature statistics on both sides of the row count from which two launches form them."""
import pytest

from test_gpu_mlp_rounds import mc  # noqa: F401
import test_gpu_mlp_rounds as rounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [19999, 20000, 20001])
def test_statistics_at_the_change_of_kernels(mc, n):  # noqa: F811
    rounds.test_feature_statistics(mc, n)
