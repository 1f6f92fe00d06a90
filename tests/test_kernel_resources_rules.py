"""Scratch and occupancy of the kernels that prepare the points' rules (no GPU needed): all of
them wait on dependent node loads, which eight waves a SIMD hide."""
import pytest

from test_kernel_resources import _find, usage  # noqa: F401  (usage: a fixture)


@pytest.mark.parametrize("pattern", [r"\d+k_horizonE", r"k_horizon_wideE", r"k_backface_prepE"])
def test_preparation_kernels(usage, pattern):  # noqa: F811
    for ru in _find(usage, pattern):
        assert ru["Occupancy"] >= 8, ru
        assert ru.get("ScratchSize", 0) == 0, ru
