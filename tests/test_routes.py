"""CPU checks of the rules that pick a call's launches (route_check.cpp) and of where
the network's weight gradient loads (wgrad_check.cpp)."""
import os

import pytest

from tests.test_device_helpers import HIPCC, _run_check


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_rules():
    assert "failures 0" in _run_check("route_check")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_weight_gradient_loads_stay_inside():
    assert " failures 0" in _run_check("wgrad_check")
