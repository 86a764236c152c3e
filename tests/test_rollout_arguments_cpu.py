"""Arguments that a rollout refuses before it touches the device."""
from __future__ import annotations

import pytest
import torch

from paper_1609_01479_amd.rollout import rollout


@pytest.mark.parametrize("interval", [-1, -3, 0.5])
def test_checkpoint_interval_below_one_is_refused(interval):
    """(A negative one would take no step at all.)"""
    with pytest.raises(ValueError, match="interval"):
        rollout(torch.zeros(4, 4, 4, dtype=torch.float64), -0.00625, 0.00625, 0.004, 4,
                interval=interval)
