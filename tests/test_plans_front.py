"""Up to which batch scan, a whole Bottom-FC and pooling share a launch (no device)."""
import pytest

from test_plans import FRONT, RIDE, plan


@pytest.mark.parametrize("dense,batch,front", [(512, 1, True), (512, 716, True), (512, 1792, True), (512, 1793, False),
                                               (513, 896, True), (513, 897, False)])
def test_bags_of_the_joint_launch(dense, batch, front):
    mask, _ = plan(batch, tables=8, dim=64, dense=dense, bottom=(64,), hidden=(64,), fuse=2)
    assert mask & RIDE and bool(mask & FRONT) == front
