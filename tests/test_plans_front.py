"""Up to which batch scan, a whole Bottom-FC and pooling share a launch (no device)."""
import pytest

from test_plans import FRONT, RIDE, plan


@pytest.mark.parametrize("dense,batch,front", [(512, 1, True), (512, 716, True), (512, 1792, True), (512, 1793, False),
                                               (513, 896, True), (513, 897, False)])
def test_bags_of_the_joint_launch(dense, batch, front):
    mask, _ = plan(batch, tables=8, dim=64, dense=dense, bottom=(64,), hidden=(64,), fuse=2)
    assert mask & RIDE and bool(mask & FRONT) == front


@pytest.mark.parametrize("tables,dim,batch,ids,front", [(26, 64, 472, 1, True), (26, 64, 473, 1, True), (26, 64, 2520, 1, True),
                                                        (26, 64, 2521, 1, False), (26, 32, 5041, 1, True), (26, 32, 5042, 1, False),
                                                        (26, 32, 600, 2, False)])
def test_lookups_of_the_joint_launch(tables, dim, batch, ids, front):
    """fp32 rows of 256 bytes in blocks of 256 bags, of 128 in blocks of 512, for 256 compute units."""
    mask, _ = plan(batch, tables=tables, dim=dim, dense=64, bottom=(), hidden=(64,), ids=ids, concat=True)
    assert bool(mask & FRONT) == front
