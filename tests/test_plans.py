"""Which stages of an untimed forward share a launch, by option and batch.  Host code
only: no device (the library counts 256 compute units until it has seen one)."""
import pytest

from paper_2203_07424_amd import binding as b

RIDE, FRONT, LAYER, TAIL = b.REC_PLAN_RIDE, b.REC_PLAN_FRONT, b.REC_PLAN_LAYER, b.REC_PLAN_TAIL


def plan(batch, tables=10, dim=32, dense=2560, bottom=(1024, 256, 32), hidden=(512, 256), ids=20, concat=False, fuse=1, overlap=0):
    z = (list(bottom) or [dense])[-1] + tables * dim if concat else dim + tables * (tables + 1) // 2
    st, m = b.rec_create(num_tables=tables, emb_dim=dim, rows=[1000] * tables, table_dtype=b.REC_F32, num_dense=dense,
                         bottom_widths=[dense, *bottom], top_widths=[z, *hidden, 1], max_batch=batch, max_nnz=tables * batch * ids,
                         interaction=b.REC_INTERACT_CONCAT if concat else b.REC_INTERACT_DOT)
    assert st == b.REC_OK
    assert b.rec_set_option(m, b.REC_OPT_FUSE_MLP, fuse) == b.REC_OK
    assert b.rec_set_option(m, b.REC_OPT_OVERLAP_DENSE, overlap) == b.REC_OK
    assert b.rec_probe_plan(m, batch + 1, 0)[0] == b.rec_probe_plan(m, batch, -1)[0] == b.REC_ERR_ARG
    st, mask, tail_from = b.rec_probe_plan(m, batch, tables * batch * ids)
    assert st == b.REC_OK
    b.rec_destroy(m)
    return mask, tail_from


def test_no_model_is_refused():
    assert b.rec_probe_plan(None, 1, 1)[0] == b.REC_ERR_ARG


@pytest.mark.parametrize("batch,overlap", [(1, 0), (300, 0), (700, 0), (2500, 0), (4096, 0), (300, 1), (4096, 1)])
def test_layer_by_layer_every_layer_has_its_own_launch(batch, overlap):
    assert plan(batch, fuse=0, overlap=overlap) == (0, 3)
    assert plan(batch, fuse=0, dense=256, bottom=(256, 32), overlap=overlap) == (0, 2)
    assert plan(batch, fuse=0, dense=32, bottom=(), overlap=overlap) == (0, 0)
    assert plan(batch, fuse=0, dense=64, bottom=(64,), ids=1, concat=True, overlap=overlap) == (0, 1)
    # no layer involved: the narrowing of the dense part
    assert plan(batch, fuse=0, dense=64, bottom=(), ids=1, concat=True, overlap=overlap)[0] == (FRONT if batch * 10 <= 12288 else 0)


@pytest.mark.parametrize("batch,mask", [(1, FRONT | LAYER | TAIL), (300, FRONT | LAYER | TAIL), (1500, LAYER | TAIL), (4096, LAYER | TAIL)])
def test_first_layer_beside_the_sparse_side(batch, mask):
    assert plan(batch)[0] == mask


@pytest.mark.parametrize("batch", [1, 300, 3000, 4096])
def test_wherever_the_shapes_allow_is_not_a_matter_of_weights(batch):
    """1024 -> 256 is 512 KiB: left to itself the joint Predict-FC launch takes it from some
    samples a compute unit on; told to, at any batch."""
    assert plan(batch, fuse=2)[1] == 1
    assert plan(batch)[1] == (2 if batch <= 8 * 256 else 1)


@pytest.mark.parametrize("batch,dense,mask", [(1536, 1536, FRONT | LAYER | TAIL), (1600, 1536, LAYER | TAIL), (1790, 2560, LAYER | TAIL)])
def test_a_layer_in_tiles_of_64_rows_leaves_pooling_its_launch(batch, dense, mask):
    assert b.rec_probe_fc_form(batch, dense, 1024, 1, b.REC_FC_ANY_ORDER | b.REC_FC_F32_ROWS)[1][1] == (64 if batch > 1536 else 32)
    assert plan(batch, tables=4, dense=dense)[0] == mask
