"""Which kernel the launch of an FC layer takes, by the shapes at which the choice was
measured.  Host code only: no device."""
import pytest

from paper_2203_07424_amd import binding as b

CUS = 256
ALONE = b.REC_FC_ANY_ORDER
PIPELINED = b.REC_FC_BESIDE_POOLING


def form(rows, inputs, outputs, stacks=1, flags=ALONE):
    st, f = b.rec_probe_fc_form(rows, inputs, outputs, stacks, flags, CUS)
    assert st == b.REC_OK
    return f


def test_what_is_no_layer_is_refused():
    for bad in ((0, 64, 64, 1), (1, 0, 64, 1), (1, 64, 0, 1), (1, 64, 64, 0), (1, 64, 64, b.REC_MAX_TOWERS + 1), (1, 2 ** 20 + 1, 64, 1),
                (2 ** 30 + 1, 64, 64, 1)):
        assert b.rec_probe_fc_form(*bad)[0] == b.REC_ERR_ARG
    assert b.rec_probe_fc_form(1, 64, 64, 1, 0, 0)[0] == b.REC_ERR_ARG
    assert b.rec_probe_fc_form(1, 64, 320, 1, b.REC_FC_DOT)[0] == b.REC_ERR_ARG
    assert form(2 ** 30, 2 ** 20, 2 ** 20, b.REC_MAX_TOWERS)[0] != b.REC_FORM_SPLIT  # offsets beyond 32 bits
    for rows in (1, 2 ** 30):
        for flags in range(16):
            b.rec_probe_fc_form(rows, 2048, 256, 1, flags, 1)


@pytest.mark.parametrize("rows", [4097, 4500, 6016])
def test_one_stack_beside_pooling_keeps_its_small_blocks(rows):
    """132 to 188 tiles of 128 x 128: eight waves and 72 KB each, no room beside pooling."""
    assert form(rows, 884, 512, flags=PIPELINED)[0] == b.REC_FORM_TILES
    assert form(rows, 884, 512)[0] == b.REC_FORM_WIDE
    assert form(6200, 884, 512, flags=PIPELINED)[0] == b.REC_FORM_WIDE  # three quarters of a round


@pytest.mark.parametrize("rows,inputs,outputs,stacks,flags", [
    (2049, 2560, 1024, 1, b.REC_FC_F32_ROWS), (2944, 2560, 1024, 1, b.REC_FC_F32_ROWS), (520, 1728, 1024, 4, 0), (1000, 1728, 1024, 4, 0)])
def test_fp32_rows_and_several_stacks_take_wide_tiles_beside_pooling(rows, inputs, outputs, stacks, flags):
    assert form(rows, inputs, outputs, stacks, flags | PIPELINED)[0] == b.REC_FORM_WIDE


@pytest.mark.parametrize("inputs,outputs,stacks,most", [
    (256, 64, 1, 8192), (2048, 64, 4, 8192), (1024, 50, 1, 8192),   # two rounds of blocks of 16 rows
    (256, 256, 1, 8192), (448, 256, 1, 8192), (512, 256, 4, 16384), (2048, 250, 1, 16384)])
def test_the_dot_layer_on_many_samples_is_left_to_the_k_tiles(inputs, outputs, stacks, most):
    assert form(most // stacks, inputs, outputs, stacks, ALONE | b.REC_FC_DOT)[0] == b.REC_FORM_SPLIT
    for rows in (most + 16 * stacks, 2 * most, 8 * most):
        assert form(rows // stacks, inputs, outputs, stacks, ALONE | b.REC_FC_DOT)[0] == b.REC_FORM_TILES


@pytest.mark.parametrize("rows,tile", [(1, 16), (4096, 16), (4097, 32), (8192, 32), (65536, 32)])
def test_blocks_of_the_dot_layer_with_128_columns(rows, tile):
    assert form(rows, 512, 128, flags=ALONE | b.REC_FC_DOT) == (b.REC_FORM_SPLIT, tile, 128, 4)


@pytest.mark.parametrize("rows,inputs,outputs,stacks", [
    (40960, 256, 192, 1), (40960, 256, 448, 1), (32768, 1024, 704, 1), (16384, 2048, 448, 4), (65536, 256, 704, 1)])
def test_blocks_of_80_rows_only_in_one_round(rows, inputs, outputs, stacks):
    f = form(rows, inputs, outputs, stacks)
    assert f[0] != b.REC_FORM_SPLIT or f[1] == 64
    assert form(300, 1728, 1024, 4) == (b.REC_FORM_SPLIT, 80, 64, 8)


@pytest.mark.parametrize("rows,outputs,tile,from_inputs", [
    (3000, 512, 48, 384), (10000, 64, 48, 1152), (1536, 704, 80, 512), (20480, 64, 80, 512),
    (1000, 1024, 64, 576), (2048, 448, 64, 576), (16384, 64, 64, None), (16384, 128, 64, 1536)])
def test_tiles_of_more_than_32_rows_need_enough_k(rows, outputs, tile, from_inputs):
    for inputs in (64, 128, 192, 256, 320, 384, 448, 512, 576, 704, 768, 1088, 1152, 1472, 1536, 2048):
        f = form(rows, inputs, outputs)
        if from_inputs and inputs >= from_inputs:
            assert f[:3] == (b.REC_FORM_SPLIT, tile, 64), (inputs, f)
        else:
            assert f[0] == b.REC_FORM_TILES, (inputs, f)


@pytest.mark.parametrize("rows,outputs,takes", [(4096, 448, {512, 576, 768, 2048}), (16384, 448, {256, 512, 576, 768, 2048})])
def test_64_rows_and_four_waves_by_units_of_k(rows, outputs, takes):
    for inputs in (64, 128, 192, 256, 320, 384, 448, 512, 576, 768, 2048):
        assert form(rows, inputs, outputs)[0] == (b.REC_FORM_SPLIT if inputs in takes else b.REC_FORM_TILES), inputs


def test_up_to_32_rows_and_fp32_rows_at_any_k():
    for inputs in (64, 320, 2560):
        f = form(300, inputs, 512)
        assert f[0] == b.REC_FORM_SPLIT and f[1] <= 32
        for rows, outputs in ((3000, 256), (4096, 448), (2100, 512)):
            assert form(rows, inputs, outputs, flags=ALONE | b.REC_FC_F32_ROWS)[0] == b.REC_FORM_SPLIT


@pytest.mark.parametrize("cus", [64, 120, 256, 304])
def test_fp32_rows_never_in_64_rows_and_eight_waves(cus):
    """The kernel is not compiled for it."""
    for rows in [2 ** k + d for k in range(0, 17) for d in (-1, 0, 1, 2 ** k // 3) if 2 ** k + d > 0]:
        for outputs in (64, 192, 320, 512, 704, 1024, 2048, 4032):
            st, f = b.rec_probe_fc_form(rows, 2560, outputs, 1, ALONE | b.REC_FC_F32_ROWS, cus)
            assert st == b.REC_OK and f != (b.REC_FORM_SPLIT, 64, 64, 8)


def test_the_device_tests_run_every_form():
    """On 256 compute units: the shapes of the towers' tests take each tile that deals k, and those
    of the first layer each tile it rides in."""
    import test_gpu_first_layer as first
    import test_gpu_split as split
    plain, dots = set(), set()
    for rows, tables, dim, dense, hidden, towers in split.TOWERS:
        widths = (dense + tables * dim,) + hidden
        for i, n in enumerate(hidden):
            dot = i + 1 == len(hidden) and -(-n // 64) in (1, 2, 4)
            f = form(rows, widths[i], n, towers, ALONE | (b.REC_FC_DOT if dot else 0))
            if f[0] == b.REC_FORM_SPLIT:
                (dots if dot else plain).add(f[1:])
    assert plain == {(16, 16, 8), (16, 32, 8), (32, 32, 4), (32, 32, 8), (32, 64, 4), (32, 64, 8), (48, 64, 8), (64, 64, 4),
                     (64, 64, 8), (80, 64, 8)}
    assert dots == {(16, 64, 8), (16, 128, 4), (32, 128, 4), (16, 256, 2), (32, 256, 2), (64, 256, 2)}
    ride = {(r[7], r[8]) for r in first.POOLED}
    small = {(16, 16, 8), (16, 32, 8), (32, 32, 4), (32, 32, 8), (32, 64, 4), (32, 64, 8)}
    assert {t for w, t in ride if w == "pooling"} == small
    assert {t for w, t in ride if w == "scan"} >= {(32, 32, 4), (32, 64, 4), (48, 64, 8), (64, 64, 4), (80, 64, 8), (128, 128, 1)}
