"""How the copy of a concatenation model's dense part is dealt to waves.  Host code only: no device."""
import pytest

from paper_2203_07424_amd import binding as b


@pytest.mark.parametrize("columns", [0, 1, 7, 24, 32, 33, 64, 65, 100, 1000, 2560])
@pytest.mark.parametrize("rows", [1, 63, 300, 1003, 4096, 30000])
@pytest.mark.parametrize("left", [-1, 0, 21, 200])
def test_a_wave_has_a_few_accesses_of_any_shape(rows, columns, left):
    pad = -columns % 64
    st, blocks, waves, units = b.rec_probe_dense_copy(rows, columns, pad, left)
    assert st == b.REC_OK and (blocks > 0) == (columns + pad > 0)
    # Two units a wave, or up to twelve beside lookups, where blocks fit the compute units these leave; in the launch of the scan that has
    # 256 blocks at most what these are for.  A unit is 256 elements, half of them unused where columns are no power of two.
    most = 256 * 4
    elements = rows * columns + rows * pad
    assert units <= (max(2, 2 * -(-elements // (256 * most)) + 1) if left < 0 else 12)
    if 0 <= left < blocks:
        assert units <= 4 and b.rec_probe_dense_copy(rows, columns, pad, 10 ** 6)[1] * 2 + 2 > 12 * left
    assert units * blocks * waves * 256 <= 4 * (elements + 256 * 2 * 64)


def test_no_copy_is_refused():
    assert b.rec_probe_dense_copy(0, 64, 0)[0] == b.rec_probe_dense_copy(1, -1, 0)[0] == b.REC_ERR_ARG
    assert b.rec_probe_dense_copy(1, 64, 64)[0] == b.rec_probe_dense_copy(1, 64, 0, -2)[0] == b.REC_ERR_ARG
