"""A round of a batch is one launch: one block more than a grid's x dimension
takes (2^31 - 1) is refused when the schedule is made, not by the launch."""
import pytest

from paper_1804_04797_amd import qsv


@pytest.mark.parametrize("n_qubits", [[30] * 4, [30] * 4 + [20]])
def test_too_many_tiles_in_a_round(n_qubits):
    with pytest.raises(qsv.QsvError) as e:
        qsv.sv_debug_batch_schedule(n_qubits, [1] * len(n_qubits), 1, 4)
    assert e.value.status == 2  # QSV_ERANGE


def test_the_limit_is_per_round():
    assert qsv.sv_debug_batch_schedule([12] * 5, [3, 1, 2, 0, 3], 4, 4) == 9 << 8
