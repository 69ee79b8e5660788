"""Slice ids as an array of their own type, as other arrays and as lists: one plan, one refusal."""

import numpy as np
import pytest

from paper_2111_03011_amd import tnc
from tests.gpu_util import random_pair_network


def _net():
    net = random_pair_network(6, 5, 3, 4)
    return tnc.tnc_net_create(0, net.n_qubits, net.ranks(), net.flat_labels(), net.flat_data(), net.out_label)


@pytest.mark.parametrize("ids", [np.arange(4, dtype=np.uint64), np.arange(8, dtype=np.uint64)[::2] // 2,
                                 np.arange(4, dtype=np.int32), [0, 1, 2, 3], range(4),
                                 np.arange(4, dtype=object)])
def test_forms_of_slice_ids(ids):
    h = _net()
    tnc.set_slices_any(h, [0, 1], ids)
    tnc.tnc_net_set_path(h, [(0, 1)])
    tnc.tnc_net_set_targets(h, list(range(5)), [0])
    p = tnc.tnc_plan_create(h, tnc.TNC_C64, 4)
    assert tnc.tnc_plan_work(p, 0, 4) > 0
    tnc.tnc_plan_destroy(p)
    tnc.tnc_net_destroy(h)


@pytest.mark.parametrize("ids", [np.array([0, 4], np.uint64), [0, 4], np.array([-1, 0])])
def test_ids_out_of_range_are_refused(ids):
    h = _net()
    with pytest.raises((tnc.TncError, OverflowError)):
        tnc.set_slices_any(h, [0, 1], ids)
    tnc.tnc_net_destroy(h)


@pytest.mark.parametrize("ids", [np.array([[0, 1], [2, 3]], np.uint64), np.matrix([0, 1], dtype=np.uint64),
                                 np.array(1, np.uint64), np.ma.array([0, 1], mask=[0, 1], dtype=np.uint64)])
def test_other_arrays_are_read_value_by_value(ids):
    """Rows of a matrix, an array without a dimension and a masked value are not slice ids."""
    h = _net()
    with pytest.raises((TypeError, ValueError, np.ma.MaskError)):
        tnc.set_slices_any(h, [0, 1], ids)
    tnc.tnc_net_destroy(h)
