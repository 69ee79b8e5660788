"""Which rows of a grouped product stack: the plan on the host, the product on the GPU.

A product whose rows hold 128 and more m each has its tiles to itself, whichever operand comes
first and however few of its rows would fill a block of the other orientation.  Tolerances
(normwise): complex64 adds 2 K products per component, each rounded at 2^-24 of a partial sum with
random signs, 2^-24 sqrt(2 K); the split forms drop products below 2^-15 (two BF16 planes) and
2^-20 (two FP16 planes)."""

import numpy as np
import pytest

from oracle import metrics
from paper_2111_03011_amd import tnc
from tests.gpu_util import log, require_gpu
from tests.test_gpu_parity import _grouped_pair, _grouped_reference


def plan_gemms(net, open_q, closed, precision=tnc.TNC_C64, batch=1):
    """The GEMM launches of a two-tensor network's plan."""
    h = tnc.tnc_net_create(0, net.n_qubits, net.ranks(), net.flat_labels(), net.flat_data(),
                           net.out_label)
    tnc.tnc_net_set_path(h, [(0, 1)])
    tnc.tnc_net_set_targets(h, open_q, closed)
    p = tnc.tnc_plan_create(h, precision, batch)
    infos = [tnc.tnc_plan_launch_info(p, i) for i in range(tnc.tnc_plan_n_launches(p))]
    tnc.tnc_plan_destroy(p)
    tnc.tnc_net_destroy(h)
    return [i for i in infos if i.kind == 1]


# closed on A, open on A, closed on B, open on B, contracted labels, groups: few rows share a row of
# B, so 64-row blocks of A's m would stay empty, and B (2^7 to 2^9 m) takes the M side
LOW_FILL = [(6, 0, 6, 8, 6, 70), (6, 2, 6, 7, 6, 100), (4, 0, 4, 9, 8, 40), (5, 1, 6, 7, 5, 65)]


@pytest.mark.parametrize("case", LOW_FILL)
def test_whole_tiles_are_not_stacked(case):
    n_ca, n_oa, n_cb, n_ob, nk, groups = case
    for c in (case, (n_cb, n_ob, n_ca, n_oa, nk, groups)):
        g, = plan_gemms(*_grouped_pair(*c, seed=sum(c)))
        assert g.m == 1 << n_ob and g.rows == groups
        assert g.row_mode == 0


@pytest.mark.parametrize("case,config,mode,m", [
    ((9, 5, 9, 6, 5, 1 << 18), 8, 2, 32),      # 2^18 rows of 32: M = 2^23, the plane kernel's largest launch
    ((9, 5, 10, 6, 5, 266240), 2, 0, 64),      # beyond it the tile kernels, the other operand on the M side
])
def test_stacked_rows_up_to_the_largest_launch(case, config, mode, m):
    net, open_q, _ = _grouped_pair(*case[:5], 2, seed=3)
    closed_q = [q for q in range(net.n_qubits) if q not in open_q]
    rows = np.arange(case[5], dtype=np.uint64)
    closed = np.zeros(case[5], np.uint64)
    for b, q in enumerate(closed_q[::-1]):
        closed |= ((rows >> np.uint64(b)) & np.uint64(1)) << np.uint64(net.n_qubits - 1 - q)
    for precision in (tnc.TNC_C64, tnc.TNC_BF16X3, tnc.TNC_FP16X3):
        g, = plan_gemms(net, open_q, closed, precision)
        assert (g.config, g.row_mode, g.rows, g.m) == (config, mode, case[5], m)


@pytest.mark.parametrize("case,stacked", [
    ((3, 3, 0, 8, 8, 8), True), ((3, 3, 0, 8, 9, 8), False), ((1, 5, 0, 6, 13, 2), False),
    ((6, 5, 2, 6, 11, 40), True), ((9, 5, 4, 8, 9, 1000), True),
])
def test_a_long_contraction_keeps_its_splits(case, stacked):
    """Rows stack on the plane kernel, which leaves K whole, only where the tile kernels leave it
    whole too: K below 512 or enough tiles."""
    for precision in (tnc.TNC_C64, tnc.TNC_BF16X3, tnc.TNC_FP16X3):
        g, = plan_gemms(*_grouped_pair(*case, seed=4), precision)
        assert (g.config == 8 and g.row_mode == 2) == stacked
        assert (g.k_splits > 1) == (not stacked)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("case", LOW_FILL)
def test_whole_tiles_in_either_operand_order(case, precision):
    require_gpu()
    from paper_2111_03011_amd.contractor import Contraction
    n_ca, n_oa, n_cb, n_ob, nk, groups = case
    for c in (case, (n_cb, n_ob, n_ca, n_oa, nk, groups)):
        net, open_q, closed = _grouped_pair(*c, seed=sum(c))
        k = Contraction(net, [(0, 1)], open_qubits=open_q, closed_bits=closed, precision=precision)
        assert [l.row_mode for l in k.launches() if l.kind == 1] == [0]
        k.contract()
        err = metrics.rel_error(k.amps.cpu().numpy(), _grouped_reference(net, open_q, closed))
        k.close()
        log(f"row modes {c} precision {precision}: {err:.2e}")
        assert err <= {0: 2.0 ** -24 * np.sqrt(2 << nk), 1: 2.0 ** -20, 2: 2.0 ** -15}[precision]
