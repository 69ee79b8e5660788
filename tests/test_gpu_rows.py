"""The row-product kernel (gemm_rows.hip) at the edges of its range: every shape of 1024 outputs, K
from 16 to 64, ragged numbers of rows, an operand shared by many rows or none, gathered or not.

Tolerances (normwise): complex64 adds 2 K <= 128 products per component, each rounded at 2^-24 of a
partial sum with random signs, 2^-24 sqrt(128) = 6.7e-7; the split forms' operand splits and products
are the tile kernels', 2^-15 for two BF16 planes and 2^-20 for two FP16.  A power of two on an operand
changes its record and its rescaling only, so it comes out as an exact factor."""

import numpy as np
import pytest

from oracle import metrics
from tests.gpu_util import log, require_gpu
from tests.test_gpu_parity import _grouped_pair, _grouped_reference

# closed on A, open on A, closed on B, open on B, contracted labels, groups
CASES = [(5, 6, 4, 4, 6, 300), (4, 4, 5, 6, 6, 512), (6, 5, 6, 5, 5, 257), (9, 5, 1, 5, 6, 1000),
         (0, 6, 9, 4, 5, 400), (9, 4, 1, 6, 6, 1000), (5, 5, 4, 5, 4, 511)]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("case", CASES)
def test_row_products(case, precision):
    require_gpu()
    from paper_2111_03011_amd.contractor import Contraction
    net, open_q, closed = _grouped_pair(*case, seed=sum(case))
    ref = _grouped_reference(net, open_q, closed)
    out = []
    for scale in (1.0, 2.0 ** -70):
        if scale != 1.0:
            net.tensors[1] = net.tensors[1] * scale
        c = Contraction(net, [(0, 1)], open_qubits=open_q, closed_bits=closed, precision=precision)
        g = [l for l in c.launches() if l.kind == 1]
        assert len(g) == 1 and g[0].m * g[0].n == 1024 and g[0].rows == case[5]
        assert (g[0].config == 9) == (precision == 0 or case[4] >= 5)
        c.contract()
        out.append(c.amps.cpu().numpy().copy())
        c.close()
    err = metrics.rel_error(out[0], ref)
    log(f"row products {case} precision {precision}: config {g[0].config} rel err {err:.2e}")
    assert err <= {0: 2.0 ** -24 * np.sqrt(128), 1: 2.0 ** -20, 2: 2.0 ** -15}[precision]
    assert np.array_equal(out[1], out[0] * 2.0 ** -70)
