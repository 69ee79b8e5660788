"""Programs of small steps (program.hip) against the steps' own kernels, over forests of every
kind the planner makes: scalar rows, gathered rows of an odd number of groups, whole states,
slices alone, in odd batches and with a shared head, operands rescaled by their records.

Tolerances: the split forms' programs round as the stream kernels do, so their bits are the same;
in complex64 each of up to 120 steps adds at most 32 roundings of 2^-24 with random signs:
2^-24 sqrt(120 * 32) = 3.7e-6, and 1e-5 against the oracle as everywhere.  Powers of two on the
leaves change records and rescalings only, so they come out as an exact factor."""

import os

import numpy as np
import pytest

import synth
from oracle import contract as ocontract
from oracle import metrics
from tests.gpu_util import log, require_gpu

# rows, cols, cycles, open qubits, groups, sliced bonds, reuse batch
CASES = [(2, 2, 4, 0, 1, 0, 0), (2, 3, 6, 6, 1, 0, 0), (3, 4, 8, 0, 61, 0, 0), (3, 4, 8, 12, 1, 0, 0),
         (4, 4, 10, 4, 37, 3, 0), (4, 4, 14, 6, 5, 6, 8)]


def _workload(case):
    from paper_2111_03011_amd.workload import make_workload
    rows, cols, cycles, n_open, groups, sliced, reuse = case
    n = rows * cols
    circ = synth.make_circuit(rows, cols, cycles, 70 + cycles)
    open_q = list(range(n - n_open, n))
    closed = synth.group_targets(n, open_q, groups, 9)
    return make_workload(circ, open_q, closed, max_log2=14, n_sliced=sliced, trials=8, seed=5,
                         reuse_batch=reuse or 1)


def _run(w, precision, batch, fuse=True, first=0, count=None):
    from paper_2111_03011_amd.contractor import Contraction
    if not fuse:
        os.environ["TNC_NO_FUSE"] = "1"
    try:
        c = Contraction(w.net, w.plan.path, sliced_labels=w.plan.sliced_labels, slice_ids=w.slice_ids,
                        open_qubits=w.open_qubits, closed_bits=w.closed_bits, precision=precision,
                        max_batch_slices=batch)
    finally:
        os.environ.pop("TNC_NO_FUSE", None)
    if count is None:
        c.contract()
        first_pass = c.amps.cpu().numpy().copy()
        c.contract()
        got = c.amps.cpu().numpy().copy()
        assert np.array_equal(got, first_pass)
    else:
        c.contract_range(first, count)
        got = c.amps.cpu().numpy().copy()
    c.close()
    return got


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("case", CASES)
def test_program_matches_step_kernels(case, precision):
    require_gpu()
    log(f"program {case} precision {precision}")
    w = _workload(case)
    batch = case[6] or max(1, min(5, 1 << case[5]))
    got = _run(w, precision, batch)
    single = _run(w, precision, batch, fuse=False)
    if precision == 0:
        err = metrics.rel_error(got, single)
        ref = ocontract.sparse_amplitudes(w.circuit, w.open_qubits, w.closed_bits)
        log(f"  {err:.2e} from the steps' kernels, {metrics.rel_error(got, ref):.2e} from the oracle")
        assert err <= 3.7e-6 and metrics.rel_error(got, ref) <= 1e-5
    else:
        assert np.array_equal(got, single)
    if case[5] and not case[6]:      # bits do not depend on the batch
        assert np.array_equal(got, _run(w, precision, 1))
        assert np.array_equal(_run(w, precision, batch, first=1, count=6),
                              _run(w, precision, 2, first=1, count=6))
    # powers of two on the leaves
    exps = np.random.default_rng(3).integers(-60, 61, len(w.net.tensors))
    plain = list(w.net.tensors)
    for i, e in enumerate(exps):
        w.net.tensors[i] = plain[i] * 2.0 ** int(e)
    scaled = _run(w, precision, batch)
    assert np.array_equal(scaled, got * 2.0 ** int(exps.sum()))
