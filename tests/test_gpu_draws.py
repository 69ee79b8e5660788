"""The sampling kernels' routes (one workgroup, running sums and search apart, groups in LDS, groups
in memory) at their edges, draw for draw against the oracle: both sides round every weight, sum and
product in FP64 in the same order, so the bits are the same."""

import numpy as np
import pytest

import synth
from oracle import sampling
from tests.gpu_util import log, require_gpu

# open qubits, groups, draws: one weight and a partial block; a tile and two of them; more than two
# (sums in memory); draws up to and beyond one workgroup's; groups down to one weight, a ragged last
# workgroup, groups that fill LDS and that it does not hold
CASES = [(0, 1, 3), (3, 1, 100), (4, 1, 1), (11, 1, 4096), (12, 1, 1000), (12, 1, 4097), (13, 1, 700),
         (14, 1, 70000), (0, 300, 300), (3, 2, 2), (6, 1001, 1001), (10, 33, 33), (12, 5, 5), (13, 3, 3)]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
def test_draws_match_oracle(case):
    require_gpu()
    import torch

    from paper_2111_03011_amd.contractor import Contraction
    from paper_2111_03011_amd.workload import make_workload
    n_open, groups, draws = case
    log(f"draws {case}")
    n = max(4, n_open + max(1, (groups - 1).bit_length()))
    n += n % 2
    circ = synth.make_circuit(2, n // 2, 2, 5)
    open_q = list(range(n - n_open, n))
    w = make_workload(circ, open_q, synth.group_targets(n, open_q, groups, 6), trials=1, n_sliced=0)
    c = Contraction(w.net, w.plan.path, open_qubits=w.open_qubits, closed_bits=w.closed_bits)
    rng = np.random.default_rng(n_open)
    x = rng.standard_normal((groups, 1 << n_open, 2)) * 2.0 ** -15
    x[rng.random(x.shape[:2]) < 0.1] = 0.0
    if groups > 1:
        x[1] = 0.0                       # a group without weight draws uniformly
    amps = x[..., 0] + 1j * x[..., 1]
    c.amps.copy_(torch.from_numpy(amps).reshape(c.amps.shape))
    got = c.sample(11, draws)
    c.close()
    want = sampling.bitstrings(sampling.sample(amps, 11, draws), w.closed_bits, w.open_qubits,
                               w.net.n_qubits)
    assert np.array_equal(got, want)


@pytest.mark.gpu
@pytest.mark.parametrize("draws", [2047, 2048, 2049])
def test_draws_on_both_sides_of_one_workgroup(draws):
    test_draws_match_oracle((12, 1, draws))
