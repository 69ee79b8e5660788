"""What a plan reports of its launches is what runs them."""

import os

import numpy as np
import pytest

import synth
from paper_2111_03011_amd import tnc
from paper_2111_03011_amd.workload import make_workload
from tests.gpu_util import log, random_pair_network, require_gpu


def _infos(net, path, open_q, closed, precision=tnc.TNC_C64, slices=None, batch=1):
    h = tnc.tnc_net_create(0, net.n_qubits, net.ranks(), net.flat_labels(), net.flat_data(), net.out_label)
    tnc.tnc_net_set_path(h, path)
    if slices:
        tnc.set_slices_any(h, *slices)
    tnc.tnc_net_set_targets(h, open_q, closed)
    p = tnc.tnc_plan_create(h, precision, batch)
    infos = [tnc.tnc_plan_launch_info(p, i) for i in range(tnc.tnc_plan_n_launches(p))]
    tnc.tnc_plan_destroy(p)
    tnc.tnc_net_destroy(h)
    return infos


def test_fused_steps_say_so():
    circ = synth.make_circuit(3, 4, 8, 1001)
    closed = synth.group_targets(12, [], 64, 1002)
    w = make_workload(circ, [], closed, trials=2, seed=3)
    small = [i for i in _infos(w.net, w.plan.path, [], closed) if i.kind in (1, 2)]
    assert sum(i.config == 10 for i in small) >= 20
    os.environ["TNC_NO_FUSE"] = "1"
    try:
        apart = [i for i in _infos(w.net, w.plan.path, [], closed) if i.kind in (1, 2)]
    finally:
        os.environ.pop("TNC_NO_FUSE")
    assert len(apart) == len(small) and all(i.config < 10 for i in apart)
    assert all(i.config == 0 for i in apart if i.kind == 2)
    # the split forms fuse their streams alone
    for precision in (tnc.TNC_BF16X3, tnc.TNC_FP16X3):
        split = [i for i in _infos(w.net, w.plan.path, [], closed, precision) if i.kind in (1, 2)]
        assert any(i.config == 10 for i in split)
        assert all(i.config < 10 for i in split if i.kind == 1)


def test_fp16_sums_in_registers_are_the_small_tile():
    """2^9 x 2^9 x 2^10, 8 slices: chains of 1024; FP16 planes close them inside the 128 x 64 tile."""
    net = random_pair_network(9 + 13, 9 + 13, 13, 3)
    for precision, config in ((tnc.TNC_C64, 7), (tnc.TNC_BF16X3, 7), (tnc.TNC_FP16X3, 8)):
        g, = [i for i in _infos(net, [(0, 1)], list(range(18)), [0], precision,
                                ([0, 1, 2], np.arange(8, dtype=np.uint64)), 8) if i.kind == 1]
        assert (g.config, g.k, g.k_splits) == (config, 1 << 10, 1)


@pytest.mark.gpu
@pytest.mark.parametrize("nm,nn,planned,twin", [(8, 7, 7, 8), (7, 6, 8, 7)])
def test_autotuner_leaves_a_twin_kernel_alone(nm, nn, planned, twin):
    """Complex64 planes have one tile size, so the other configuration is not a choice."""
    require_gpu()
    from paper_2111_03011_amd.contractor import Contraction
    net = random_pair_network(nm + 10, nn + 10, 10, 3)
    c = Contraction(net, [(0, 1)], open_qubits=list(range(net.n_qubits)), closed_bits=[0])
    assert [l.config for l in c.launches() if l.kind == 1] == [planned]
    changed = c.autotune(reps=2)
    tuned = [l.config for l in c.launches() if l.kind == 1]
    log(f"2^{nm} x 2^{nn} x 2^10: planned {planned}, tuned {tuned}, {changed} changed")
    assert tuned != [twin]
    c.contract()
    ref = net.tensors[0].reshape(1 << nm, -1) @ net.tensors[1].reshape(1 << 10, -1)
    err = np.linalg.norm(c.amps.cpu().numpy()[0] - ref.reshape(-1)) / np.linalg.norm(ref)
    c.close()
    assert err <= 1e-5
