"""The plane GEMM's rounding has no direction.

The 16-bit matrix instructions round a little downwards where products and accumulator are alike in
size (2% of 2^-24 of the result each).  An error with a direction is the same in every slice: S slices
add S of it and only sqrt(S) of a chance error.  So the mean error of a product's components is
compared with their spread: at most 1 / sqrt(S) of it, for complex64 with S = 1024 (a 30-qubit sum),
for the two-plane forms with S = 64, plus 4 standard deviations of the mean itself."""

import os

import numpy as np
import pytest

from tests.gpu_util import log, random_pair_network, require_gpu
from tests.test_gpu_parity import _grouped_pair, _grouped_reference


def _check(got, ref, precision, name):
    d = np.asarray(got - ref).reshape(-1)
    d = np.r_[d.real, d.imag]
    rms = np.sqrt(np.mean(d * d))
    bound = (1.0 / 32 if precision == 0 else 1.0 / 8) + 4.0 / np.sqrt(d.size)
    log(f"{name} precision {precision}: mean error {d.mean() / rms:+.4f} of its spread (bound {bound:.4f})")
    assert abs(d.mean()) <= bound * rms


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("nk", [5, 6, 8, 10, 12])
def test_products(nk, precision):
    require_gpu()
    from paper_2111_03011_amd.contractor import Contraction
    net = random_pair_network(9 + nk, 8 + nk, nk, 40 + nk)
    os.environ["TNC_GEMM_CONFIG"], os.environ["TNC_SPLITK_BLOCKS"] = "8", "1"
    try:
        c = Contraction(net, [(0, 1)], open_qubits=list(range(net.n_qubits)), closed_bits=[0],
                        precision=precision)
    finally:
        os.environ.pop("TNC_GEMM_CONFIG")
        os.environ.pop("TNC_SPLITK_BLOCKS")
    assert [(l.config, l.k_splits) for l in c.launches() if l.kind == 1] == [(8, 1)]
    c.contract()
    got = c.amps.cpu().numpy()[0].reshape(1 << 9, -1)
    c.close()
    a, b = (t.astype(np.complex64).astype(np.complex128) for t in net.tensors)
    _check(got, a.reshape(1 << 9, -1) @ b.reshape(1 << nk, -1), precision, f"K 2^{nk}")


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1, 2])
def test_stacked_rows(precision):
    require_gpu()
    from paper_2111_03011_amd.contractor import Contraction
    net, open_q, closed = _grouped_pair(7, 2, 2, 8, 9, 201, seed=5)
    net.tensors = [t.astype(np.complex64).astype(np.complex128) for t in net.tensors]
    c = Contraction(net, [(0, 1)], open_qubits=open_q, closed_bits=closed, precision=precision)
    assert [(l.config, l.row_mode) for l in c.launches() if l.kind == 1] == [(8, 2)]
    c.contract()
    got = c.amps.cpu().numpy()
    c.close()
    _check(got, _grouped_reference(net, open_q, closed), precision, "stacked rows, K 2^9")


@pytest.mark.gpu
def test_fp16_chains_are_as_short_as_the_tile_kernels():
    """FP16 planes and the 128 x 64 tile kernel round as often per product, so a sliced step errs as
    much on either (1.05 for chance: 2^18 components) when their chains are as long: planes in chunks
    of 1024 close theirs every 256 k."""
    require_gpu()
    from paper_2111_03011_amd import tnc
    from paper_2111_03011_amd.contractor import Contraction
    net = random_pair_network(9 + 14, 8 + 14, 14, 8)
    a, b = (t.astype(np.complex64).astype(np.complex128) for t in net.tensors)
    ref = a.reshape(1 << 9, -1) @ b.reshape(1 << 14, -1)
    err = []
    for force in ("0", None):
        if force:
            os.environ["TNC_GEMM_CONFIG"] = force
        try:
            c = Contraction(net, [(0, 1)], sliced_labels=[0, 1, 2, 3], slice_ids=list(range(16)),
                            max_batch_slices=16, open_qubits=list(range(net.n_qubits)), closed_bits=[0], precision=tnc.TNC_FP16X3)
        finally:
            os.environ.pop("TNC_GEMM_CONFIG", None)
        g, = [l for l in c.launches() if l.kind == 1]
        assert (g.config, g.k, g.k_splits) == (0, 1 << 10, 4) if force else (8, 1 << 10, 1)
        c.contract()
        err.append(np.linalg.norm(c.amps.cpu().numpy()[0] - ref.reshape(-1)) / np.linalg.norm(ref))
        c.close()
    log(f"FP16x3, K 2^10: tile kernel {err[0]:.2e}, planes {err[1]:.2e}")
    assert err[1] <= 1.05 * err[0]


@pytest.mark.parametrize("nm,nn,nk,slices,splits", [
    (9, 9, 10, 8, 1), (9, 9, 10, 4, 4), (10, 9, 10, 4, 1), (10, 9, 10, 2, 4), (9, 8, 11, 8, 2), (9, 8, 11, 4, 8)])
def test_splits_follow_the_plans_slices(nm, nn, nk, slices, splits):
    """Chunks of 1024 where all slices together have a workgroup for each of the 256 CUs, whatever
    the batch; else of 256."""
    from paper_2111_03011_amd import tnc
    from paper_2111_03011_amd.network import TensorNetwork
    bits = slices.bit_length() - 1
    k = list(range(nk + bits))
    fa, fb = list(range(nk + bits, nk + bits + nm)), list(range(nk + bits + nm, nk + bits + nm + nn))
    ones = [np.broadcast_to(np.complex128(1.0), (2,) * len(x)) for x in (fa + k, k + fb)]
    net = TensorNetwork(n_qubits=nm + nn, tensors=ones, labels=[fa + k, k + fb], out_label=fa + fb, bond_label={})
    h = tnc.tnc_net_create(0, net.n_qubits, net.ranks(), net.flat_labels(), net.flat_data(), net.out_label)
    tnc.tnc_net_set_path(h, [(0, 1)])
    tnc.set_slices_any(h, list(range(bits)), np.arange(slices, dtype=np.uint64))
    tnc.tnc_net_set_targets(h, list(range(net.n_qubits)), [0])
    for precision, batch in ((tnc.TNC_C64, 1), (tnc.TNC_C64, slices), (tnc.TNC_BF16X3, 1), (tnc.TNC_FP16X3, slices)):
        p = tnc.tnc_plan_create(h, precision, batch)
        g, = [i for i in (tnc.tnc_plan_launch_info(p, j) for j in range(tnc.tnc_plan_n_launches(p))) if i.kind == 1]
        assert g.config in (7, 8) and g.k_splits == splits
        tnc.tnc_plan_destroy(p)
    tnc.tnc_net_destroy(h)
