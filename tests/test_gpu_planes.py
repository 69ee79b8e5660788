"""The plane GEMM (gemm_planes.hip): operands split into 16-bit planes, at the edges of its range.

Tolerances (normwise), from the arithmetic: every value is its planes' sum up to 2^-24 (three BF16
planes: exact), 2^-16 (two BF16) or 2^-22 (two FP16), the dropped products are below those, and each
group of 16 products adds one FP32 rounding (2^-24) per plane pair; with random signs errors add in
quadrature, so 2^-15 and 2^-20 bound the two-plane forms and the FP32 matrix kernel's own error
(configuration 0, one rounding per product) bounds the three-plane one."""

import os

import numpy as np
import pytest

from tests.gpu_util import log, random_pair_network, require_gpu


def _orders(rng, n_free, shared, first):
    """Labels of an operand in a random order: shared labels 0.., free labels first.."""
    return [int(x) for x in rng.permutation(np.r_[np.arange(shared), np.arange(first, first + n_free)])]


def _run(net, config, precision, blocks="1"):
    from paper_2111_03011_amd.contractor import Contraction
    os.environ["TNC_GEMM_CONFIG"], os.environ["TNC_SPLITK_BLOCKS"] = str(config), blocks
    try:
        c = Contraction(net, [(0, 1)], open_qubits=list(range(net.n_qubits)), closed_bits=[0],
                        precision=precision)
    finally:
        os.environ.pop("TNC_GEMM_CONFIG")
        os.environ.pop("TNC_SPLITK_BLOCKS")
    g = [l for l in c.launches() if l.kind == 1]
    assert len(g) == 1 and g[0].config == config
    c.contract()
    got = c.amps.cpu().numpy()[0]
    c.close()
    return got, g[0].k_splits


def _exact(net):
    (ta, tb), (la, lb) = net.tensors, net.labels
    sh = [x for x in la if x in lb]
    r = np.tensordot(ta, tb, axes=([la.index(x) for x in sh], [lb.index(x) for x in sh]))
    lab = [x for x in la if x not in sh] + [x for x in lb if x not in sh]
    return r.transpose([lab.index(x) for x in net.out_label]).reshape(-1)


# (log2 M, log2 N, log2 K, scale of A, split-K blocks): one K tile pair, a tile smaller than the
# kernel's in each direction, exactly one, several; operands far from 1 (rescaled); split-K
CASES = [(7, 6, 5, 1.0, "1"), (8, 7, 5, 1.0, "1"), (6, 4, 6, 1.0, "1"), (9, 5, 7, 1.0, "1"),
         (5, 8, 6, 1.0, "1"), (10, 8, 9, 2.0 ** -70, "1"), (8, 7, 10, 2.0 ** 60, "100000")]


@pytest.mark.gpu
@pytest.mark.parametrize("config", [7, 8])
@pytest.mark.parametrize("case", CASES)
def test_plane_gemm_edges(case, config):
    require_gpu()
    nm, nn, nk, scale, blocks = case
    rng = np.random.default_rng(nm * 100 + nn * 10 + nk)
    net = random_pair_network(nm + nk, nn + nk, nk, 31 + nk, _orders(rng, nm, nk, nk),
                              _orders(rng, nn, nk, nk + nm))
    net.tensors[0] = net.tensors[0] * scale
    ref = _exact(net)
    err = lambda x: np.linalg.norm(x - ref) / np.linalg.norm(ref)
    fp32 = err(_run(net, 0, 0, blocks)[0])
    for precision, tol in ((0, fp32), (1, 2.0 ** -20), (2, 2.0 ** -15)):
        got, splits = _run(net, config, precision, blocks)
        assert (splits > 1) == (blocks != "1")
        log(f"planes {config} M 2^{nm} N 2^{nn} K 2^{nk} x{scale:g} precision {precision}: "
            f"{err(got):.2e} (bound {tol:.2e})")
        assert err(got) <= tol


@pytest.mark.gpu
@pytest.mark.parametrize("nn,nk", [(6, 10), (8, 12), (6, 13)])
def test_sixty_four_rows_by_a_long_contraction(nn, nk):
    """M = 64 and K >= 1024: the 64 x 64 tile in the split forms (bounds as above), by the plan's own
    choice and in as many splits as it makes; complex64 keeps the FP32 kernel."""
    from paper_2111_03011_amd.contractor import Contraction
    require_gpu()
    rng = np.random.default_rng(nn + nk)
    net = random_pair_network(6 + nk, nn + nk, nk, 17, _orders(rng, 6, nk, nk), _orders(rng, nn, nk, nk + 6))
    ref = _exact(net)
    for precision, tol in ((0, 1e-5), (1, 2.0 ** -20), (2, 2.0 ** -15)):
        c = Contraction(net, [(0, 1)], open_qubits=list(range(net.n_qubits)), closed_bits=[0],
                        precision=precision)
        g = [l for l in c.launches() if l.kind == 1]
        c.contract()
        err = np.linalg.norm(c.amps.cpu().numpy()[0] - ref) / np.linalg.norm(ref)
        c.close()
        log(f"M {g[0].m} N {g[0].n} K {g[0].k} precision {precision}: config {g[0].config}, {err:.2e}")
        if g[0].m == 64:                # 256 x 64 takes the 128 x 64 tile
            assert (g[0].config == 8) == (precision != 0)
        assert err <= tol


@pytest.mark.gpu
def test_plane_tiles_give_the_same_bits():
    """Both tile sizes add every output's products in one order, so a launch may take either."""
    require_gpu()
    rng = np.random.default_rng(3)
    net = random_pair_network(17, 15, 7, 5, _orders(rng, 10, 7, 7), _orders(rng, 8, 7, 17))
    for precision in (0, 1, 2):
        assert np.array_equal(_run(net, 7, precision)[0], _run(net, 8, precision)[0])


@pytest.mark.gpu
@pytest.mark.parametrize("n_oa", [7, 8])
def test_plane_gemm_folded_rows(n_oa):
    """Rows folded into M: 128-row and 256-row tiles inside one row; several rows, odd row count."""
    from oracle import contract as ocontract
    from paper_2111_03011_amd.contractor import Contraction
    from tests.test_host_logic import _grouped_pair_net
    require_gpu()
    net, open_q, closed = _grouped_pair_net(3, n_oa, 0, 7, 6, 5, seed=23)
    c = Contraction(net, [(0, 1)], open_qubits=open_q, closed_bits=closed)
    g = [l for l in c.launches() if l.kind == 1]
    assert len(g) == 1 and g[0].config in (7, 8) and g[0].row_mode == 1
    c.contract()
    got = c.amps.cpu().numpy()
    c.close()
    full = ocontract.contract_path(net.tensors, net.labels, [(0, 1)], net.out_label)
    n = net.n_qubits
    closed_q = [q for q in range(n) if q not in open_q]
    ref = []
    for bits in closed:
        at = tuple(((int(bits) >> (n - 1 - q)) & 1) if q in closed_q else slice(None) for q in range(n))
        rest = [q for q in range(n) if q in open_q]
        ref.append(np.transpose(full.reshape((2,) * n)[at], [rest.index(q) for q in open_q]).reshape(-1))
    err = np.linalg.norm(got - np.asarray(ref)) / np.linalg.norm(ref)
    log(f"folded rows, M 2^{n_oa}: {err:.2e}")
    assert err <= 1e-6


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("case", [(6, 3, 3, 6, 5, 60), (7, 0, 2, 7, 6, 250), (4, 5, 3, 6, 5, 37),
                                  (7, 2, 2, 8, 9, 201), (2, 7, 7, 1, 8, 90)])
def test_stacked_rows_on_planes(case, precision):
    """Rows below a tile that share the other operand's row, in 64-row blocks: M from 1 to 32, ragged
    blocks, either orientation.  Bounds as above, complex64 by its FP32 accumulation; a power of two
    on an operand comes out as an exact factor."""
    from paper_2111_03011_amd.contractor import Contraction
    from tests.test_gpu_parity import _grouped_pair, _grouped_reference
    require_gpu()
    net, open_q, closed = _grouped_pair(*case, seed=sum(case))
    ref = _grouped_reference(net, open_q, closed)
    out = []
    for scale in (1.0, 2.0 ** -60):
        if scale != 1.0:
            net.tensors[0] = net.tensors[0] * scale
        c = Contraction(net, [(0, 1)], open_qubits=open_q, closed_bits=closed, precision=precision)
        g = [l for l in c.launches() if l.kind == 1]
        assert len(g) == 1 and g[0].config == 8 and g[0].row_mode == 2
        c.contract()
        out.append(c.amps.cpu().numpy().copy())
        c.close()
    err = np.linalg.norm(out[0] - ref) / np.linalg.norm(ref)
    log(f"stacked rows {case} precision {precision}: {err:.2e}")
    assert err <= {0: 2.0 ** -24 * np.sqrt(2 << case[4]), 1: 2.0 ** -20, 2: 2.0 ** -15}[precision]
    assert np.array_equal(out[1], out[0] * 2.0 ** -60)


def test_non_finite_leaves_keep_the_fp32_kernels():
    """The split of an infinity is infinity and NaN, so a network holding one is not split."""
    from paper_2111_03011_amd import tnc
    for bad in (None, np.inf, -np.inf, np.nan, 1e300):     # 1e300 is infinite in FP32
        net = random_pair_network(14, 13, 6, 9)
        if bad is not None:
            net.tensors[1].reshape(-1)[5] = bad
        h = tnc.tnc_net_create(0, net.n_qubits, net.ranks(), net.flat_labels(), net.flat_data(), net.out_label)
        tnc.tnc_net_set_path(h, [(0, 1)])
        tnc.tnc_net_set_targets(h, list(range(net.n_qubits)), [0])
        p = tnc.tnc_plan_create(h, tnc.TNC_C64, 1)
        g = [tnc.tnc_plan_launch_info(p, i) for i in range(tnc.tnc_plan_n_launches(p))]
        assert [i.config for i in g if i.kind == 1] == [7 if bad is None else 0]
        tnc.tnc_plan_destroy(p)
        tnc.tnc_net_destroy(h)
