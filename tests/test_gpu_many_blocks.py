"""Recurrences on many blocks in one launch per operation: every block gets the
bits it gets alone, whatever blocks (one row, ragged, large) stand beside it."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def X():
    import paper_2505_02901_amd as X
    return X


SETS = {
    "real": [W.chain_model(n, n_up=u, l=0) for n, u in ((12, 6), (20, 10), (12, 1), (12, 5), (18, 7))],
    "complex": [W.chain_model(n, l=l) for n, l in ((14, 3), (20, 1), (14, 0), (9, 2), (16, 5))],
    "u1": [W.chain_model(n, n_up=u) for n, u in ((10, 5), (16, 8), (9, 4), (13, 1))],
}


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nvec", [1, 2, 4, 8])
@pytest.mark.parametrize("name", sorted(SETS))
def test_blocks_do_not_mix(X, name, nvec, prec):
    bs = [X.Basis.from_model(m) for m in SETS[name]]
    hs = [X.Hamiltonian.from_model(b, m) for b, m in zip(bs, SETS[name])]
    # complex vectors where any block is complex: the lone run of a real block is then real
    keep = [i for i, b in enumerate(bs) if b.is_complex or name != "complex"]
    n_iter = 4
    _, al, be = X.xdg_lanczos_eigval_batched([h.handle for h in hs], nvec, n_iter, seed=11, prec=prec)
    u, u2 = X.xdg_tpq_micro_batched([h.handle for h in hs], 0.5, n_iter, nvec, seed=11, prec=prec)
    for i in keep:
        _, a1, b1 = X.xdg_lanczos_eigval_batched([hs[i].handle], nvec, n_iter, seed=11 + i, prec=prec)
        live = n_iter if bs[i].dim > n_iter else 1
        assert np.array_equal(al[i][:, :live], a1[0][:, :live]), (name, nvec, i)
        assert np.array_equal(be[i][:, :live], b1[0][:, :live]), (name, nvec, i)
        v1, v2 = X.xdg_tpq_micro_batched([hs[i].handle], 0.5, n_iter, nvec, seed=11 + i, prec=prec)
        assert np.array_equal(u[i], v1[0], equal_nan=True), (name, nvec, i)
        assert np.array_equal(u2[i], v2[0], equal_nan=True), (name, nvec, i)


@pytest.mark.parametrize("nvec", [2, 8])
def test_blocks_of_many_sizes(X, nvec):
    """Small blocks that share an allocation, blocks that fill one together and a
    block larger than that (2.7 M rows), in every neighbourhood."""
    ups = (2, 9, 3, 12, 4, 9, 10, 5, 12, 12, 2, 11, 6)
    ms = {u: W.chain_model(24, n_up=u) for u in ups}
    bs = {u: X.Basis.from_model(m) for u, m in ms.items()}
    hs = {u: X.Hamiltonian.from_model(bs[u], m) for u, m in ms.items()}
    n_iter = 3
    H = [hs[u].handle for u in ups]
    _, al, be = X.xdg_lanczos_eigval_batched(H, nvec, n_iter, seed=11)
    u1, u2 = X.xdg_tpq_micro_batched(H, 0.5, n_iter, nvec, seed=11)
    for i, u in enumerate(ups):
        _, a, b = X.xdg_lanczos_eigval_batched([H[i]], nvec, n_iter, seed=11 + i)
        assert np.array_equal(al[i], a[0]) and np.array_equal(be[i], b[0]), (u, i)
        v1, v2 = X.xdg_tpq_micro_batched([H[i]], 0.5, n_iter, nvec, seed=11 + i)
        assert np.array_equal(u1[i], v1[0]) and np.array_equal(u2[i], v2[0]), (u, i)
