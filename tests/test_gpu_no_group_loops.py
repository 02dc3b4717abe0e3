"""Blocks without a group: the loop with all lanes on one bond (near exchanges by
Pascal steps, far ones through Lin's or the rank tables) and the loop over each
lane's own bonds give the same bits.  Which one runs follows from filling, type,
number of vectors and, in a batch, from its largest block."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def X():
    import paper_2505_02901_amd as X
    return X


def square(a, b, n_up, j2=0.0):
    t = W.Torus((a, 0), (0, b), blocked=False)
    sites, jz, jxy = t.j1j2_bonds(1.0, j2)
    return W.Model(f"{a}x{b}", t.n_sites, n_up, sites, 0.7 * jz, jxy)


BATCHES = {
    "thin beside half filled": [W.chain_model(16, n_up=8), W.chain_model(24, n_up=3), square(4, 5, 4),
                                W.chain_model(9, n_up=1)],
    "half filled beside thin": [W.chain_model(14, n_up=7), W.chain_model(30, n_up=4), square(4, 4, 8)],
    "wide": [W.chain_model(34, n_up=6), W.chain_model(34, n_up=4), square(6, 6, 3), W.chain_model(41, n_up=2)],
}


@pytest.mark.parametrize("dtype", ["float64", "float32", "complex64"])
@pytest.mark.parametrize("name", sorted(BATCHES))
def test_batches_take_one_loop(X, name, dtype):
    ms = BATCHES[name]
    bs = [X.Basis.from_model(m) for m in ms]
    hs = [X.Hamiltonian.from_model(b, m) for b, m in zip(bs, ms)]
    for nvec in (1, 3, 8):
        xs = [torch.randn(b.dim, nvec, dtype=getattr(torch, dtype), device="cuda") for b in bs]
        for f in (X.xdg_apply_batched, X.xdg_apply_batched_noalloc):
            ys = [torch.full_like(x, 3.0) for x in xs]
            f([h.handle for h in hs], xs, ys)
            for h, x, y in zip(hs, xs, ys):
                assert torch.equal(y, h.apply(x, torch.full_like(x, 4.0))), (name, nvec, f.__name__)


@pytest.mark.parametrize("m", [square(4, 6, 8, 0.5), W.chain_model(24, n_up=8), W.chain_model(36, n_up=6)],
                         ids=lambda m: m.name)
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_vectors_alone_and_together(X, m, dtype):
    """0.7 and 1.9 M rows: one vector and eight take different loops"""
    b = X.Basis.from_model(m)
    H = X.Hamiltonian.from_model(b, m)
    x = torch.randn(b.dim, 8, dtype=getattr(torch, dtype), device="cuda")
    for nvec in (2, 5, 8):
        xs = x[:, :nvec].contiguous()
        y = H.apply(xs, torch.full_like(xs, 3.0))
        for v in range(nvec):
            one = x[:, v].contiguous()
            assert torch.equal(y[:, v], H.apply(one, torch.full_like(one, 4.0))), (nvec, v)
