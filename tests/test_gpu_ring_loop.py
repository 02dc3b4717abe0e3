"""Full rings with the rank index and equal neighbour bonds: bitwise the
products of the general loop, which a hash index or an unequal bond list
takes, for both state widths, all word-filling lengths, momenta, reflections,
precisions and numbers of vectors, alone and in batches."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

HASH, FP32 = 4, 2   # index by hashing; FP32 accumulation


@pytest.fixture(scope="module")
def X():
    import paper_2505_02901_amd as X
    return X


def dihedral(n, up):
    return W.chain_model(n, n_up=up).with_sector(W.chain_dihedral(n), np.ones(2 * n, complex))


# more rows than the few-rows loop takes
CASES = {"24_k0": lambda: W.chain_model(24, l=0), "24_k12": lambda: W.chain_model(24, l=12),
         "24_k5": lambda: W.chain_model(24, l=5), "25_k1": lambda: W.chain_model(25, n_up=11, l=1),
         "26_dihedral": lambda: dihedral(26, 13), "31_k0": lambda: W.chain_model(31, n_up=8, l=0),
         "32_k0": lambda: W.chain_model(32, n_up=8, l=0), "32_k3": lambda: W.chain_model(32, n_up=8, l=3),
         "32_dihedral": lambda: dihedral(32, 8), "33_k0": lambda: W.chain_model(33, n_up=7, l=0),
         "33_k2": lambda: W.chain_model(33, n_up=7, l=2), "40_dihedral": lambda: dihedral(40, 7),
         "63_k0": lambda: W.chain_model(63, n_up=5, l=0), "63_k1": lambda: W.chain_model(63, n_up=5, l=1),
         "64_k0": lambda: W.chain_model(64, n_up=5, l=0)}


@pytest.mark.parametrize("name", sorted(CASES))
def test_same_bits_as_the_general_loop(X, name):
    m = CASES[name]()
    for acc in (0, FP32):
        b, c = X.Basis.from_model(m, flags=acc), X.Basis.from_model(m, flags=HASH | acc)
        assert b.dim == c.dim and b.dim >= 1 << 16
        H, G = X.Hamiltonian.from_model(b, m), X.Hamiltonian.from_model(c, m)
        for dt in (torch.float32, torch.float64, torch.complex64, torch.complex128):
            if b.is_complex and not dt.is_complex:
                continue
            for nvec in (1, 3, 8, 9):
                x = torch.randn(b.dim, nvec, dtype=dt, device="cuda")
                y, z = torch.full_like(x, 3.0), torch.full_like(x, 4.0)
                H.apply(x, y)
                G.apply(x, z)
                assert torch.equal(y, z), (name, acc, dt, nvec)


def test_against_the_oracle(X):
    m = W.chain_model(24, l=5)
    b = X.Basis.from_model(m)
    H = X.Hamiltonian.from_model(b, m)
    basis = oracle.basis(m)
    x = torch.randn(b.dim, 1, dtype=torch.complex128, device="cuda")
    y = torch.empty_like(x)
    H.apply(x, y)
    want = oracle.apply(m, basis, x.cpu().numpy())
    # a row has at most 25 terms, each rounded a few times
    assert np.abs(y.cpu().numpy() - want).max() <= 200 * 2.0 ** -53 * np.abs(want).max()


@pytest.mark.parametrize("n", [25, 32, 33])
@pytest.mark.parametrize("one_general", [False, True])
def test_batches(X, n, one_general):
    """real and complex blocks together; one that takes the general loop takes
    the others with it"""
    up = {25: 11, 32: 8, 33: 7}[n]
    ms = [W.chain_model(n, n_up=up, l=l) for l in (0, 1, 2)]
    bs = [X.Basis.from_model(m, flags=HASH if one_general and i == 1 else 0)
          for i, m in enumerate(ms)]
    gs = [X.Basis.from_model(m, flags=HASH) for m in ms]
    Hs = [X.Hamiltonian.from_model(b, m) for b, m in zip(bs, ms)]
    Gs = [X.Hamiltonian.from_model(b, m) for b, m in zip(gs, ms)]
    for dt in (torch.complex64, torch.complex128):
        for nvec in (1, 3, 8):
            xs = [torch.randn(b.dim, nvec, dtype=dt, device="cuda") for b in bs]
            ys = [torch.full_like(x, 3.0) for x in xs]
            X.xdg_apply_batched([h.handle for h in Hs], xs, ys)
            for G, x, y in zip(Gs, xs, ys):
                z = torch.empty_like(x)
                G.apply(x, z)
                assert torch.equal(y, z), (n, one_general, dt, nvec)
