"""Bases whose candidate lists are cut short: rings (lowest site up, top site
down) and sublattice blocks (minimal top contents), at every filling of small
lattices, bit-exact against the oracle's sweep over all states."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def X():
    import paper_2505_02901_amd as X
    return X


CASES = {f"ring{n}_k{l}": (n, lambda up, n=n, l=l: W.chain_model(n, n_up=up, l=l))
         for n in (2, 3, 4, 7, 12) for l in sorted({0, 1, n // 2})}
CASES.update({f"dihedral{n}": (n, lambda up, n=n: W.chain_model(n, n_up=up).with_sector(
    W.chain_dihedral(n), np.ones(2 * n, complex))) for n in (3, 8)})
CASES.update({
    "square16_A1": (16, lambda up: W.torus_model((4, 0), (0, 4), 1.0, 0.5, "A1", n_up=up)),
    "square16_B2": (16, lambda up: W.torus_model((4, 0), (0, 4), 1.0, 0.0, "B2", n_up=up)),
    "square10_2": (10, lambda up: W.sublattice_model("square2", (3, 1), (-1, 3), n_up=up)),
    "triangle9_3": (9, lambda up: W.sublattice_model("triangle3", (3, 0), (0, 3), n_up=up)),
})


@pytest.mark.parametrize("name", sorted(CASES))
def test_every_filling(X, name):
    n, make = CASES[name]
    for up in range(n + 1):
        m = make(up)
        b = X.Basis.from_model(m)
        want = oracle.basis(m)
        assert np.array_equal(b.states(), want), (name, up, b.dim, len(want))
        if b.dim:
            at = b.index(want)
            assert np.array_equal(at, np.arange(len(want))), (name, up)
            orbit = np.array([[sum(((int(s) >> int(g[i])) & 1) << i for i in range(n)) == int(s)
                               for g in m.perm] for s in want[:64]]).sum(axis=1)
            assert np.array_equal(b.stabilisers(0, min(64, b.dim)), orbit), (name, up)


# four blocks of 5 to 10 sites (both state widths) in the packed form, with
# characters 1, signs and complex ones; few and half-filled blocks
PACKED = {
    "20_A1": ((4, 2), (-2, 4), "A1", (0, 1, 2, 7, 10, 19, 20)), "20_B1": ((4, 2), (-2, 4), -1.0, (1, 2, 7, 10)),
    "20_E": ((4, 2), (-2, 4), 1j, (1, 2, 7, 10)),
    "24_A1": ((4, 0), (0, 6), "A1", (1, 4, 12)), "32_A1": ((4, 4), (-4, 4), "A1", (1, 4, 5, 28)),
    "36_A1": ((6, 0), (0, 6), "A1", (1, 2, 4, 32)), "36_B1": ((6, 0), (0, 6), "B1", (2, 4)),
    "40_A1": ((6, 2), (-2, 6), "A1", (1, 2, 3, 4)),
}


@pytest.mark.parametrize("name", sorted(PACKED))
def test_packed_blocks(X, name):
    l1, l2, gamma, ups = PACKED[name]
    for up in ups:
        refl = l1[1] == 0 or l1[0] == l1[1]
        turn = not isinstance(gamma, str)   # the character of a quarter turn
        m = W.torus_model(l1, l2, 1.0, 0.0, "A1" if turn else gamma, n_up=up, reflections=refl)
        if turn:
            perm, labels = W.Torus(l1, l2).symmetry_group(True, False)
            m = m.with_sector(perm, W.gamma_characters(labels, gamma, 1.0))
        b = X.Basis.from_model(m)
        want = oracle.basis(m)
        assert np.array_equal(b.states(), want), (name, up, b.dim, len(want))
        n = m.perm.shape[1]
        if len(want):
            count = np.zeros(len(want), int)
            for g in m.perm:
                im = np.zeros(len(want), np.uint64)
                for i in range(n):
                    im |= ((want.astype(np.uint64) >> np.uint64(int(g[i]))) & np.uint64(1)) << np.uint64(i)
                count += im == want.astype(np.uint64)
            assert np.array_equal(b.stabilisers(0, b.dim), count), (name, up)
