"""Small blocks, whose terms are shared out over the lanes of a wave: bitwise the
row loop's products for every search, width, precision and number of vectors,
alone and in batches (row counts below, at and above a wave's share)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def X():
    import paper_2505_02901_amd as X
    return X


def turned(n_up):
    t = W.Torus((4, 2), (-2, 4))
    m = W.torus_model((4, 2), (-2, 4), 1.0, 0.0, None, n_up=n_up)
    perm, labels = t.symmetry_group(True, False)
    return m.with_sector(perm, W.gamma_characters(labels, 1j, 1.0))


def long_range(n):
    """every pair of sites of a ring coupled: more bonds than a pass has pairs"""
    sites = np.array([(i, j) for i in range(n) for j in range(i)], np.int32)
    d = np.array([min(i - j, n - i + j) for i, j in sites], float)
    return W.Model("all_pairs", n, n // 2, sites, 1 / d, 0.5 / d, W.chain_translations(n),
                   W.momentum_characters(n, 0))


CASES = {
    "u1_6": (W.chain_model(6), {}), "u1_12": (W.chain_model(12, n_up=5), {}),
    "ring3": (W.chain_model(3, n_up=1, l=0), {}), "ring14": (W.chain_model(14, l=0), {}),
    "ring15_complex": (W.chain_model(15, n_up=7, l=4), {}), "ring40": (W.chain_model(40, n_up=3, l=1), {}),
    "ring14_hash": (W.chain_model(14, l=3), {"flags": 4}),
    "pairs15": (long_range(15), {}), "ring14_fp32": (W.chain_model(14, l=0), {"flags": 2}),
    "square16_table": (W.torus_model((4, 0), (0, 4), 1.0, 0.5, "B1"), {"search": 4}),
    "square20": (W.torus_model((4, 2), (-2, 4), 1.0, 0.0, "A1", n_up=7, reflections=False), {}),
    "square20_complex": (turned(7), {}), "square24_2": (W.torus_model((4, 0), (0, 6), 1.0, 0.5, "A1", n_up=6), {}),
    "square36": (W.torus_model((6, 0), (0, 6), 1.0, 0.5, "B1", n_up=5), {}),
    "triangle36": (W.sublattice_model("triangle3", (6, 0), (0, 6), n_up=4), {"search": 3, "n_sublattices": 3}),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_same_bits_as_the_row_loop(X, name):
    m, kw = CASES[name]
    b = X.Basis.from_model(m, **kw)
    H = X.Hamiltonian.from_model(b, m)
    basis = oracle.basis(m)
    for dt in (torch.float32, torch.float64, torch.complex64, torch.complex128):
        if b.is_complex and not dt.is_complex:
            continue
        for nvec in (1, 3, 8, 70):
            x = torch.randn(b.dim, nvec, dtype=dt, device="cuda")
            y, z = torch.full_like(x, 3.0), torch.full_like(x, 4.0)
            H.apply(x, y)
            X.xdg_apply_with_config(H.handle, x, z)
            assert torch.equal(y, z), (name, dt, nvec)
            if nvec == 3:
                want = oracle.apply(m, basis, x.cpu().numpy())
                tol = 1e-12 if dt in (torch.float64, torch.complex128) else 2e-6
                assert np.max(np.abs(y.cpu().numpy() - want)) < tol * np.max(np.abs(want)), (name, dt)


@pytest.mark.parametrize("nvec", [1, 5, 8])
def test_batches(X, nvec):
    ms = [W.chain_model(n, l=l) for n, l in ((14, 3), (20, 1), (14, 0), (9, 2), (16, 5), (4, 2))]
    bs = [X.Basis.from_model(m) for m in ms]
    hs = [X.Hamiltonian.from_model(b, m) for b, m in zip(bs, ms)]
    xs = [torch.randn(b.dim, nvec, dtype=torch.complex128, device="cuda") for b in bs]
    for f in (X.xdg_apply_batched, X.xdg_apply_batched_noalloc, X.xdg_apply_batched):
        ys = [torch.full_like(x, 3.0) for x in xs]
        f([h.handle for h in hs], xs, ys)
        for h, x, y in zip(hs, xs, ys):
            z = torch.empty_like(x)
            X.xdg_apply_with_config(h.handle, x, z)
            assert torch.equal(y, z)


@pytest.mark.parametrize("name", ["chain", "open", "square", "pairs", "wide", "wide_pairs", "one"])
def test_blocks_without_a_group(X, name):
    """neighbouring and far exchanges, one and several vectors, 32 bits and more"""
    def plain(m):
        return W.Model(m.name, m.n_sites, m.n_up, m.sites, m.jz, 0.3 + m.jxy)
    m = {"chain": lambda: plain(W.chain_model(13, n_up=5)),
         "open": lambda: W.Model("open", 11, 6, *W.chain_bonds(11, 1.0, 0.4, periodic=False)),
         "square": lambda: plain(W.torus_model((4, 0), (0, 4), 1.0, 0.5, "A1", n_up=7)),
         "pairs": lambda: plain(long_range(10)), "wide": lambda: plain(W.chain_model(33, n_up=3)),
         "wide_pairs": lambda: plain(W.torus_model((6, 0), (0, 6), 1.0, 0.5, "A1", n_up=3)),
         "one": lambda: plain(W.chain_model(5, n_up=5))}[name]()
    b = X.Basis.from_model(m)
    H = X.Hamiltonian.from_model(b, m)
    basis = oracle.basis(m)
    for dt in (torch.float32, torch.float64, torch.complex128):
        for nvec in (1, 2, 5):
            x = torch.randn(b.dim, nvec, dtype=dt, device="cuda")
            y, z = torch.full_like(x, 3.0), torch.full_like(x, 4.0)
            H.apply(x, y)
            X.xdg_apply_with_config(H.handle, x, z, nv=1, grid=2)
            assert torch.equal(y, z), (name, dt, nvec)
            want = oracle.apply(m, basis, x.cpu().numpy())
            tol = 2e-6 if dt == torch.float32 else 1e-12
            assert np.max(np.abs(y.cpu().numpy() - want)) <= tol * max(np.max(np.abs(want)), 1e-3)


@pytest.mark.parametrize("n,n_up,far", [(42, 40, False), (24, 3, True)])
def test_many_bonds_without_a_group(X, n, n_up, far):
    """6700 bonds, whose records take all but 3 KB of a compute unit's LDS:
    repeated pairs add their couplings"""
    rng = np.random.default_rng(3)
    i = rng.integers(0, n - 1, 6700)
    sites = np.stack([i, (i + (rng.integers(2, n - 1, 6700) if far else 1)) % n], 1).astype(np.int32)
    m = W.Model("many", n, n_up, sites, rng.uniform(-1, 1, 6700), rng.uniform(-1, 1, 6700))
    b = X.Basis.from_model(m)
    H = X.Hamiltonian.from_model(b, m)
    x = torch.randn(b.dim, dtype=torch.float64, device="cuda")
    want = oracle.apply(m, oracle.basis(m), x.cpu().numpy()).real
    s = b.states()
    assert H.nnz == b.dim + sum(int(np.sum((s >> np.uint64(p) ^ s >> np.uint64(q)) & np.uint64(1)))
                                for p, q in sites)
    for run in (lambda y: H.apply(x, y), lambda y: X.xdg_apply_with_config(H.handle, x, y),
                lambda y: X.xdg_apply_batched([H.handle], [x], [y]),
                lambda y: X.xdg_apply_batched_noalloc([H.handle], [x], [y])):
        y = torch.full_like(x, 3.0)
        run(y)
        # up to 6701 terms of size max |x|, each rounded once against a sum of that many
        assert np.max(np.abs(y.cpu().numpy() - want)) < 6701 * 6701 * 1.2e-16 * float(x.abs().max())


def shifts(n, step, up):
    i = np.arange(n)
    perm = (np.array([i, i[::-1]]) if step is None else
            np.array([(i + step * k) % n for k in range(n // step)])).astype(np.int32)
    return W.chain_model(n, n_up=up).with_sector(perm, np.ones(len(perm), complex))


THIN = {f"ring{n}_{up}": W.chain_model(n, n_up=up, l=0)
        for n, up in ((12, 0), (12, 1), (12, 3), (12, 4), (16, 4), (24, 4), (24, 5), (40, 3), (40, 4))}
THIN |= {f"ring{n}_{up}_k1": W.chain_model(n, n_up=up, l=1) for n, up in ((8, 2), (28, 4))}
THIN |= {f"dihedral{n}_{up}": W.chain_model(n, n_up=up).with_sector(
    W.chain_dihedral(n), np.ones(2 * n, complex)) for n, up in ((20, 3), (20, 17), (20, 4))}
THIN |= {f"mirror{n}_{up}": shifts(n, None, up) for n, up in ((8, 3), (16, 3), (16, 4), (40, 2), (40, 3))}
THIN |= {f"shifts{n}_{up}": shifts(n, s, up) for n, s, up in ((16, 2, 2), (16, 2, 3), (12, 4, 3))}
THIN |= {f"square{a[0]}x{b[1]}_{up}": W.torus_model(a, b, 1.0, 0.5, "A1", n_up=up, rotations=False,
                                                    reflections=False)
         for a, b in (((4, 0), (0, 4)), ((4, 0), (0, 6))) for up in (0, 1, 2)}


@pytest.mark.parametrize("name", sorted(THIN))
def test_thin_fillings(X, name):
    """rows of few terms, on both sides of the line between the loops, and blocks
    of a single wave"""
    m = THIN[name]
    b = X.Basis.from_model(m)
    H = X.Hamiltonian.from_model(b, m)
    basis = oracle.basis(m)
    for dt in (torch.float32, torch.float64, torch.complex128):
        if b.is_complex and not dt.is_complex:
            continue
        for nvec in (1, 2, 8):
            x = torch.randn(b.dim, nvec, dtype=dt, device="cuda")
            y, z = torch.full_like(x, 3.0), torch.full_like(x, 4.0)
            H.apply(x, y)
            X.xdg_apply_with_config(H.handle, x, z)
            assert torch.equal(y, z), (name, dt, nvec)
            want = oracle.apply(m, basis, x.cpu().numpy())
            tol = 2e-6 if dt == torch.float32 else 1e-12
            assert np.max(np.abs(y.cpu().numpy() - want)) <= tol * max(np.max(np.abs(want)), 1.0)
