"""Correlations and S^z_q transfers at the sizes where their kernels branch:
states of 32 bits and more, ring distances and general orbits in one call,
more pairs than a pass holds, rank, hash and no index, both widths of vectors.
Reference: the definitions on the device basis's states, in numpy."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def X():
    import paper_2505_02901_amd as X
    return X


def models():
    chain = lambda n, up, l=None: W.chain_model(n, n_up=up, l=l)
    mirror = W.chain_model(9, n_up=4)            # two elements: orbits of one and two pairs
    perm = np.array([np.arange(9), np.arange(9)[::-1]], np.int32)
    return {
        "ring31": chain(31, 3, 0), "ring32": chain(32, 3, 5), "ring33": chain(33, 3, 0),
        "ring40": chain(40, 2, 20), "u1_33": chain(33, 2), "u1_40": chain(40, 2), "u1_9": chain(9, 4),
        "torus16": W.torus_model((4, 0), (0, 4), 1.0, 0.5, "B1"),
        "torus36": W.torus_model((6, 0), (0, 6), 1.0, 0.0, "A1", n_up=4),
        "mirror9": mirror.with_sector(perm, np.array([1.0, -1.0]) + 0j),
    }


MODELS = models()


@pytest.mark.parametrize("single", [False, True])
@pytest.mark.parametrize("name", sorted(MODELS))
def test_correlations_by_definition(X, name, single):
    m = MODELS[name]
    b = X.Basis.from_model(m)
    s = b.states()
    psi = W.random_vector(3, b.dim, 1, kind="uniform", complex_=b.is_complex)
    if single:
        psi = psi.astype(np.complex64 if b.is_complex else np.float32)
    N = m.n_sites
    pairs = [(0, d % N) for d in range(20)] + [(N - 1, 0), (2, 2), (1, N // 2), (N - 1, 1)]
    got = X.xdg_expect_szsz(b.handle, torch.from_numpy(psi).cuda(), pairs)
    sz = np.array([((s >> np.uint64(i)) & np.uint64(1)).astype(float) - 0.5 for i in range(N)])
    p = np.abs(psi.astype(np.complex128)) ** 2
    G = m.perm if m.perm is not None else np.arange(N)[None]
    want = np.array([np.mean([(p * sz[g[a]] * sz[g[c]]).sum() for g in G]) for a, c in pairs])
    # sums of dim positive terms of total |psi|^2 / 4: 1e-13 of it covers every order
    assert np.max(np.abs(got - want)) <= 1e-13 * p.sum(), np.max(np.abs(got - want))


@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
@pytest.mark.parametrize("n,up,l,q", [(31, 3, 0, 4), (32, 3, 5, 16), (33, 3, 2, 32), (40, 2, 0, 7),
                                      (17, 4, 0, 1), (64, 2, 1, 33), (9, 9, 0, 3)])
@pytest.mark.parametrize("hash_index", [0, 4])
def test_transfer_by_definition(X, n, up, l, q, dtype, hash_index):
    mi, mo = W.chain_model(n, n_up=up, l=l), W.chain_model(n, n_up=up, l=(l + q) % n)
    bi = X.Basis.from_model(mi, flags=hash_index)
    bo = X.Basis.from_model(mo, flags=hash_index)
    x = W.random_vector(5, max(bi.dim, 1), 1, kind="uniform", complex_=True)[:bi.dim].astype(dtype)
    coef = np.exp(2j * np.pi * ((q * np.arange(n)) % n) / n)
    y = torch.full((bo.dim,), 7.0, dtype=getattr(torch, dtype), device="cuda")
    X.xdg_apply_sz_transfer(bi.handle, bo.handle, coef, torch.from_numpy(x).cuda(), y)
    so, si = bo.states(), list(bi.states())
    at = {int(s): i for i, s in enumerate(si)}
    want = np.zeros(bo.dim, complex)
    for r, s in enumerate(so):
        if int(s) in at:
            want[r] = sum(coef[j] * (0.5 if int(s) >> j & 1 else -0.5) for j in range(n)) * x[at[int(s)]]
    if bo.dim:
        # sums of n terms of modulus 1/2, then one product; one rounding to the stored type
        tol = 0.5 * n * (n * 2.3e-16 if dtype == "complex128" else 1.2e-7) * np.abs(x).max(initial=1.0)
        assert np.max(np.abs(y.cpu().numpy() - want)) <= tol


def test_transfer_without_group(X):
    m = W.chain_model(33, n_up=2)
    b = X.Basis.from_model(m)
    x = W.random_vector(6, b.dim, 1, kind="uniform")
    c = np.linspace(-1, 2, 33)
    y = torch.empty(b.dim, dtype=torch.float64, device="cuda")
    X.xdg_apply_sz_transfer(b.handle, b.handle, c, torch.from_numpy(x).cuda(), y)
    s = b.states()
    o = sum(c[j] * (((s >> np.uint64(j)) & np.uint64(1)).astype(float) - 0.5) for j in range(33))
    assert np.max(np.abs(y.cpu().numpy() - o * x)) <= 33 * 33 * 2.3e-16
