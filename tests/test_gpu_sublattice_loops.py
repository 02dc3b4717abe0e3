"""The row loops of the two sublattice searches, of single blocks (workgroups of
256 to 1024 lanes) and of batches beyond the few-rows line: the same bits from the
single loop, the compacted loop and batches that mix both searches."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def X():
    import paper_2505_02901_amd as X
    return X


def lattice(a1, a2, n_up, blocked, reflections=False, chi=None):
    t = W.Torus(a1, a2, blocked=blocked)
    sites, jz, jxy = t.j1j2_bonds(1.0, 0.0)
    perm, labels = t.symmetry_group(chi is not None, reflections)
    chi = W.gamma_characters(labels, *(chi or (1.0, 1.0)))
    return W.Model(f"{a1}{a2}{n_up}", t.n_sites, n_up, sites, 0.7 * jz, jxy, perm, chi)


PACKED = [lattice((4, 0), (0, 6), 9, True), lattice((4, 0), (0, 6), 11, True, True),
          lattice((4, 4), (-4, 4), 8, True, chi=(1j, 1.0))]
BLOCKS = [lattice((5, 0), (0, 5), 8, False), lattice((5, 0), (0, 5), 11, False), lattice((3, 0), (0, 6), 9, False)]


@pytest.mark.parametrize("dtype", ["float64", "complex64"])
@pytest.mark.parametrize("m", PACKED[:2] + BLOCKS[:2], ids=lambda m: m.name)
def test_one_block(X, m, dtype):
    b = X.Basis.from_model(m)
    assert b.search_kind[0] == X.XDG_SEARCH_SUBLATTICE
    H = X.Hamiltonian.from_model(b, m)
    for nvec in (1, 3, 8):
        x = torch.randn(b.dim, nvec, dtype=getattr(torch, dtype), device="cuda")
        y = H.apply(x, torch.full_like(x, 3.0))
        for shape in ({}, {"grid": 5}, {"occ": 0}, {"compact": 1}, {"compact": 1, "nv": 4}, {"sub_form": 2},
                      {"xr": 1}, {"xr": 1, "sub_form": 2}):
            z = torch.full_like(x, 4.0)
            X.xdg_apply_with_config(H.handle, x, z, **shape)
            assert torch.equal(y, z), (nvec, shape)


@pytest.mark.parametrize("ms", [PACKED[:2] * 2, BLOCKS[:2] * 2, BLOCKS + PACKED, PACKED[2:] + BLOCKS[2:]],
                         ids=["packed", "blocks", "mixed", "mixed few"])
def test_batches(X, ms):
    ms = [m for m in ms if (m.n_sites > 32) == (ms[0].n_sites > 32)]
    bs = [X.Basis.from_model(m) for m in ms]
    hs = [X.Hamiltonian.from_model(b, m) for b, m in zip(bs, ms)]
    for dtype, nvec in ((torch.complex128, 1), (torch.complex64, 3), (torch.complex128, 8)):
        xs = [torch.randn(b.dim, nvec, dtype=dtype, device="cuda") for b in bs]
        for f in (X.xdg_apply_batched, X.xdg_apply_batched_noalloc):
            ys = [torch.full_like(x, 3.0) for x in xs]
            f([h.handle for h in hs], xs, ys)
            for i, (h, x, y) in enumerate(zip(hs, xs, ys)):
                assert torch.equal(y, h.apply(x, torch.full_like(x, 4.0))), (i, nvec, f.__name__)
