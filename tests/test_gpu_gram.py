"""Densities and the two-electron operator on CI vectors where the gram kernels can go wrong: one
determinant, fewer determinants than a slice, slices that cross alpha strings, rows and factors
around the block sizes (one list of up to 17 blocks, several groups of B rows, more than 64
factors), bra equal to and different from ket, and repeated calls on one problem."""
import numpy as np
import pytest

import synth
from oracle import fci

pytestmark = pytest.mark.gpu


def _setup(n, na, nb, nq):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_09990_amd as pk
    h, B, e0 = synth.make_hamiltonian(n, nq, 2)
    space = fci.DetSpace(n, na, nb)
    rng = np.random.default_rng(n + 10 * na + nb)
    print(f"case n={n} ({na},{nb}) nq={nq}", flush=True)
    return torch, pk.Problem(h, B, na, nb, e0), B, space, rng


# sums of N_det products of unit-scale numbers in fp64: 1e-12 of the largest element, as for the
# other density tests
@pytest.mark.parametrize("n,na,nb", [(2, 1, 1), (3, 3, 0), (4, 1, 1), (8, 2, 1), (13, 1, 2), (16, 1, 1)])
def test_rdm12_edges(n, na, nb):
    torch, prob, B, space, rng = _setup(n, na, nb, 1)
    bra, ket = rng.normal(size=space.shape), rng.normal(size=space.shape)
    db, dk = torch.from_numpy(bra).cuda(), torch.from_numpy(ket).cuda()
    for x, y, dx, dy in ((bra, bra, db, db), (bra, ket, db, dk), (bra, bra, db, db)):
        g, G, ov = prob.ci_rdm12(dx, dy)
        rg, rG = fci.trdm12(space, x, y)
        scale = max(np.abs(rG).max(), 1.0)
        assert np.abs(g - rg).max() <= 1e-12 * scale
        assert np.abs(G - rG).max() <= 1e-12 * scale
        assert abs(ov - np.sum(x * y)) <= 1e-12 * scale


@pytest.mark.parametrize("n,na,nb,same", [(2, 1, 0, True), (2, 1, 1, False), (4, 2, 3, True), (6, 2, 2, False)])
def test_rdm3_edges(n, na, nb, same):
    torch, prob, B, space, rng = _setup(n, na, nb, 1)
    bra = rng.normal(size=space.shape)
    ket = bra if same else rng.normal(size=space.shape)
    db = torch.from_numpy(bra).cuda()
    G = prob.ci_rdm3(db, db if same else torch.from_numpy(ket).cuda())
    for _ in range(60):
        p, q, r, s, t, u = (int(x) for x in rng.integers(0, n, size=6))
        ref = np.sum(space.apply_E(q, p, bra) * space.apply_E(r, s, space.apply_E(t, u, ket)))
        assert abs(G[p, q, r, s, t, u] - ref) <= 1e-12 * max(np.abs(G).max(), 1.0)


@pytest.mark.parametrize("n,na,nb,nq", [(2, 1, 1, 1), (3, 1, 2, 65), (5, 2, 2, 64), (13, 1, 1, 130), (16, 1, 0, 3)])
def test_apply_v_edges(n, na, nb, nq):
    torch, prob, B, space, rng = _setup(n, na, nb, nq)
    c = rng.normal(size=space.shape)
    got = prob.ci_apply_v(torch.from_numpy(c).cuda()).cpu().numpy()
    T = np.stack([space.apply_E(r, s, c) for r in range(n) for s in range(n)])
    F = B.reshape(nq, n * n)
    U = np.tensordot(F.T @ F, T, axes=1)
    ref = 0.5 * sum(space.apply_E(x // n, x % n, U[x]) for x in range(n * n))
    assert np.abs(got - ref).max() <= 1e-12 * max(np.abs(ref).max(), 1.0)


# the largest call whose scratch is kept: a second one allocates nothing
def test_largest_rdm3_keeps_its_scratch():
    torch, prob, B, space, rng = _setup(12, 6, 6, 1)
    import paper_2609_09990_amd as pk
    h, B, e0 = synth.make_hamiltonian(4, 2, 2)
    count = pk.Solver(pk.Problem(h, B, 2, 2, e0), M=4, workspace=True)  # for the library's allocation count
    db, dk = (torch.from_numpy(rng.normal(size=space.shape)).cuda() for _ in range(2))
    first = prob.ci_rdm3(db, dk)
    n0 = count.stats()["device_allocs_since_attach"]
    assert n0 > 0
    second = prob.ci_rdm3(db, dk)
    assert count.stats()["device_allocs_since_attach"] == n0
    assert np.array_equal(first, second)


# the product instance of 11 and 12 orbitals (up to 272 rows): three-body densities sampled, and a
# transition 1-/2-RDM; tolerances as above
@pytest.mark.parametrize("n,na,nb,same", [(11, 2, 2, False), (11, 1, 2, True), (12, 2, 1, False)])
def test_rdm3_of_eleven_and_twelve_orbitals(n, na, nb, same):
    torch, prob, B, space, rng = _setup(n, na, nb, 1)
    bra = rng.normal(size=space.shape)
    ket = bra if same else rng.normal(size=space.shape)
    db = torch.from_numpy(bra).cuda()
    G = prob.ci_rdm3(db, db if same else torch.from_numpy(ket).cuda())
    for _ in range(60):
        p, q, r, s, t, u = (int(x) for x in rng.integers(0, n, size=6))
        ref = np.sum(space.apply_E(q, p, bra) * space.apply_E(r, s, space.apply_E(t, u, ket)))
        assert abs(G[p, q, r, s, t, u] - ref) <= 1e-12 * max(np.abs(G).max(), 1.0)


@pytest.mark.parametrize("n,na,nb", [(11, 3, 2), (12, 2, 3), (14, 2, 2)])
def test_transition_rdm12_of_many_orbitals(n, na, nb):
    torch, prob, B, space, rng = _setup(n, na, nb, 1)
    bra, ket = rng.normal(size=space.shape), rng.normal(size=space.shape)
    g, G, ov = prob.ci_rdm12(torch.from_numpy(bra).cuda(), torch.from_numpy(ket).cuda())
    rg, rG = fci.trdm12(space, bra, ket)
    scale = max(np.abs(rG).max(), 1.0)
    assert np.abs(g - rg).max() <= 1e-12 * scale
    assert np.abs(G - rG).max() <= 1e-12 * scale
    assert abs(ov - np.sum(bra * ket)) <= 1e-12 * scale


# more determinants than the grid's 512 workgroups of 32: the loop over slices and the gather of the
# next one, in both row-block instances, with one and with two passes of factors
@pytest.mark.parametrize("n,na,nb,nq", [(12, 3, 3, 40), (13, 3, 2, 70), (16, 2, 3, 5)])
def test_apply_v_many_slices(n, na, nb, nq):
    torch, prob, B, space, rng = _setup(n, na, nb, nq)
    assert space.size > 512 * 32
    c = rng.normal(size=space.shape)
    got = prob.ci_apply_v(torch.from_numpy(c).cuda()).cpu().numpy()
    T = np.stack([space.apply_E(r, s, c) for r in range(n) for s in range(n)])
    F = B.reshape(nq, n * n)
    U = np.tensordot(F.T @ F, T, axes=1)
    ref = 0.5 * sum(space.apply_E(x // n, x % n, U[x]) for x in range(n * n))
    assert np.abs(got - ref).max() <= 1e-12 * max(np.abs(ref).max(), 1.0)


# an infinite amplitude gives infinities where every term has one sign: the rows that fill a block of
# factors or determinants up bring no 0 x inf into it
@pytest.mark.parametrize("nq", [1, 3, 4, 66])
def test_apply_v_of_an_infinite_amplitude(nq):
    torch, prob, _, space, rng = _setup(3, 1, 0, nq)
    import paper_2609_09990_amd as pk
    B = rng.uniform(0.5, 1.0, (nq, 3, 3))
    prob = pk.Problem(np.eye(3), B + B.transpose(0, 2, 1), 1, 0, 0.0)
    c = torch.tensor([1.0, np.inf, 2.0], dtype=torch.float64, device="cuda")
    assert torch.isposinf(prob.ci_apply_v(c)).all()
