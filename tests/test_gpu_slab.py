"""GPU parity of the slab kernel (sigma phase A) where its units can go wrong: row ranges that
span factors, strips of one and of more than 64 columns, blocks deeper than the strip in LDS
(16), one-deep blocks, in every precision."""
import numpy as np
import pytest

import synth
from oracle import embed

pytestmark = pytest.mark.gpu


def _solver(n, na, nb, nq, M, k):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_09990_amd as pk
    h, B, e0 = synth.make_hamiltonian(n, nq, 3)
    mps = synth.random_mps(n, na, nb, M, seed=8)
    sol = pk.Solver(pk.Problem(h, B, na, nb, e0), M=M)
    sol.set_mps(mps["bonds"], mps["sites"])
    sol.prepare(k)
    return torch, sol, h, B, mps


# the tolerances of every sigma parity test: operands rounded once, fp32 accumulation
@pytest.mark.parametrize("n,na,nb,nq,M,k", [(2, 1, 1, 1, 1, 0), (6, 3, 3, 4, 40, 3), (7, 2, 4, 6, 17, 2), (8, 4, 4, 9, 200, 4)])
@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 2e-6), (2, 1e-2)])
def test_slab_sigma_matches_oracle(n, na, nb, nq, M, k, prec, tol):
    torch, sol, h, B, mps = _solver(n, na, nb, nq, M, k)
    psi = synth.random_twosite(mps["bonds"], k, seed=12)
    x = torch.from_numpy(psi).cuda()
    y = torch.zeros_like(x)
    print(f"case n={n} M={M} k={k} prec={prec}", flush=True)
    sol.sigma(k, x, y, prec)
    torch.cuda.synchronize()
    ref = embed.sigma_twosite(h, B, mps, k, psi, na, nb)
    err = np.linalg.norm(y.cpu().numpy() - ref) / np.linalg.norm(ref)
    assert err <= tol, err


# left sectors of up to 100 states (deeper than a strip): the operator's columns against its
# diagonal, which another kernel computes, and its symmetry; errors as above, relative to the
# norm of a product
@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 2e-6), (2, 1e-2)])
def test_slab_deep_blocks(prec, tol):
    n, k = 10, 5
    torch, sol, h, B, mps = _solver(n, 5, 5, 3, 1024, k)
    assert max(b[-1] for b in mps["bonds"][k]) > 64
    size = len(synth.random_twosite(mps["bonds"], k, seed=12))
    d = torch.zeros(size, dtype=torch.float64, device="cuda")
    sol.diag(k, d)
    y, z = torch.zeros_like(d), torch.zeros_like(d)
    rng = np.random.default_rng(5)
    for i in [0, size - 1] + [int(j) for j in rng.integers(0, size, 6)]:
        e = torch.zeros_like(d)
        e[i] = 1.0
        sol.sigma(k, e, y, prec)
        assert abs(float(y[i] - d[i])) <= tol * float(y.norm()), i
    u, v = (torch.from_numpy(rng.standard_normal(size)).cuda() for _ in range(2))
    sol.sigma(k, u, y, prec)
    sol.sigma(k, v, z, prec)
    scale = float(v.norm() * y.norm() + u.norm() * z.norm())
    assert abs(float(torch.dot(v, y) - torch.dot(u, z))) <= tol * scale
