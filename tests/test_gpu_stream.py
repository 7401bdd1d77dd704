"""GPU parity of the stream kernel (sigma phase B) where its windows and tiles can go wrong:
odd and one-deep items, items longer than a window, blocks of one, of 63..65 and of more
than 64 rows or columns, output blocks without a product."""
import numpy as np
import pytest

import synth
from oracle import embed

pytestmark = pytest.mark.gpu


# fp64 sums of at most a few thousand terms of unit scale: 1e-12 as for every sigma parity test;
# fp32 operands rounded once, fp32 accumulation: 2e-6 as there
@pytest.mark.parametrize("n,na,nb,nq,M,k", [
    (2, 1, 1, 1, 1, 0),
    (5, 3, 2, 4, 3, 1),
    (7, 2, 4, 6, 17, 2),
    (8, 4, 4, 9, 200, 3),
    (9, 5, 4, 5, 430, 4),
])
@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 2e-6)])
def test_stream_sigma_matches_oracle(n, na, nb, nq, M, k, prec, tol):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_09990_amd as pk
    h, B, e0 = synth.make_hamiltonian(n, nq, 3)
    mps = synth.random_mps(n, na, nb, M, seed=8)
    sol = pk.Solver(pk.Problem(h, B, na, nb, e0), M=M)
    sol.set_mps(mps["bonds"], mps["sites"])
    sol.prepare(k)
    psi = synth.random_twosite(mps["bonds"], k, seed=12)
    x = torch.from_numpy(psi).cuda()
    y = torch.zeros_like(x)
    print(f"case n={n} M={M} k={k} prec={prec}", flush=True)
    sol.sigma(k, x, y, prec)
    torch.cuda.synchronize()
    ref = embed.sigma_twosite(h, B, mps, k, psi, na, nb)
    err = np.linalg.norm(y.cpu().numpy() - ref) / np.linalg.norm(ref)
    assert err <= tol, err


# output blocks without a product: with one left factor per chunk, the first chunk writes zeros to
# every block that its factor does not reach; without integrals no block has a product
@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 2e-6), (2, 1e-2)])
@pytest.mark.parametrize("zero", [False, True])
def test_blocks_without_a_product(zero, prec, tol):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_09990_amd as pk
    n, na, nb, M, k = 6, 3, 3, 30, 2
    h, B, e0 = synth.make_hamiltonian(n, 4, 3)
    if zero:
        h, B = np.zeros_like(h), np.zeros_like(B)
    mps = synth.random_mps(n, na, nb, M, seed=8)
    sol = pk.Solver(pk.Problem(h, B, na, nb, e0), M=M, sigma_chunk_bytes=0 if zero else 1)
    sol.set_mps(mps["bonds"], mps["sites"])
    sol.prepare(k)
    psi = synth.random_twosite(mps["bonds"], k, seed=12)
    x = torch.from_numpy(psi).cuda()
    y = torch.full_like(x, 7.0)
    print(f"case zero={zero} prec={prec}", flush=True)
    sol.sigma(k, x, y, prec)
    torch.cuda.synchronize()
    if zero:
        assert torch.count_nonzero(y) == 0
        return
    ref = embed.sigma_twosite(h, B, mps, k, psi, na, nb)
    err = np.linalg.norm(y.cpu().numpy() - ref) / np.linalg.norm(ref)
    assert err <= tol, err
