"""The integral gradient where the device-made row products can go wrong: one-state bonds, edge
sites whose classes have no source block, odd electron counts, and blocks of more than 64 rows
and 32 columns; against the densities of the same MPS through its CI vector."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,na,nb,nq,M", [(2, 1, 1, 2, 1), (3, 2, 0, 4, 2), (6, 2, 3, 5, 11), (9, 5, 4, 6, 512)])
def test_gradient_equals_densities(n, na, nb, nq, M):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_09990_amd as pk
    print(f"case n={n} ({na},{nb}) M={M}", flush=True)
    h, B, e0 = synth.make_hamiltonian(n, nq, 4)
    sol = pk.Solver(pk.Problem(h, B, na, nb, e0), M=M)
    mps = synth.random_mps(n, na, nb, M, seed=3)
    sol.set_mps(mps["bonds"], mps["sites"])
    g, G, _ = sol.rdm12()
    for _ in range(2):  # fresh and kept buffers
        dh, dB, e = sol.grad()
        # two fp64 routes of a few thousand unit-scale terms each
        assert np.abs(dh - g).max() <= 1e-11 * np.abs(g).max()
        ref = np.einsum("pqrs,Qrs->Qpq", G, B)
        assert np.abs(dB - ref).max() <= 1e-11 * max(np.abs(ref).max(), 1.0)
        assert abs(e[0] - (np.sum(h * g) + 0.5 * np.sum(B * ref) + e0)) <= 1e-11 * max(1.0, abs(e[0]))


def test_gradient_in_small_workspaces():
    """In every workspace the gradient gives the same numbers, whether its classes run together, one by
    one or in chunks of their rows, or it reports DMRG_ENOMEM."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_09990_amd as pk
    n, na, nb, nq, M = 8, 4, 4, 12, 120
    h, B, e0 = synth.make_hamiltonian(n, nq, 4)
    prob = pk.Problem(h, B, na, nb, e0)
    mps = synth.random_mps(n, na, nb, M, seed=3)

    def solver(size):
        s = pk.Solver(prob, M=M)
        s.set_mps(mps["bonds"], mps["sites"])
        s.attach_workspace(size)
        return s

    ref = solver(1 << 31)
    want = ref.grad()
    full = ref.stats()["workspace_peak_bytes"]
    ran = 0
    for pct in (105, 100, 90, 80, 75, 70, 60, 50, 40, 30, 20):
        sol = solver(int(full * pct / 100) + 4096)
        try:
            got = sol.grad()
        except pk.DMRGError as e:
            assert e.code == -2
            print(f"{pct}% of {full / 2**20:.0f} MiB: DMRG_ENOMEM", flush=True)
            continue
        ran += 1
        diff = [float(np.abs(a - b).max() / max(np.abs(b).max(), 1.0)) for a, b in zip(got, want)]
        print(f"{pct}% of {full / 2**20:.0f} MiB: {diff}", flush=True)
        assert max(diff) <= 1e-11  # two fp64 orders of a few thousand unit-scale terms each
    assert ran > 0
