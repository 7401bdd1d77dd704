"""Training step of the preconditioner network at the edges of its tiles: widths around 64 and
128 that are no multiple of 4 or 16, one row, rows around the 128- and 512-row tiles, one and
more than 16 inputs, against the fp64 oracle."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,W,nseg,L", [
    (1, 1, 1, 1),
    (16, 65, 2, 64),
    (17, 130, 1, 513),
    (8, 64, 3, 171),
    (5, 127, 4, 128),
])
def test_training_step_edges(F, W, nseg, L):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_09990_amd as pk
    print(f"case F={F} W={W} nseg={nseg} L={L}", flush=True)
    P = omlp.init(F, W, seed=5)
    rng = np.random.default_rng(6)
    P = {k: (v + rng.normal(0, 0.1, v.shape)).astype(np.float32) for k, v in P.items()}
    X = rng.normal(size=(nseg * L, F)).astype(np.float32)
    T = rng.normal(size=nseg * L).astype(np.float32)
    net = pk.MLP(F, W)
    net.set_params(pk.MLP.pack(P))
    loss, g = net.loss_grad(torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda(), nseg, L, want_grad=True)
    Pd = {k: v.astype(np.float64) for k, v in P.items()}
    ref, rl = None, 0.0
    for s in range(nseg):
        sl = slice(s * L, (s + 1) * L)
        y, cache = omlp.forward(Pd, X[sl].astype(np.float64))
        ls, dy = omlp.cosine_loss(y, T[sl].astype(np.float64))
        rl += ls / nseg
        gs = omlp.backward(Pd, cache, dy / nseg)
        ref = gs if ref is None else {k: ref[k] + gs[k] for k in gs}
    got = net.unpack(g)
    # fp32 operands and sums of at most a few hundred terms: 2^-24 sqrt(513) ~ 1.4e-6 of the
    # largest term, a few of them per entry; scaled by the whole gradient
    scale = np.sqrt(sum(float((ref[k] ** 2).sum()) for k in ref))
    assert abs(loss - rl) <= 1e-5
    for k in ref:
        assert np.linalg.norm(got[k].astype(np.float64) - ref[k].reshape(got[k].shape)) <= 2e-5 * scale + 1e-7, k
