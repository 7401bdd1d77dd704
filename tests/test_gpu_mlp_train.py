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


# around the rules of the forward: 64 tiles of 128 rows (fewer take 64 x 64 tiles and a wave per row),
# and 2^18 activations (fewer take a thread per activation in layer 1); forward and gradient
@pytest.mark.parametrize("F,W,nseg,L", [
    (8, 1, 5, 1613),    # 64 tiles
    (16, 65, 63, 128),  # 63 tiles
    (16, 65, 5, 1613),  # 64
    (5, 130, 31, 128),  # 62
    (5, 130, 63, 63),   # 64
    (8, 64, 9, 455),    # 2^18 - 64 activations
    (8, 64, 8, 512),    # 2^18
    (17, 64, 5, 1613),  # 64 tiles, more inputs than layer 1 keeps in registers
])
def test_forward_rules(F, W, nseg, L):
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
    dx = torch.from_numpy(X).cuda()
    y = torch.zeros(nseg * L, device="cuda")
    Pd = {k: v.astype(np.float64) for k, v in P.items()}
    ry, cache = omlp.forward(Pd, X.astype(np.float64))
    loss, g = net.loss_grad(dx, torch.from_numpy(T).cuda(), nseg, L, want_grad=True)
    rl, dy = 0.0, np.zeros(nseg * L)
    for s in range(nseg):
        sl = slice(s * L, (s + 1) * L)
        ls, d = omlp.cosine_loss(ry.reshape(-1)[sl], T[sl].astype(np.float64))
        rl += ls / nseg
        dy[sl] = d.reshape(-1) / nseg
    ref = omlp.backward(Pd, cache, dy.reshape(ry.shape))
    got = net.unpack(g)
    net.forward(dx, y, 1)
    # as above: fp32 products over at most 130 terms, and row sums in chunks of 512 added in fp64
    assert np.linalg.norm(y.cpu().numpy() - ry.reshape(-1)) <= 2e-5 * np.linalg.norm(ry)
    assert abs(loss - rl) <= 1e-5
    scale = np.sqrt(sum(float((ref[k] ** 2).sum()) for k in ref))
    for k in ref:
        assert np.linalg.norm(got[k].astype(np.float64) - ref[k].reshape(got[k].shape)) <= 2e-5 * scale + 1e-7, k
