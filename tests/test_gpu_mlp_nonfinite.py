"""Non-finite and very large values in the network: a diverged parameter or
sample reaches the outputs, the loss and the gradient as in plain float32
arithmetic, and does not pass for a dead unit or spread where it is switched
off."""
import numpy as np
import pytest
import torch

import gpu_common as U
from oracle import ahr_oracle as O
from oracle import mlp_oracle as M
from synth import netlist as N

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2511_10073_amd")

INF = float("inf")


def setup(n, seed=5, scale=0.2):
    rng = np.random.default_rng(seed)
    p = rng.normal(0, scale, M.NPARAM).astype(np.float32)
    F = np.zeros((n, M.FEAT_PAD), np.float32)
    F[:, :M.NFEAT] = rng.normal(0, 1, (n, M.NFEAT))
    return p, F, rng.normal(0, 1, n).astype(np.float32)


def cuda(*a):
    return [torch.as_tensor(np.asarray(v)).cuda() for v in a]


@pytest.mark.parametrize("n", [1, 33])
@pytest.mark.parametrize("unit", [0, 21, 63])
def test_infinite_first_bias(n, unit):
    p, F, r = setup(n)
    at = M.OFFSETS["b1"][0] + unit
    p[at] = INF
    P, X, R = cuda(p, F, r)
    assert not torch.isfinite(A.mlp_forward(P, X)).any()
    g, loss = A.mlp_loss_grad(P, X, R)
    assert not torch.isfinite(loss).any() and not torch.isfinite(g).all()
    # a unit held below zero is dead, however far below
    p[at] = -INF
    q = p.copy()
    q[at] = -1e30
    P, Q = cuda(p, q)
    g, loss = A.mlp_loss_grad(P, X, R)
    gq, lq = A.mlp_loss_grad(Q, X, R)
    assert torch.isfinite(lq).all() and torch.equal(loss, lq) and torch.equal(g, gq)
    assert torch.equal(A.mlp_forward(P, X), A.mlp_forward(Q, X))


@pytest.mark.parametrize("n", [1, 17, 65])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_infinite_first_weight_of_a_dead_unit(n, sign):
    """W1 f is -inf in every sample: the unit is dead, the others are untouched."""
    p, F, r = setup(n)
    F[:, 2] = -sign * (np.abs(F[:, 2]) + 0.1)
    at = M.OFFSETS["W1"][0] + 11 * M.FEAT_PAD + 2
    p[at] = sign * INF
    q = p.copy()
    q[at] = sign * 1e30
    P, Q, X, R = cuda(p, q, F, r)
    o = A.mlp_forward(Q, X)
    assert torch.isfinite(o).all() and torch.equal(A.mlp_forward(P, X), o)
    (g, loss), (gq, lq) = A.mlp_loss_grad(P, X, R), A.mlp_loss_grad(Q, X, R)
    assert torch.equal(loss, lq) and torch.equal(g, gq)


@pytest.mark.parametrize("n", [1, 17, 65])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_infinite_first_weight_of_a_live_unit(n, sign):
    """W1 f is +inf in every sample: no output is finite."""
    p, F, r = setup(n)
    F[:, 2] = sign * (np.abs(F[:, 2]) + 0.1)
    p[M.OFFSETS["W1"][0] + 11 * M.FEAT_PAD + 2] = sign * INF
    P, X, R = cuda(p, F, r)
    assert not torch.isfinite(A.mlp_forward(P, X)).any()
    assert not torch.isfinite(A.mlp_loss_grad(P, X, R)[1]).any()


@pytest.mark.parametrize("cols", [2, 4])
def test_infinite_first_weight_in_the_learned_filter(cols):
    """The same where the samples' lanes own them (feature 4 is log1p of the degree, positive)."""
    nl = N.generate(N.small(1003, 5, ncols=4))
    x = torch.as_tensor(np.ascontiguousarray(nl["g0"][:, :cols])).cuda()
    gr = A.Graph(A.Netlist(nl), U.to_c_params(A, O.HintParams(nbx=8, nby=8)), x)
    spec = U.to_c_spec(A, O.FilterSpec(ks=(3,), alphas=(1.0,)))
    p, at, mov = setup(1)[0], M.OFFSETS["W1"][0] + 40 * M.FEAT_PAD + 4, U.movable_rows(nl)

    def learned(w):
        p[at] = w
        y, fallback = gr.filter_learned(spec, A.Mlp(cuda(p)[0], (-2.0, 4.5, -3.1, 1.6), True), x)
        assert not fallback
        return y.cpu().numpy()[mov]
    try:
        assert not np.isfinite(learned(INF)).any()
        dead = learned(-1e30)
        assert np.isfinite(dead).all() and np.array_equal(learned(-INF), dead)
    finally:
        gr.close()


def rows_of(p, F):
    """z2 and the rounded w3 of one sample, in float64 from the bfloat16 operands."""
    W1, b1, W2, b2, w3, _ = M.unpack(p)
    a1 = M.bf16(np.maximum(M.bf16(W1) @ M.bf16(F[0]) + b1, 0))
    return a1, M.bf16(W2) @ a1 + b2, M.bf16(w3)


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_infinite_output_gradient(sign):
    p, F, _ = setup(1)
    a1, z2, w3 = rows_of(p, F)
    assert np.abs(z2).min() > 1e-3 and (a1 > 0).any() and (z2 > 0).any() and (z2 < 0).any()
    P, X, R = cuda(p, F, np.float32([-sign * INF]))
    g, loss = A.mlp_loss_grad(P, X, R)
    g = g.cpu().numpy()
    part = lambda k: g[M.OFFSETS[k][0]:sum(M.OFFSETS[k])]
    assert float(loss.cpu()) == INF and part("b3")[0] == sign * INF
    want = np.where(z2 > 0, sign * np.sign(w3) * INF, 0.0)
    assert np.array_equal(part("b2"), want)
    assert np.array_equal(part("W2").reshape(64, 64)[:, a1 > 0], np.repeat(want[:, None], (a1 > 0).sum(), 1))
    assert not part("W2").reshape(64, 64)[z2 < 0].any()
    assert np.all(part("w3")[z2 > 0] == sign * INF)


def test_nan_target_leaves_dead_units():
    p, F, _ = setup(1)
    _, z2, _ = rows_of(p, F)
    P, X, R = cuda(p, F, np.float32([np.nan]))
    g, loss = A.mlp_loss_grad(P, X, R)
    g = g.cpu().numpy()
    assert not torch.isfinite(loss).any()
    o, k = M.OFFSETS["b2"]
    assert np.isnan(g[o:o + k][z2 > 0]).all() and not g[o:o + k][z2 < 0].any()


@pytest.mark.parametrize("grad", [3.0e38, 3.389e38, 3.3953e38, 3.4e38])
def test_largest_output_gradients(grad):
    """2 (o - t) up to the largest float32, past the largest bfloat16 (3.3895e38)."""
    p, F, _ = setup(1, scale=0.1)
    F *= 0.5
    t = np.float32([-grad / 2])
    P, X, R = cuda(p, F, t)
    g, loss = A.mlp_loss_grad(P, X, R)
    loss_ref, ref = M.loss_grad(p, F[:, :M.NFEAT].astype(np.float64), t.astype(np.float64))
    a1, _, _ = rows_of(p, F)
    assert a1.max() < 1 and np.isfinite(ref).all()
    assert abs(float(loss.cpu()) / loss_ref - 1) <= 1e-6
    g = g.cpu().numpy().astype(np.float64)
    for name, (o, k) in M.OFFSETS.items():
        e = np.linalg.norm((g[o:o + k] - ref[o:o + k]) / grad) / max(np.linalg.norm(ref[o:o + k] / grad), 1e-30)
        assert e <= 4e-5, (name, e)      # (as test_grad_at_tile_edges without its rounding term: one exact sample)
