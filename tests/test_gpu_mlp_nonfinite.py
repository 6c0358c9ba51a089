"""Non-finite values in the network: a diverged parameter reaches the outputs
and the loss as in plain float32 arithmetic, and does not pass for a dead unit
or spread where it is switched off."""
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
