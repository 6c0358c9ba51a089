"""The network's 16-sample tiles: a sample's output does not depend on the
other samples of its tile or on where in it the sample lies, in the forward
pass and in the learned filter (which takes its samples from the lanes that
loaded them)."""
import numpy as np
import pytest
import torch

import gpu_common as U
from oracle import ahr_oracle as O
from synth import netlist as N

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2511_10073_amd")


def params(seed):
    p = np.random.default_rng(seed).normal(0, 0.2, A.MLP_NPARAM).astype(np.float32)
    return torch.as_tensor(p).cuda()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 65])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_forward_ignores_the_other_samples(n, bad):
    F = torch.as_tensor(np.random.default_rng(n).normal(0, 1, (n, 8)).astype(np.float32)).cuda()
    p = params(3)
    want = A.mlp_forward(p, F)
    for k in range(min(n, 16)):
        G = F.clone()
        G[k] = bad
        got = A.mlp_forward(p, G)
        keep = torch.arange(n, device="cuda") != k
        assert torch.equal(got[keep], want[keep])


@pytest.mark.parametrize("cols", [2, 4, 8])
def test_learned_filter_is_the_forward_pass_of_its_features(cols):
    nl = N.generate(N.small(1003, 5, ncols=2))
    g0 = np.repeat(nl["g0"], 4, axis=1)[:, :cols]
    g0 = (g0 + np.random.default_rng(cols).normal(0, 2, g0.shape)).astype(np.float32)
    x = torch.as_tensor(g0).cuda()
    gr = A.Graph(A.Netlist(nl), U.to_c_params(A, O.HintParams(nbx=8, nby=8)), x)
    spec = U.to_c_spec(A, O.FilterSpec(ks=(3,), alphas=(1.0,)))
    p, beta = params(7), (-2.0, 4.5, -3.1, 1.6)
    try:
        out, fallback = gr.filter_learned(spec, A.Mlp(p, beta, True), x)
        feats, hops, stats = gr.features(spec, x)
    finally:
        gr.close()
    assert not fallback
    o = A.mlp_forward(p, feats.reshape(-1, 8)).reshape(x.shape).double().cpu().numpy()
    h = hops.double().cpu().numpy()
    terms = np.stack([b * hj for b, hj in zip(np.float32(beta).astype(np.float64), h)] + [stats[2].cpu().numpy() * o])
    mov = U.movable_rows(nl)
    # five float32 products and four additions
    err = np.abs(out.double().cpu().numpy() - terms.sum(0))[mov]
    assert np.all(err <= 9 * 2.0 ** -24 * np.abs(terms).sum(0)[mov])
