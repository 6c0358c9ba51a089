"""The matrix-core training gradient at the edges of its tiles (16 and 32
samples), of a workgroup's share (128) and of the full grid (65,536 samples a
round), and on features at any 4-byte alignment."""
import numpy as np
import pytest
import torch

from oracle import mlp_oracle as M

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2511_10073_amd")


@pytest.mark.parametrize("n,shift", [(1, 0), (15, 1), (16, 0), (17, 0), (32, 2), (33, 0), (128, 0), (129, 3),
                                     (65536, 0), (65536 + 45, 1)])
def test_grad_at_tile_edges(n, shift):
    rng = np.random.default_rng(100 + n)
    p = M.init_params(n % 97).astype(np.float32)
    for name, sd in (("b1", 0.2), ("b2", 0.2), ("b3", 0.1)):
        o, k = M.OFFSETS[name]
        p[o:o + k] = rng.normal(0, sd, k)
    F = np.zeros((n, M.FEAT_PAD), np.float32)
    F[:, :M.NFEAT] = rng.normal(0, 1, (n, M.NFEAT))
    r = rng.normal(0, 1, n).astype(np.float32)
    buf = torch.zeros(8 * n + 4, dtype=torch.float32, device="cuda")
    feats = buf[shift:shift + 8 * n].view(n, 8)
    feats.copy_(torch.as_tensor(F))
    P, R = torch.as_tensor(p).cuda(), torch.as_tensor(r).cuda()
    g, loss = A.mlp_loss_grad(P, feats, R)
    g2, loss2 = A.mlp_loss_grad(P, feats, R)
    assert torch.equal(g, g2) and torch.equal(loss, loss2)
    loss_ref, ref = M.loss_grad(p, F[:, :M.NFEAT].astype(np.float64), r.astype(np.float64))
    # float32 sums are good to 1e-6; one hidden value crossing a bfloat16
    # rounding boundary moves by 2^-8 of itself in one of n samples
    tol = 1e-5 + 2.0 ** -7 / n
    assert abs(float(loss.cpu()) - loss_ref) <= tol * loss_ref
    g = g.cpu().numpy().astype(np.float64)
    for name, (o, k) in M.OFFSETS.items():
        e = np.linalg.norm(g[o:o + k] - ref[o:o + k]) / max(np.linalg.norm(ref[o:o + k]), 1e-30)
        assert e <= 4 * tol, (name, e, tol)


def test_grad_of_nothing_and_without_loss():
    p = torch.as_tensor(M.init_params(1).astype(np.float32)).cuda()
    g, loss = A.mlp_loss_grad(p, torch.zeros(0, 8, device="cuda"), torch.zeros(0, device="cuda"))
    assert float(loss.cpu()) == 0.0 and not g.any()
