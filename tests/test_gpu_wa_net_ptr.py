"""WA wirelength where net_ptr decreases (no netlist, but not seen by the
host): the call ends, every net is read over its own pins alone, and a net
without pins counts for nothing, as in the netlist of the other nets."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2511_10073_amd")


def wa(ptr, pins, off, n, g):
    nl = dict(n_inst=n, net_ptr=np.asarray(ptr, np.int32), pin_node=pins, pin_off=off,
              node_flags=np.zeros(n, np.uint8), node_size=np.ones((n, 2), np.float32),
              die=np.array([-50, -50, 50, 50], np.float32))
    wl = A.Wirelength(A.Netlist(nl))
    try:
        tot, grad = wl.wa(torch.as_tensor(g).cuda(), 2.0)
        return tot.cpu().numpy(), grad.cpu().numpy()
    finally:
        wl.close()


@pytest.mark.parametrize("cols", [2, 4, 8])
@pytest.mark.parametrize("ptr", [[3, 2, 5], [3, 2, 5, 9, 9, 80, 82, 140],
                                 [6, 5, 5, 3, 3, 1, 7, 7] + list(range(9, 609, 2))])
def test_decreasing_net_ptr(ptr, cols):
    rng = np.random.default_rng(cols)
    n, m = 900, max(ptr)
    pins, off = rng.permutation(n)[:m].astype(np.int32), rng.uniform(-3, 3, (m, 2)).astype(np.float32)
    g = rng.uniform(-50, 50, (n, cols)).astype(np.float32)
    nets = [range(a, b) for a, b in zip(ptr[:-1], ptr[1:]) if b > a]
    flat = np.concatenate([np.array(e) for e in nets])
    assert len(set(flat.tolist())) == flat.size          # no pin in two nets
    tot, grad = wa(ptr, pins, off, n, g)
    want, wgrad = wa(np.concatenate([[0], np.cumsum([len(e) for e in nets])]), pins[flat], off[flat], n, g)
    # float32 weights taken two ways: twice the bounds of test_gpu_wl
    assert np.allclose(tot, want, rtol=8e-7, atol=0)
    assert np.allclose(grad[pins[flat]], wgrad[pins[flat]], rtol=4e-6, atol=4e-6)
