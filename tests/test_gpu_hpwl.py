"""HPWL on degree sequences that reach every way a net is summed: inside one
window of pins, across windows, big nets by a wave and by the workgroup, next
to one another, alone in a batch of 256 nets, and at the batch's edges."""
import numpy as np
import pytest
import torch

from oracle import ahr_oracle as O

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2511_10073_amd")

SEQUENCES = {
    "one-net": [3],
    "empty-and-single": [0, 1, 0, 2, 1] * 60,
    "window-edges": [64] * 40 + [2] * 300,
    "last-small-first-big": [64, 65] * 130,
    "all-big": [65 + (k % 7) for k in range(300)],
    "one-big-in-a-batch": [2] * 100 + [900] + [3] * 154 + [1] * 256 + [2048] + [4] * 20,
    "wave-and-workgroup": [5] * 10 + [2048, 2049, 70, 6000] + [5] * 250 + [8000],
    "batch-edges": [5000] + [2] * 254 + [300] + [66] + [2] * 255,
}


@pytest.mark.parametrize("name", SEQUENCES)
@pytest.mark.parametrize("cols", [2, 4, 8])
def test_hpwl_of_degree_sequences(name, cols):
    deg = np.array(SEQUENCES[name])
    rng = np.random.default_rng(len(deg) + cols)
    n = 9000
    pins = np.concatenate([rng.choice(n, d, replace=False) for d in deg] or [np.zeros(0, int)])
    nl = dict(n_inst=n, net_ptr=np.concatenate([[0], np.cumsum(deg)]).astype(np.int32), pin_node=pins.astype(np.int32),
              pin_off=rng.uniform(-3, 3, (pins.size, 2)).astype(np.float32), node_flags=np.zeros(n, np.uint8),
              node_size=np.ones((n, 2), np.float32), die=np.array([-50, -50, 50, 50], np.float32))
    g = rng.uniform(-50, 50, (n, cols)).astype(np.float32)
    want, _ = O.hpwl(nl, g)
    got = A.hpwl(A.Netlist(nl), torch.as_tensor(g).cuda()).cpu().numpy()
    # float64 sums of at most 600 nets on both sides
    assert np.all(np.abs(got - want) <= 1e-12 * want)
