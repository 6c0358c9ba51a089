"""WA wirelength and gradient on degree sequences that reach every way a net
is taken: runs of whole small nets that end below, at and across 1024 pins,
nets of 64 and 65 pins side by side, large nets between small ones, alone in a
batch of 256 nets, and at the batch's edges."""
import numpy as np
import pytest

import test_gpu_wl as T

pytestmark = pytest.mark.gpu

SEQUENCES = {
    "one-net": [3],
    "empty-and-single": [0, 1, 0, 2, 1] * 60,
    "runs-end-at-edge": [64] * 40 + [1] * 216,
    "runs-end-short": [63] * 40 + [2] * 300,
    "small-beside-large": [64, 65] * 130,
    "all-large": [65 + (k % 7) for k in range(300)],
    "large-alone-in-a-batch": [9] * 100 + [900] + [8] * 155 + [0] * 255 + [1024] + [4] * 20,
    "large-passes": [5] * 10 + [256, 1023, 1025, 6000] + [5] * 242 + [2049],
}


@pytest.mark.parametrize("name", SEQUENCES)
@pytest.mark.parametrize("cols", [2, 4, 8])
def test_wa_of_degree_sequences(name, cols):
    deg = np.array(SEQUENCES[name])
    rng = np.random.default_rng(len(deg) + cols)
    n = 9000
    pins = np.concatenate([rng.choice(n, d, replace=False) for d in deg])
    nl = dict(n_inst=n, net_ptr=np.concatenate([[0], np.cumsum(deg)]).astype(np.int32), pin_node=pins.astype(np.int32),
              pin_off=rng.uniform(-3, 3, (pins.size, 2)).astype(np.float32), node_flags=np.zeros(n, np.uint8),
              node_size=np.ones((n, 2), np.float32), die=np.array([-50, -50, 50, 50], np.float32))
    # the bounds of test_gpu_wl
    T.check(nl, rng.uniform(-50, 50, (n, cols)).astype(np.float32), 2.0)
