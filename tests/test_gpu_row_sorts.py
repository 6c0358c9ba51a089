"""Netlist rows at the edges of the ways they are sorted and merged (8 to 64
lanes a row, workgroups of 256 and 1024 threads in LDS, the network in global
memory above 16384 raw entries), with few and with many repeated columns, and
the same rows in execution order: hubs of 2-pin nets, structure bit-exact
against the oracle's, the filter within its FP32 bound."""
import numpy as np
import pytest
import torch

import gpu_common as U
import netlists as H
from oracle import ahr_oracle as O

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2511_10073_amd")

SIZES = [1, 2, 7, 8, 9, 16, 17, 32, 33, 63, 64, 65, 127, 255, 256, 257, 511, 769, 1793, 2047, 2048, 2049, 3073, 5000,
         8192, 15360, 15361, 16384, 16385, 17000]


@pytest.mark.parametrize("pool", [5, 3000, 20000])
def test_rows_of_every_size(pool):
    rng = np.random.default_rng(pool)
    first = len(SIZES)
    nets = [[h, first + int(c)] for h, n in enumerate(SIZES) for c in rng.integers(0, pool, n)]
    rng.shuffle(nets)
    nl = H.make([list(e) for e in nets], first + pool)
    p = U.params32(O.HintParams(nbx=4, nby=4, detection_ratio=0.2))
    og = O.build_graph(nl, p, nl["g0"])
    x = torch.as_tensor(nl["g0"]).cuda()
    gr = A.Graph(A.Netlist(nl), U.to_c_params(A, p), x)
    try:
        ex = gr.export()
        assert np.array_equal(ex["net_row_ptr"], og.net_row_ptr.astype(np.int32))
        assert np.array_equal(ex["net_col"], og.net_col.astype(np.int32))
        assert np.array_equal(ex["net_q"], og.net_q)
        spec = U.spec32(O.FilterSpec(ks=(2, 4), alphas=(0.4, 0.6)))
        out = gr.filter(U.to_c_spec(A, spec), x).cpu().numpy()
        U.check_filter(out, O.apply_filter(nl, og, spec, nl["g0"]), U.movable_rows(nl))
    finally:
        gr.close()
