"""Graphs whose row, net and pin counts lie at the edges of the scans' forms
(4 items a thread of 1024 in the one-launch form, 16384 items and the tiled
form above): structure bit-exact against the oracle's, with and without
hints."""
import numpy as np
import pytest
import torch

import gpu_common as U
import netlists as H
from oracle import ahr_oracle as O

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2511_10073_amd")


@pytest.mark.parametrize("hints", [False, True])
@pytest.mark.parametrize("n", [3, 1023, 1025, 4095, 4096, 4097, 16383, 16384, 16385, 20481])
def test_rings_at_scan_edges(n, hints):
    nl = H.ring(n)
    p = U.params32(O.HintParams(nbx=4, nby=4, detection_ratio=0.3, macro_hints=hints, bin_hints=hints))
    og = O.build_graph(nl, p, nl["g0"])
    gr = A.Graph(A.Netlist(nl), U.to_c_params(A, p), torch.as_tensor(nl["g0"]).cuda())
    try:
        ex = gr.export()
    finally:
        gr.close()
    assert np.array_equal(ex["net_row_ptr"], og.net_row_ptr.astype(np.int32))
    assert np.array_equal(ex["net_col"], og.net_col.astype(np.int32))
    assert np.array_equal(ex["net_q"], og.net_q)
    assert np.array_equal(ex["hint_row_ptr"], og.hint_row_ptr.astype(np.int32))
    r1, c1, _ = U.sorted_rows(ex["hint_row_ptr"], ex["hint_col"], ex["hint_val"])
    r0, c0, _ = U.sorted_rows(og.hint_row_ptr, og.hint_col, og.hint_val)
    assert np.array_equal(r1, r0) and np.array_equal(c1, c0)
