"""Graphs whose bucket sorts sit at the edges of the sort's forms: the largest
input of the one-workgroup form and one element more, key counts that leave
it 16, 8 and 2 waves, and the tiled form with 8 waves down to one wave and
with its longest tiles.  The sort is exact, so the hint structure equals the
oracle's and the filter stays within the float32 bound."""
import numpy as np
import pytest
import torch

import gpu_common as U
from oracle import ahr_oracle as O
from synth import netlist as N

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2511_10073_amd")


@pytest.mark.parametrize("n_inst,nbx,nby", [(16384, 9, 7), (16385, 9, 7), (8192, 64, 64), (8193, 64, 64),
                                            (2048, 128, 128), (2049, 128, 128), (70001, 128, 128), (70001, 31, 33)])
def test_graph_at_sort_edges(n_inst, nbx, nby):
    nl = N.generate(N.small(n_inst - 100, n_inst % 1000, n_macro=60, n_io=40))
    assert nl["n_inst"] == n_inst
    p = U.params32(O.HintParams(nbx=nbx, nby=nby, detection_ratio=3.5 / max(nbx, nby)))
    og = O.build_graph(nl, p, nl["g0"][:, :2])
    x = torch.as_tensor(nl["g0"]).cuda()
    gr = A.Graph(A.Netlist(nl), U.to_c_params(A, p), x)
    ex = gr.export()
    assert np.array_equal(ex["net_row_ptr"], og.net_row_ptr.astype(np.int32))
    assert np.array_equal(ex["net_col"], og.net_col.astype(np.int32))
    assert np.array_equal(ex["hint_row_ptr"], og.hint_row_ptr.astype(np.int32))
    r1, c1, _ = U.sorted_rows(ex["hint_row_ptr"], ex["hint_col"], ex["hint_val"])
    r0, c0, _ = U.sorted_rows(og.hint_row_ptr, og.hint_col, og.hint_val)
    assert np.array_equal(r1, r0) and np.array_equal(c1, c0)
    spec = U.spec32(O.FilterSpec(ks=(3,), alphas=(1.0,)))
    y = gr.filter(U.to_c_spec(A, spec), x).cpu().numpy()
    gr.close()
    U.check_filter(y, O.apply_filter(nl, og, spec, nl["g0"]), U.movable_rows(nl))
