"""Detection windows on both sides of the size from which the bin rows' windows
are walked in a launch of their own (9 slots), below and above the row count of
the one-launch scan, with and without pruning (decided in the count pass up to
64 slots, by holes above): hint structure exact against the oracle's, and the
filter within its FP32 bound."""
import numpy as np
import pytest
import torch

import gpu_common as U
from oracle import ahr_oracle as O
from synth import netlist as N

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2511_10073_amd")


def slots(nbx, nby, ratio):
    half = lambda nb: max(1, int(np.floor(np.float32(ratio) * np.float32(nb)))) // 2
    return (2 * half(nbx) + 1) * (2 * half(nby) + 1)


@pytest.mark.parametrize("tau", [0.0, 0.2])
@pytest.mark.parametrize("cells", [900, 18000])
@pytest.mark.parametrize("nbx,nby,ratio,want", [(7, 9, 0.3, 9), (10, 5, 0.5, 15), (1, 40, 0.5, 21), (8, 9, 0.5, 25),
                                                (9, 12, 0.8, 63), (30, 24, 0.3, 63), (24, 30, 0.4, 117)])
def test_windows(nbx, nby, ratio, want, cells, tau):
    assert slots(nbx, nby, ratio) == want
    nl = N.generate(N.small(cells, 5, ncols=2))
    p = U.params32(O.HintParams(nbx=nbx, nby=nby, detection_ratio=ratio, prune_tau=tau))
    og = O.build_graph(nl, p, nl["g0"])
    x = torch.as_tensor(nl["g0"]).cuda()
    gr = A.Graph(A.Netlist(nl), U.to_c_params(A, p), x)
    spec = U.spec32(O.FilterSpec(ks=(2, 4), alphas=(0.4, 0.6)))
    try:
        ex = gr.export()
        out = gr.filter(U.to_c_spec(A, spec), x).cpu().numpy()
    finally:
        gr.close()
    assert np.array_equal(ex["hint_row_ptr"], og.hint_row_ptr.astype(np.int32))
    r1, c1, _ = U.sorted_rows(ex["hint_row_ptr"], ex["hint_col"], ex["hint_val"])
    r0, c0, _ = U.sorted_rows(og.hint_row_ptr, og.hint_col, og.hint_val)
    assert np.array_equal(r1, r0) and np.array_equal(c1, c0)
    U.check_filter(out, O.apply_filter(nl, og, spec, nl["g0"]), U.movable_rows(nl))
