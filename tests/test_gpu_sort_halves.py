"""Bucket sorts on both sides of the table size from which the keys are sorted
in two passes by halves of their bits (2^21 counters of a key in a tile), for
key counts that are a power of two and that are not, and with cells bunched in
the first bins (long stretches of empty keys): hint structure exact against the
oracle's."""
import numpy as np
import pytest
import torch

import gpu_common as U
from oracle import ahr_oracle as O
from synth import netlist as N

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2511_10073_amd")


@pytest.mark.parametrize("n_inst,nbx,nby,bunched", [(262144, 128, 128, False), (262145, 128, 128, False),
                                                    (300000, 113, 127, False), (270000, 128, 128, True)])
def test_hints_of_large_tables(n_inst, nbx, nby, bunched):
    nl = N.generate(N.small(n_inst - 100, n_inst % 1000, n_macro=60, n_io=40))
    assert nl["n_inst"] == n_inst
    if bunched:
        lo, hi = nl["die"][:2], nl["die"][2:]
        nl["g0"] = (lo + (nl["g0"] - lo) * 0.4).astype(np.float32)
        assert np.all(nl["g0"] < (lo + hi) / 2 + 1)
    p = U.params32(O.HintParams(nbx=nbx, nby=nby, detection_ratio=1.5 / max(nbx, nby), macro_hints=False))
    og = O.build_graph(nl, p, nl["g0"][:, :2])
    gr = A.Graph(A.Netlist(nl), U.to_c_params(A, p), torch.as_tensor(nl["g0"]).cuda())
    try:
        ex = gr.export()
    finally:
        gr.close()
    assert np.array_equal(ex["hint_row_ptr"], og.hint_row_ptr.astype(np.int32))
    r1, c1, _ = U.sorted_rows(ex["hint_row_ptr"], ex["hint_col"], ex["hint_val"])
    r0, c0, _ = U.sorted_rows(og.hint_row_ptr, og.hint_col, og.hint_val)
    assert np.array_equal(r1, r0) and np.array_equal(c1, c0)
