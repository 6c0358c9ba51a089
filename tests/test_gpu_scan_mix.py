"""Rows of every sorted length, star and big nets and fixed and movable macros
on both sides of the scans' edges (4 items a thread of 1024 in the one-launch
form, 16384 items and the tiled form above), so that every rank and class
count is carried across them: structure bit-exact against the oracle's, with
and without hints, and the filter within its FP32 bound."""
import numpy as np
import pytest
import torch

import gpu_common as U
import netlists as H
from oracle import ahr_oracle as O

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2511_10073_amd")

EDGES = (0, 4096, 16384)
HUBS = (9, 17, 33, 65, 2049)
STARS = (11, 20, 64, 65, 70, 300)


def mixed(n):
    """A ring of n cells; hubs, star nets and macros next to every edge below n."""
    rng = np.random.default_rng(n)
    flags, pos = np.zeros(n, np.uint8), [e for e in EDGES if e < n] + [n - 12]
    nets = [[i, (i + 1) % n] for i in range(n)]
    at = {}                                   # ring net -> the nets put before it
    for e in pos:
        near = [(e + k) % n for k in range(-8, 9)]
        for h, d in enumerate(HUBS):
            cells = rng.permutation(n)[:min(d, n - 1)]
            at.setdefault(near[h + 5], []).extend([near[h + 5], int(c)] for c in cells if c != near[h + 5])
        for k, d in enumerate(STARS):
            at.setdefault(near[3 * k % 17], []).append([int(c) for c in rng.permutation(n)[:min(d, n)]])
        for k, v in enumerate(near):
            if k % 3 == 0:
                flags[v] = H.MACRO | (H.FIXED if k % 2 else 0)
    nets = [x for i, e in enumerate(nets) for x in at.get(i, []) + [e]]
    sizes = np.where((flags & H.MACRO) > 0, 3.0, 0.1).astype(np.float32)[:, None].repeat(2, 1)
    offsets = rng.uniform(-0.05, 0.05, (sum(map(len, nets)), 2)).astype(np.float32)
    return H.make(nets, n, flags=flags, sizes=sizes, offsets=offsets)


@pytest.mark.parametrize("hints", [False, True])
@pytest.mark.parametrize("n", [700, 4080, 4095, 4097, 12000, 16385, 20481])
def test_mixed_rows_at_scan_edges(n, hints):
    nl = mixed(n)
    p = U.params32(O.HintParams(nbx=4, nby=5, detection_ratio=0.5, macro_hints=hints, bin_hints=hints,
                                expand_macro_pins=hints))
    og = O.build_graph(nl, p, nl["g0"])
    x = torch.as_tensor(nl["g0"]).cuda()
    gr = A.Graph(A.Netlist(nl), U.to_c_params(A, p), x)
    spec = U.spec32(O.FilterSpec(ks=(2, 4), alphas=(0.4, 0.6)))
    try:
        ex = gr.export()
        out = gr.filter(U.to_c_spec(A, spec), x).cpu().numpy()
    finally:
        gr.close()
    assert np.array_equal(ex["net_row_ptr"], og.net_row_ptr.astype(np.int32))
    assert np.array_equal(ex["net_col"], og.net_col.astype(np.int32))
    assert np.array_equal(ex["net_q"], og.net_q)
    assert np.array_equal(ex["hint_row_ptr"], og.hint_row_ptr.astype(np.int32))
    r1, c1, _ = U.sorted_rows(ex["hint_row_ptr"], ex["hint_col"], ex["hint_val"])
    r0, c0, _ = U.sorted_rows(og.hint_row_ptr, og.hint_col, og.hint_val)
    assert np.array_equal(r1, r0) and np.array_equal(c1, c0)
    U.check_filter(out, O.apply_filter(nl, og, spec, nl["g0"]), U.movable_rows(nl))
