"""Rows at the edges of the chunks that long rows are summed in (128 entries
and more, 2048 a chunk, 1 to 8 entries a lane), with and without hints, every
column count, alone and as members of a batch: the filter within its FP32
bound of the oracle, first and second call (the first forms the spectral bound
inside its first hop) and both launch forms of the hop alike."""
import numpy as np
import pytest
import torch

import gpu_common as U
import netlists as H
from oracle import ahr_oracle as O

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2511_10073_amd")

SIZES = [100, 127, 128, 129, 255, 256, 257, 511, 513, 1024, 1025, 2047, 2048, 2049, 4096, 4100, 6200]
BANK = U.spec32(O.FilterSpec(ks=(2, 4), alphas=(0.4, 0.6)))


def hubs(hints):
    """One hub per size, joined to that many cells by 2-pin nets, and a star of as many pins."""
    rng = np.random.default_rng(7)
    first, n = len(SIZES), 7000
    nets = []
    for h, d in enumerate(SIZES):
        cells = first + rng.permutation(n)[:d]
        nets += [[h, int(c)] for c in cells]
        nets.append([int(c) for c in cells])
    nl = H.make(nets, first + n, ncols=8)
    p = U.params32(O.HintParams(nbx=3, nby=3, detection_ratio=0.4, macro_hints=hints, bin_hints=hints))
    return nl, p


@pytest.mark.parametrize("hints", [False, True])
@pytest.mark.parametrize("cols", [1, 2, 4, 8])
def test_chunk_edges(hints, cols):
    nl, p = hubs(hints)
    og = O.build_graph(nl, p, nl["g0"][:, :2])
    g = np.ascontiguousarray(nl["g0"][:, :cols])
    ref, mov = O.apply_filter(nl, og, BANK, g), U.movable_rows(nl)
    x, saved = torch.as_tensor(g).cuda(), A.filter_get_tune()
    try:
        for lanes in (4, A.HOP_ROW_BLOCK):
            A.filter_tune(lanes, -1)
            gr = A.Graph(A.Netlist(nl), U.to_c_params(A, p), torch.as_tensor(nl["g0"]).cuda())
            try:
                y = gr.filter(U.to_c_spec(A, BANK), x).clone()
                assert torch.equal(y, gr.filter(U.to_c_spec(A, BANK), x))
            finally:
                gr.close()
            U.check_filter(y.cpu().numpy(), ref, mov)
    finally:
        A.filter_tune(*saved)


def test_chunk_edges_in_a_batch():
    members = [hubs(False), hubs(True)]
    x = torch.as_tensor(np.concatenate([nl["g0"][:, :4] for nl, _ in members])).cuda()
    b = A.Batch([A.Netlist(nl) for nl, _ in members], [U.to_c_params(A, p) for _, p in members], x)
    out = b.filter(U.to_c_spec(A, BANK), x).cpu().numpy()
    n = members[0][0]["n_inst"]
    for k, (nl, p) in enumerate(members):
        og = O.build_graph(nl, p, nl["g0"][:, :2])
        ref = O.apply_filter(nl, og, BANK, np.ascontiguousarray(nl["g0"][:, :4]))
        U.check_filter(out[k * n:(k + 1) * n], ref, U.movable_rows(nl))
