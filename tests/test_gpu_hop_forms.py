"""The forms of a hop that its size decides: more than 12M entries (with 8
columns or 2 lanes a row, long rows are summed in parts whatever their length),
no long row at all, and every number of lanes; within the FP32 bound of the
oracle."""
import numpy as np
import pytest
import torch

import gpu_common as U
import netlists as H
from oracle import ahr_oracle as O

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2511_10073_amd")

BANK = U.spec32(O.FilterSpec(ks=(1, 2), alphas=(0.4, 0.6)))
OFF = dict(nbx=3, nby=3, macro_hints=False, bin_hints=False)


def cliques(n, nets, deg, hub):
    """`nets` nets of `deg` pins among n cells, 61 apart in steps that differ, and a hub with `hub` cells."""
    at = np.random.default_rng(nets).integers(0, n - 1, (nets, 1))
    lists = ((at + 61 * np.arange(deg) ** 2) % (n - 1) + 1).tolist()
    return H.make([[0, 1 + k] for k in range(hub)] + lists, n, ncols=8)


def check(nl, lanes, cols):
    p = U.params32(O.HintParams(**OFF))
    og = O.build_graph(nl, p, nl["g0"][:, :2])
    net, spec, mov = A.Netlist(nl), U.to_c_spec(A, BANK), U.movable_rows(nl)
    gr = A.Graph(net, U.to_c_params(A, p), torch.as_tensor(nl["g0"]).cuda())
    saved = A.filter_get_tune()
    try:
        for c in cols:
            g = np.ascontiguousarray(nl["g0"][:, :c])
            ref, x = O.apply_filter(nl, og, BANK, g), torch.as_tensor(g).cuda()
            for l in lanes:
                A.filter_tune(l, -1)
                y = gr.filter(spec, x).clone()
                assert torch.equal(y, gr.filter(spec, x))
                U.check_filter(y.cpu().numpy(), ref, mov)
    finally:
        A.filter_tune(*saved)
        gr.close()
    return og


def test_more_than_12M_entries():
    og = check(cliques(1_000_000, 150_000, 10, 2500), (2, 4, A.HOP_ROW_BLOCK), (2, 8))
    assert int(og.net_row_ptr[-1]) > 12_000_000


@pytest.mark.parametrize("hub", [0, 100, 3000])
def test_lanes(hub):
    og = check(cliques(4000, 900, 6, hub), (1, 2, 4, 8, 16, 32, 64, A.HOP_ROW_BLOCK), (1, 4))
    assert (int(np.diff(og.net_row_ptr).max()) > 128) == (hub == 3000)
