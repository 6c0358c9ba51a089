"""The longest row's chunks of 2048 entries and the graph's entries decide how
its hops finish the long rows: inside the hop (up to 2 chunks, 3 in small
graphs, 4 of a hint node; in large graphs up to 8), or in partial sums that a launch of their own adds up.  Both sides of
those edges, for an instance's row, a star's and a bin's (where no instance has
a long row), in every column count and both launch forms, within the FP32 bound
of the oracle; and in batches, which take one form for all members, every
member the same bits as by itself, where the other form may be taken."""
import numpy as np
import pytest
import torch

import gpu_common as U
import netlists as H
from oracle import ahr_oracle as O

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2511_10073_amd")

WHOLE = 8 * 2048
BANK = U.spec32(O.FilterSpec(ks=(2, 4), alphas=(0.4, 0.6)))
FIXED = U.spec32(O.FilterSpec(ks=(3,), alphas=(1.0,), lambda_mode="fixed", lambda_fixed=2.5))
OFF = dict(nbx=3, nby=3, macro_hints=False, bin_hints=False)


def graph(kind, d):
    """A graph whose longest row, of d entries, is an instance's, a star's or a
    bin's; "large": a hub's, beside 6.3M entries of 10-pin nets."""
    if kind in ("hub", "large"):        # the hub, its d cells, and a second hub on a few of them
        nets, n = [[0, 2 + k] for k in range(d)] + [[1, 2 + k] for k in range(0, d, 61)], d + 2
        if kind == "large":
            n = 200_000
            at = np.random.default_rng(d).integers(0, n - 2, (92_000, 1))
            nets += ((at + 1009 * np.arange(10) ** 2) % (n - 2) + 2).tolist()
        return H.make(nets, n, ncols=8), U.params32(O.HintParams(**OFF))
    if kind == "star":
        nets = [list(range(d))] + [[k, k + 1] for k in range(0, d - 1, 3)]
        return H.make(nets, d + 5, ncols=8), U.params32(O.HintParams(**OFF))
    nl = H.make([[k, (k + 1) % d] for k in range(d)], d, ncols=8)
    return nl, U.params32(O.HintParams(nbx=1, nby=1, macro_hints=False))


def longest_row(og):
    return int((np.diff(og.net_row_ptr) + np.diff(og.hint_row_ptr)).max())


@pytest.mark.parametrize("kind,d", [(k, d) for k in ("hub", "star", "bin")
                                    for d in (4096, 4097, 6144, 6145, 8192, 8193, WHOLE - 1, WHOLE, WHOLE + 1, 20000)]
                         + [("large", 4097), ("large", WHOLE), ("large", WHOLE + 1)])
def test_longest_row(kind, d):
    nl, p = graph(kind, d)
    og = O.build_graph(nl, p, nl["g0"][:, :2])
    assert longest_row(og) == d
    mov, saved = U.movable_rows(nl), A.filter_get_tune()
    net, spec, place = A.Netlist(nl), U.to_c_spec(A, BANK), torch.as_tensor(nl["g0"]).cuda()
    try:
        for cols in (1, 2, 4, 8):
            g = np.ascontiguousarray(nl["g0"][:, :cols])
            ref, x = O.apply_filter(nl, og, BANK, g), torch.as_tensor(g).cuda()
            for lanes in (4, A.HOP_ROW_BLOCK):
                A.filter_tune(lanes, -1)
                gr = A.Graph(net, U.to_c_params(A, p), place)
                try:
                    y = gr.filter(spec, x).clone()      # (with up to 4 columns the bound is formed in this hop)
                    assert torch.equal(y, gr.filter(spec, x))
                finally:
                    gr.close()
                U.check_filter(y.cpu().numpy(), ref, mov)
    finally:
        A.filter_tune(*saved)


@pytest.mark.parametrize("cols", [1, 2, 4, 8])
@pytest.mark.parametrize("long", [[("hub", WHOLE), ("hub", WHOLE + 1)], [("star", 20000), ("star", WHOLE)],
                                  [("hub", 3000), ("bin", 20000), ("star", WHOLE - 1)],
                                  [("large", 3000), ("hub", WHOLE), ("star", 6200), ("bin", 9000)]])
def test_one_longer_row_in_a_batch(cols, long):
    members = [graph(kind, d) for kind, d in long]
    nets = [A.Netlist(nl) for nl, _ in members]
    xs = [np.ascontiguousarray(nl["g0"][:, :cols]) for nl, _ in members]
    place = torch.as_tensor(np.concatenate([nl["g0"] for nl, _ in members])).cuda()
    x = torch.as_tensor(np.concatenate(xs)).cuda()
    b = A.Batch(nets, [U.to_c_params(A, p) for _, p in members], place)
    ends = np.cumsum([0] + [nl["n_inst"] for nl, _ in members])
    saved = A.filter_get_tune()
    try:
        for lanes in (4, A.HOP_ROW_BLOCK):
            A.filter_tune(lanes, -1)
            b.set_config(cols, lanes)
            for s in (BANK, FIXED):
                out = b.filter(U.to_c_spec(A, s), x).clone()
                for k, (nl, p) in enumerate(members):
                    gr = A.Graph(nets[k], U.to_c_params(A, p), torch.as_tensor(nl["g0"]).cuda())
                    try:
                        alone = gr.filter(U.to_c_spec(A, s), torch.as_tensor(xs[k]).cuda())
                        assert torch.equal(out[ends[k]:ends[k + 1]], alone), (k, lanes)
                    finally:
                        gr.close()
                    if s is FIXED:
                        og = O.build_graph(nl, p, nl["g0"][:, :2])
                        U.check_filter(out[ends[k]:ends[k + 1]].cpu().numpy(), O.apply_filter(nl, og, s, xs[k]),
                                       U.movable_rows(nl))
    finally:
        A.filter_tune(*saved)
        b.close()
