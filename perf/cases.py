"""The work that a user of this library has it do, as cases that can be timed.

Every case goes through the public Python binding.  Netlists are synthetic, of
the shapes that the repository's own generator states (synth/netlist.py:
degree mix, locality-biased pins on a hidden lattice, macro sizes and area
share, pins at macro boundaries, a centre-concentrated first placement), drawn
here on the GPU so that a 2.2M-cell netlist takes well under a second.
"""
from __future__ import annotations

import json
import math

import numpy as np
import torch

import paper_2511_10073_amd as A

DEV = "cuda"
F64 = torch.float64
MODEL = "paper_2511_10073_amd/weights/surrogate_bank248.json"
BANK = ((2, 4, 8), (0.2, 0.3, 0.5))          # the order-8 three-band bank of the benchmark
GIFT = ((2, 2, 4), (2.0, 4.0, 4.0), (0.2, 0.3, 0.5))


def listed():
    return [
        # Scoring one small placement, as an outer loop does after each move: latency alone.
        dict(name="hpwl-2k", kind="hpwl", cells=2000, cols=2),
        # Scoring two candidate placements of a full-size design.
        dict(name="hpwl-1.1M", kind="hpwl", cells=1_100_003, cols=4),
        # The initializer (Algorithm 1, three rounds, graph built from the netlist in the call) on
        # a small block with movable macros and the order-4 filter of one (x, y) placement.
        dict(name="refine-2k", kind="refine", cells=2000, cols=2, bins=8, rounds=3, order=4, prune=0.0, movable=True),
        # The same on a mid-size design with fixed macros and the order-8 bank, two placements at a time.
        dict(name="refine-210k", kind="refine", cells=210_000, cols=4, bins=32, rounds=3, order=8, prune=0.0,
             movable=False),
        # One round with sparsified hints (only salient bin edges kept), an odd size and one placement.
        dict(name="refine-73k-pruned", kind="refine", cells=73_013, cols=2, bins=24, rounds=1, order=8, prune=0.1,
             movable=False),
        # The headline: the initializer on 2.2M cells.
        dict(name="refine-2.2M", kind="refine", cells=2_200_000, cols=4, bins=32, rounds=3, order=8, prune=0.0,
             movable=False),
        # A graph that is kept, filtering new signals: four placements at once on an odd size.
        dict(name="filter-517k", kind="filter", cells=517_019, cols=8, bins=32, order=8),
        # The learned filter in place of the order-8 bank on a kept graph.
        dict(name="learned-880k", kind="learned", cells=880_001, cols=4, bins=32),
        # The initializer's own start: graph build and GiFt's bank on uniformly drawn positions.
        dict(name="gift-600k", kind="gift", cells=600_000, cols=2),
        # Many netlists of uneven size filtered in one captured call.
        dict(name="batch-24", kind="batch", members=24, smallest=5000, largest=100_000, cols=4),
        # What a global placer asks for at every iteration: WA wirelength and its gradient.
        dict(name="wa-2.2M", kind="wa", cells=2_200_000, cols=2),
        # One full-batch training step of the surrogate's network (gradient and Adam).
        dict(name="train-1.6M", kind="train", rows=1_600_000),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["hpwl", "refine", "refine", "filter", "learned", "gift", "batch", "wa", "train", "charge"])
    if kind == "hpwl":
        return dict(kind=kind, cells=_size(rng, 2000, 2_200_000), cols=rng.choice([2, 4, 8]))
    if kind == "refine":
        cells = _size(rng, 2000, 1_500_000)
        return dict(kind=kind, cells=cells, cols=rng.choice([2, 4]), bins=rng.choice([8, 16, 27, 32, 40]),
                    rounds=rng.choice([1, 2, 3]), order=rng.choice([4, 8]), prune=rng.choice([0.0, 0.0, 0.05, 0.2]),
                    movable=cells < 20_000 and rng.random() < 0.5)
    if kind == "filter":
        return dict(kind=kind, cells=_size(rng, 2000, 1_000_000), cols=rng.choice([1, 2, 4, 8]),
                    bins=rng.choice([8, 16, 32]), order=rng.choice([4, 8]))
    if kind == "learned":
        return dict(kind=kind, cells=_size(rng, 20_000, 1_500_000), cols=rng.choice([2, 4]), bins=rng.choice([16, 32]))
    if kind == "gift":
        return dict(kind=kind, cells=_size(rng, 2000, 1_500_000), cols=rng.choice([2, 4]))
    if kind == "batch":
        return dict(kind=kind, members=rng.randint(2, 24), smallest=rng.randint(3000, 8000),
                    largest=rng.randint(20_000, 100_000), cols=rng.choice([2, 4]))
    if kind == "wa":
        return dict(kind=kind, cells=_size(rng, 2000, 2_200_000), cols=rng.choice([2, 4]))
    if kind == "train":
        return dict(kind=kind, rows=_size(rng, 5000, 1_600_000))
    # Per-bin macro charge of a placer's density step, all four models.
    return dict(kind="charge", cells=_size(rng, 20_000, 1_000_000), model=rng.randint(0, 3), t=rng.randint(1, 299),
                bins=rng.choice([32, 64, 100]))


# ---------------------------------------------------------------- inputs

def _shape(cells, movable=False):
    """Macros, I/O pins, nets and the large nets' share and sizes of a netlist
    of `cells` standard cells: the rates of the repository's tiny, mid and
    large configurations, interpolated in log(size)."""
    t = min(1.0, max(0.0, math.log(cells / 210_000) / math.log(2_200_000 / 210_000)))
    mix = lambda a, b: (1 - t) * a + t * b
    if cells < 20_000:
        return dict(macros=max(8, cells // 250), io=max(32, cells // 200), nets=int(cells * 1.1),
                    big=(0.0, 51, 51), side=(20.0, 60.0), area=-1.0 if movable else 0.3)
    return dict(macros=int(cells * mix(500 / 210e3, 8000 / 2.2e6)), io=int(cells * mix(1200 / 210e3, 8000 / 2.2e6)),
                nets=int(cells * mix(220 / 210, 225 / 220)),
                big=(mix(0.005, 0.0001), 51, int(min(cells / 50, mix(2000, 10_000)))), side=(10.0, 200.0), area=0.4)


def _member_shape(cells):
    """A netlist of the uneven batched workload (3.5 % macros)."""
    return dict(macros=max(2, int(cells * 0.035)), io=max(8, cells // 200), nets=int(cells * 1.05),
                big=(0.002, 51, max(52, min(2000, cells // 50))), side=(4.0, 80.0), area=0.3)


def _shelves(rng, w, h, die):
    """Non-overlapping macro centres: shelves of similar heights in random
    order, the free length of every shelf and of the die spread evenly."""
    order, shelves, x = np.argsort(-h, kind="stable"), [[]], 0.0
    for m in order:
        if x + w[m] > 0.92 * die and shelves[-1]:
            shelves.append([])
            x = 0.0
        shelves[-1].append(m)
        x += w[m]
    rng.shuffle(shelves)
    pos = np.zeros((w.size, 2))
    gap_y = max(0.0, die - sum(max(h[s]) for s in shelves)) / (len(shelves) + 1)
    y = -die / 2
    for s in shelves:
        s = np.array(s)
        rng.shuffle(s)
        gap = max(0.0, die - w[s].sum()) / (s.size + 1)
        pos[s, 0] = -die / 2 + np.cumsum(w[s] + gap) - w[s] / 2
        pos[s, 1] = y + gap_y + h[s].max() / 2
        y += gap_y + h[s].max()
    return pos


def _netlist(cells, shape, cols, seed, movable=False, uniform=False):
    """Device arrays of one netlist and its first placement g0 [n_inst, cols]."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng(seed)
    rand = lambda *n: torch.rand(n, generator=gen, device=DEV, dtype=F64)
    ints = lambda lo, hi, n: torch.randint(lo, hi, (n,), generator=gen, device=DEV)
    ar = lambda n: torch.arange(n, device=DEV)
    nm, nio = shape["macros"], shape["io"]
    n_inst = cells + nm + nio

    std_w = ints(1, 5, cells).double()
    lo, hi = shape["side"]
    side, aspect = np.exp(rng.uniform(math.log(lo), math.log(hi), nm)), rng.uniform(0.8, 1.25, nm)
    mw, mh = side * np.sqrt(aspect), side / np.sqrt(aspect)
    std_area = float(std_w.sum())
    if shape["area"] > 0:
        f = math.sqrt(shape["area"] / (1 - shape["area"]) * std_area / float((mw * mh).sum()))
        mw, mh = mw * f, mh * f
    mw, mh = np.maximum(np.round(mw), 2.0), np.maximum(np.round(mh), 2.0)
    die = float(math.ceil(math.sqrt((std_area + float((mw * mh).sum())) / 0.70)))
    half = die / 2
    if movable:
        mpos = np.stack([rng.uniform(-half + mw / 2, half - mw / 2), rng.uniform(-half + mh / 2, half - mh / 2)], 1)
    else:
        mpos = _shelves(rng, mw, mh, die)
    t = (np.arange(nio) + rng.uniform(0.2, 0.8, nio)) / nio * 4.0
    k, f = np.floor(t), (t - np.floor(t)) * die - half
    iopos = np.stack([np.choose(k.astype(int), [f, half + 0 * f, -f, -half + 0 * f]),
                      np.choose(k.astype(int), [-half + 0 * f, f, half + 0 * f, -f])], 1)

    # nets: degrees, pins near an anchor on the hidden lattice, no repeated cell in a net
    lw = math.ceil(math.sqrt(cells))
    lh = math.ceil(cells / lw)
    share, big_lo, big_hi = shape["big"]

    def local(anchor, rad):
        n = anchor.numel()
        off = lambda: torch.floor(rand(n) * (2 * rad + 1)).long() - rad
        x, y = (anchor % lw + off()).clamp(0, lw - 1), (anchor // lw + off()).clamp(0, lh - 1)
        c = y * lw + x
        return torch.where((rand(n) < 0.9) & (c < cells), c, ints(0, cells, n))

    n_main = max(1, int(shape["nets"] * 0.97))
    u = rand(n_main)
    deg = torch.where(u < 0.6, 2, torch.where(u < 0.8, 3, torch.where(u < 0.97, ints(4, 11, n_main),
                                                                      ints(11, 51, n_main))))
    big = torch.exp(math.log(big_lo) + rand(n_main) * math.log((big_hi + 1) / big_lo)).long().clamp(big_lo, big_hi)
    deg = torch.where(u >= 1 - share, big, deg) if share > 0 else deg
    deg = deg.clamp(max=max(2, cells // 4))
    anchor = ints(0, cells, n_main)
    net = torch.repeat_interleave(ar(n_main), deg)
    first = torch.cumsum(deg, 0) - deg
    rad = torch.round(2 * torch.sqrt(deg.double())).long().clamp(min=1)
    pin = local(anchor[net], rad[net])
    pin[first] = anchor
    for _ in range(20):
        key = net * (2 * cells) + 2 * pin + 1
        key[first] -= 1                                   # the anchor sorts first and stays
        skey, o = torch.sort(key)
        dup = o[1:][(skey[1:] >> 1) == (skey[:-1] >> 1)]
        if dup.numel() == 0:
            break
        pin[dup] = local(anchor[net[dup]], rad[net[dup]])
    lone = torch.ones(cells, dtype=torch.bool, device=DEV)
    lone[pin] = False
    lone = torch.nonzero(lone).ravel()
    more = max(0, shape["nets"] - n_main - lone.numel())
    a2 = torch.cat([lone, ints(0, cells, more)])
    b2 = torch.where(a2 + 1 < cells, a2 + 1, a2 - 1)
    n_nets = n_main + a2.numel()
    extra = n_main + ar(a2.numel())
    anchor = torch.cat([anchor, a2])

    # macro boundary pins and I/O pins join a net anchored near them
    at = lambda a, l: (a.double() + 0.5) / l * die - half
    coarse = max(1, int(math.sqrt(n_nets / 8)))
    tile = lambda x, y: (((y + half) / die * coarse).long().clamp(0, coarse - 1) * coarse
                         + ((x + half) / die * coarse).long().clamp(0, coarse - 1))
    tiles, by_tile = torch.sort(tile(at(anchor % lw, lw), at(anchor // lw, lh)), stable=True)

    def nets_near(x, y):
        b = tile(x, y)
        lo_, hi_ = torch.searchsorted(tiles, b), torch.searchsorted(tiles, b + 1)
        got = by_tile[(lo_ + (rand(b.numel()) * (hi_ - lo_)).long()).clamp(max=n_nets - 1)]
        return torch.where(hi_ > lo_, got, ints(0, n_nets, b.numel()))

    dev = lambda a: torch.as_tensor(a).to(DEV)
    w_, h_, mp, ip = dev(mw), dev(mh), dev(mpos), dev(iopos)
    owner = torch.repeat_interleave(ar(nm), (1.5 * (w_ + h_)).round().long().clamp(8, 512))
    wo, ho = w_[owner], h_[owner]
    s = rand(owner.numel()) * 2 * (wo + ho)
    ox = torch.where(s < wo, s - wo / 2, torch.where(s < wo + ho, wo / 2, torch.where(
        s < 2 * wo + ho, wo / 2 - (s - wo - ho), -wo / 2)))
    oy = torch.where(s < wo, -ho / 2, torch.where(s < wo + ho, -ho / 2 + (s - wo), torch.where(
        s < 2 * wo + ho, ho / 2, ho / 2 - (s - 2 * wo - ho))))
    off = torch.stack([ox, oy], 1).mul(2).round().div(2)
    all_net = torch.cat([net, extra, extra, nets_near(mp[owner, 0] + off[:, 0], mp[owner, 1] + off[:, 1]),
                         nets_near(ip[:, 0], ip[:, 1])])
    perm = torch.randperm(n_inst, generator=gen, device=DEV)
    node = perm[torch.cat([pin, a2, b2, cells + owner, cells + nm + ar(nio)])]
    pin_off = torch.zeros(node.numel(), 2, device=DEV)
    pin_off[node.numel() - nio - owner.numel():node.numel() - nio] = off.float()
    all_net, o = torch.sort(all_net, stable=True)
    net_ptr = torch.zeros(n_nets + 1, dtype=torch.int64, device=DEV)
    net_ptr[1:] = torch.cumsum(torch.bincount(all_net, minlength=n_nets), 0)

    flags = torch.zeros(n_inst, dtype=torch.uint8, device=DEV)
    flags[perm[cells:cells + nm]] = A.MACRO | (0 if movable else A.FIXED)
    flags[perm[cells + nm:]] = A.FIXED
    size = torch.zeros(n_inst, 2, device=DEV)
    size[perm[:cells], 0], size[perm[:cells], 1] = std_w.float(), 1.0
    size[perm[cells:cells + nm]] = torch.stack([w_, h_], 1).float()

    # movable cells: a centre-concentrated warp of the lattice with noise of one spacing per
    # placement, or uniform in the die; macros and I/O pins where they were drawn
    g0 = torch.empty(n_inst, cols, device=DEV)
    c = ar(cells)
    for j in range(cols):
        if uniform:
            v = (rand(cells) - 0.5) * die
        else:
            q = ((c % lw if j % 2 == 0 else c // lw).double() + 0.5) / (lw if j % 2 == 0 else lh)
            v = die / 6 * torch.special.ndtri(q) + torch.randn(cells, generator=gen, device=DEV, dtype=F64) * die / lw
        g0[perm[:cells], j] = v.clamp(-half, half).float()
        g0[perm[cells:], j] = torch.cat([mp, ip])[:, j % 2].float()
    return dict(n_inst=n_inst, net_ptr=net_ptr, pin_node=node[o], pin_off=pin_off[o], node_flags=flags,
                node_size=size, die=[-half, -half, half, half], g0=g0)


def _handle(nl):
    host = {k: (v.cpu().numpy() if torch.is_tensor(v) else v) for k, v in nl.items() if k != "g0"}
    return A.Netlist(host, DEV)


def _hints(case):
    return A.hint_params(nbx=case["bins"], nby=case["bins"], prune_tau=case.get("prune", 0.0))


def _bands(case):
    return ((4,), (1.0,)) if case.get("order") == 4 else BANK


def _members(case, seed):
    rng = np.random.default_rng(case["members"])      # the sizes are the case's, whatever the inputs' seed
    sizes = np.exp(rng.uniform(math.log(case["smallest"]), math.log(case["largest"]), case["members"])).astype(int)
    sizes[0], sizes[-1] = case["smallest"], case["largest"]
    return [_netlist(int(n), _member_shape(int(n)), case["cols"], 1000 * seed + i) for i, n in enumerate(sizes)]


def _member_bins(n):
    return int(min(32, max(8, round(math.sqrt(n / 200)))))


def _one(case, seed):
    return _netlist(case["cells"], _shape(case["cells"], case.get("movable", False)), case.get("cols", 2), seed,
                    movable=case.get("movable", False), uniform=case["kind"] == "gift")


def _training(case, seed):
    """Feature rows with the features' scales (hop differences near 1, the standardised hop, log
    degree, hint share, log scale ratio), unit-deviation targets and a half-trained network."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    n = lambda *s: torch.randn(s, generator=gen, device=DEV)
    rows = case["rows"]
    F = torch.zeros(rows, 8, device=DEV)
    F[:, :4] = n(rows, 4) * torch.tensor([1.0, 0.6, 0.3, 1.0], device=DEV)
    F[:, 4] = 1.4 + 0.4 * n(rows)
    F[:, 5] = -0.3 + 0.2 * n(rows)
    F[:, 6] = 2.3 + 1.2 * torch.rand(rows, generator=gen, device=DEV)
    R = 0.5 * F[:, 0] * F[:, 1] - 0.4 * F[:, 2].abs() + 0.7 * n(rows)
    W1 = torch.zeros(64, 8, device=DEV)
    W1[:, :7] = n(64, 7) * math.sqrt(2 / 7)
    P = torch.cat([W1.ravel(), 0.1 * n(64), (n(64, 64) * math.sqrt(2 / 64)).ravel(), 0.1 * n(64), 0.1 * n(64),
                   0.1 * n(1)])
    m, v = 1e-3 * n(P.numel()), (1e-3 * (1 + torch.rand(P.numel(), generator=gen, device=DEV))) ** 2
    return F, R, P, m, v


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        F, R, P, m, v = _training(case, seed)
        return dict(kind=kind, F=F, R=R, P=P, m=m, v=v, grad=torch.empty_like(P),
                    loss=torch.empty(1, dtype=F64, device=DEV), step=500)
    if kind == "batch":
        nls = _members(case, seed)
        x = torch.cat([nl["g0"] for nl in nls])
        spec = A.filter_spec(*BANK)
        b = A.Batch([_handle(nl) for nl in nls],
                    [A.hint_params(nbx=_member_bins(nl["n_inst"]), nby=_member_bins(nl["n_inst"])) for nl in nls], x)
        b.autotune(spec, case["cols"])
        return dict(kind=kind, batch=b, spec=spec, x=x, out=torch.empty_like(x))
    nl = _one(case, seed)
    net, x = _handle(nl), nl["g0"]
    s = dict(kind=kind, net=net, x=x, out=torch.empty_like(x))
    if kind == "hpwl":
        s["out"] = torch.empty(case["cols"] // 2, dtype=F64, device=DEV)
    elif kind == "refine":
        s.update(hints=_hints(case), spec=A.filter_spec(*_bands(case)), rounds=case["rounds"])
    elif kind in ("filter", "learned"):
        s.update(graph=A.Graph(net, _hints(case), x), spec=A.filter_spec(*_bands(case)))
        if kind == "learned":
            s["model"] = A.Mlp.load(MODEL, DEV)
    elif kind == "gift":
        s.update(hints=A.hint_params(flags=0), spec=A.gift_spec(*GIFT))
    elif kind == "wa":
        s["wl"] = A.Wirelength(net)
    elif kind == "charge":
        s["charge"] = A.charge_params(case["model"], t=case["t"], nbx=case["bins"], nby=case["bins"])
        s["out"] = torch.empty(case["bins"] ** 2, dtype=F64, device=DEV)
    return s


def run(s):
    kind = s["kind"]
    if kind == "hpwl":
        return A.hpwl(s["net"], s["x"], s["out"])
    if kind == "refine":
        return A.refine(s["net"], s["hints"], s["spec"], s["x"], s["rounds"], 0.5, s["out"])
    if kind == "filter":
        return s["graph"].filter(s["spec"], s["x"], s["out"])
    if kind == "learned":
        return s["graph"].filter_learned(s["spec"], s["model"], s["x"], s["out"])[0]
    if kind == "gift":
        g = A.Graph(s["net"], s["hints"], s["x"])
        g.gift(s["spec"], s["x"], s["out"])
        g.close()
        return s["out"]
    if kind == "batch":
        return s["batch"].filter(s["spec"], s["x"], s["out"])
    if kind == "wa":
        return s["wl"].wa(s["x"], 4.0)
    if kind == "charge":
        return A.macro_charge(s["net"], s["x"], s["charge"], s["out"])
    A.mlp_loss_grad(s["P"], s["F"], s["R"], s["grad"], s["loss"])
    A.mlp_adam(s["P"], s["m"], s["v"], s["grad"], s["step"], 1e-3)
    return dict(grad=s["grad"], params=s["P"], m=s["m"], v=s["v"])


def work(case):
    kind = case["kind"]
    if kind == "train":
        # features and targets in; forward 2 (8 + 64 + 1) 64, backward twice that without the input's
        return dict(bytes=36.0 * case["rows"], flops=case["rows"] * 64 * (2.0 * 73 + 2.0 * 73 + 2.0 * 65))
    if kind == "batch":
        lo, hi = case["smallest"], case["largest"]
        cells = case["members"] * (hi - lo) / max(math.log(hi / lo), 1e-9)
        shape = dict(nets=1.05 * cells, macros=0.035 * cells)
    else:
        cells = case["cells"]
        shape = _shape(cells, case.get("movable", False))
    N = cells * 1.01 + shape["macros"]
    E, P, C = shape["nets"], 4.0 * shape["nets"] + 40 * shape["macros"], case.get("cols", 2)
    netlist, signal = 4.0 * E + 12.0 * P + 9.0 * N, 4.0 * C * N
    nnz = 12.5 * E + (0 if kind == "gift" else 18.0 * cells)      # graph entries, a hint edge counted both ways
    hop = 2.0 * nnz * C
    if kind == "hpwl":
        return dict(bytes=4.0 * E + 12.0 * P + signal, flops=6.0 * P * C)
    if kind == "wa":
        return dict(bytes=4.0 * E + 12.0 * P + 2 * signal, flops=30.0 * P * C)
    if kind == "charge":
        return dict(bytes=17.0 * N + 8.0 * case["bins"] ** 2, flops=200.0 * (shape["macros"] + case["bins"] ** 2))
    if kind == "refine":
        hops = case["rounds"] * max(_bands(case)[0])
        return dict(bytes=netlist + 2 * signal, flops=hop * hops)
    if kind == "gift":
        return dict(bytes=netlist + 2 * signal, flops=6 * hop)
    # a kept graph: its entries (column and weight) once, the signal in and out
    hops = 3 if kind == "learned" else max(_bands(case)[0])
    return dict(bytes=8.0 * nnz + 2 * signal, flops=hop * hops + (9000.0 * N * C if kind == "learned" else 0))


# ---------------------------------------------------------------- the same in 64 bits

def _expand(n, lens):
    """For rows 0..n-1 with lens entries each: row of every entry, its place in the row."""
    row = torch.repeat_interleave(torch.arange(n, device=DEV), lens)
    return row, torch.arange(row.numel(), device=DEV) - (torch.cumsum(lens, 0) - lens)[row]


class _Graph64:
    """The netlist's weighted clique/star graph, merged, in 64 bits."""

    def __init__(self, nl, expand=True, hints=True, bins=0, clique_max=10):
        f = nl["node_flags"].long()
        self.nl, self.n, self.bins = nl, nl["n_inst"], bins
        self.fixed, self.macro = (f & 1) > 0, (f & 2) > 0
        ptr, pin = nl["net_ptr"], nl["pin_node"].clone()
        deg = ptr[1:] - ptr[:-1]
        self.mp = torch.nonzero(self.fixed[pin] & self.macro[pin]).ravel() if expand else pin[:0]
        self.mp_owner = pin[self.mp]
        pin[self.mp] = self.n + torch.arange(self.mp.numel(), device=DEV)
        self.star0 = self.n + self.mp.numel()
        stars = torch.nonzero(deg > clique_max).ravel()
        self.mv0 = self.star0 + stars.numel()
        self.macros = torch.nonzero(self.macro).ravel() if hints else pin[:0]
        self.bv0 = self.mv0 + self.macros.numel()
        self.total = self.bv0 + (bins * bins if hints else 0)
        r, c, w = [], [], []
        for p in range(2, clique_max + 1):
            nets = torch.nonzero(deg == p).ravel()
            ids = pin[ptr[nets][:, None] + torch.arange(p, device=DEV)]
            a, b = ids[:, :, None].expand(-1, p, p).reshape(-1), ids[:, None, :].expand(-1, p, p).reshape(-1)
            keep = a != b
            r.append(a[keep]), c.append(b[keep])
            w.append(torch.full((int(keep.sum()),), round(2.0 ** 32 / (p - 1)) / 2.0 ** 32, dtype=F64, device=DEV))
        k, j = _expand(stars.numel(), deg[stars])
        a, z, p = pin[ptr[stars][k] + j], self.star0 + k, deg[stars][k].double()
        q = torch.round(2.0 ** 32 * p / (p - 1)) / 2.0 ** 32
        self.star_row, self.star_pin = k, a
        r, c, w = torch.cat(r + [a, z]), torch.cat(c + [z, a]), torch.cat(w + [q, q])
        key, inv = torch.unique(r * self.total + c, return_inverse=True)
        self.w = torch.zeros(key.numel(), dtype=F64, device=DEV).index_add_(0, inv, w)
        self.r, self.c = key // self.total, key % self.total
        self.qdeg, cnt = self.sum(self.r, self.w), torch.bincount(self.r, minlength=self.total)
        self.base = self.qdeg / cnt.clamp(min=1)

    def sum(self, rows, v):
        return torch.zeros((self.total,) + v.shape[1:], dtype=F64, device=DEV).index_add_(0, rows, v)

    def set_hints(self, pos, prune):
        """The area hints of the float32 placement pos [n, 2], both directions, after the netlist's entries."""
        nl, nb = self.nl, self.bins
        xl, yl, xh, yh = np.asarray(nl["die"], np.float32)
        bw, bh = (float(xh) - float(xl)) / nb, (float(yh) - float(yl)) / nb
        cell = torch.nonzero(~self.fixed & ~self.macro).ravel()
        # (a whole tensor of divisors: a scalar one may become a product with its reciprocal)
        spot = lambda v, lo, hi: torch.floor((v - float(lo)) / torch.full_like(v, float((hi - lo) / np.float32(nb)))
                                             ).clamp(0, nb - 1).long()
        bx, by = spot(pos[cell, 0], xl, xh), spot(pos[cell, 1], yl, yh)
        size, p64 = nl["node_size"].double(), pos.double()
        area = torch.zeros(nb * nb, dtype=F64, device=DEV).index_add_(0, by * nb + bx, size[cell].prod(1))
        m = torch.nonzero(self.macro).ravel()
        edge = torch.arange(nb + 1, device=DEV, dtype=F64)

        def overlap(c, s, lo, step):
            e = float(lo) + edge * step
            lo_, hi_ = torch.maximum((c - s / 2)[:, None], e[:-1]), torch.minimum((c + s / 2)[:, None], e[1:])
            return (hi_ - lo_).clamp(min=0)

        area += (overlap(p64[m, 1], size[m, 1], yl, bh).T @ overlap(p64[m, 0], size[m, 0], xl, bw)).ravel()
        phi = 2 / (1 + torch.exp(-4.0 * (area / (bw * bh) - 1.0))) - 1
        keep = self.qdeg[cell] > 0
        cell, bx, by = cell[keep], bx[keep], by[keep]
        hw = max(1, int(np.floor(np.float32(0.1) * np.float32(nb)))) // 2
        r, c, w = [], [], []
        for dy in range(-hw, hw + 1):
            for dx in range(-hw, hw + 1):
                tx, ty = bx + dx, by + dy
                ok = (tx >= 0) & (tx < nb) & (ty >= 0) & (ty < nb)
                i, tx, ty = cell[ok], tx[ok], ty[ok]
                rx = (p64[i, 0] - (float(xl) + (tx.double() + 0.5) * bw)).abs() / (bw / 2)
                ry = (p64[i, 1] - (float(yl) + (ty.double() + 0.5) * bh)).abs() / (bh / 2)
                e, b = torch.exp(-torch.maximum(rx, ry)), ty * nb + tx
                ok = e * phi[b].abs() >= prune if prune > 0 else slice(None)
                i, e, b = i[ok], e[ok], b[ok]
                r.append(i), c.append(self.bv0 + b), w.append(-e * phi[b] * self.base[i])
        i, k = self.inside(pos, cell, size)
        rx = (p64[i] - p64[self.macros[k]]).abs() / (size[self.macros[k]] / 2)
        r.append(i), c.append(self.mv0 + k), w.append(-torch.exp(-rx.amax(1)) * self.base[i])
        r, c, w = torch.cat(r), torch.cat(c), torch.cat(w)
        self.hr, self.hc, self.hw = torch.cat([r, c]), torch.cat([c, r]), torch.cat([w, w])

    def inside(self, pos, cell, size, tiles=256):
        """(cell, macro) pairs with the cell's centre in the macro's footprint, tested in float32."""
        die = self.nl["die"][2] * 2
        at = lambda v: ((v.double() / die + 0.5) * tiles).long().clamp(0, tiles - 1)
        mp, mh = pos[self.macros], size[self.macros].float() * 0.5
        a, b = at(mp - mh * 1.001 - 1e-3), at(mp + mh * 1.001 + 1e-3)
        span = b - a + 1
        k, j = _expand(self.macros.numel(), span.prod(1))
        t = (a[k, 1] + j // span[k, 0]) * tiles + a[k, 0] + j % span[k, 0]
        t, o = torch.sort(t, stable=True)
        k = k[o]
        ct = at(pos[cell, 1]) * tiles + at(pos[cell, 0])
        lo, hi = torch.searchsorted(t, ct), torch.searchsorted(t, ct + 1)
        i, j = _expand(cell.numel(), hi - lo)
        i, k = cell[i], k[lo[i] + j]
        ok = ((pos[i] - mp[k]).abs() <= mh[k]).all(1)
        return i[ok], k[ok]

    def signal(self, G):
        """Instance values extended to the added nodes."""
        X = torch.zeros(self.total, G.shape[1], dtype=F64, device=DEV)
        xy = torch.arange(G.shape[1], device=DEV) % 2
        X[:self.n] = G
        X[self.n:self.star0] = X[self.mp_owner] + self.nl["pin_off"].double()[self.mp][:, xy]
        if self.mv0 > self.star0:
            X[self.star0:self.mv0] = (self.sum(self.star0 + self.star_row, X[self.star_pin])[self.star0:self.mv0]
                                      / torch.bincount(self.star_row)[:, None])
        X[self.mv0:self.bv0] = X[self.macros]
        if self.total > self.bv0:
            b = torch.arange(self.bins ** 2, device=DEV)
            lo, w = float(np.float32(self.nl["die"][0])), 2 * float(np.float32(self.nl["die"][2])) / self.bins
            X[self.bv0:, 0::2] = (lo + ((b % self.bins).double() + 0.5) * w)[:, None]
            X[self.bv0:, 1::2] = (lo + ((b // self.bins).double() + 0.5) * w)[:, None]
        return X

    def operator(self, sigma=0.0, lam=None):
        """y -> T y with T = I - L / lambda, and the absolute degrees."""
        r, c, w = self.r, self.c, self.w
        if hasattr(self, "hr"):
            r, c, w = torch.cat([r, self.hr]), torch.cat([c, self.hc]), torch.cat([w, self.hw])
        d = self.sum(r, w.abs()) + sigma
        s = torch.where(d > 0, d.clamp(min=1e-300).rsqrt(), 0.0)
        v = s[r] * w * s[c]
        diag = (d > 0).double() - sigma * s * s
        lam = float((diag.abs() + self.sum(r, v.abs())).max()) if lam is None else lam

        def T(y):
            z = torch.zeros_like(y)
            for a in range(0, r.numel(), 1 << 24):
                k = slice(a, a + (1 << 24))
                z.index_add_(0, r[k], v[k][:, None] * y[c[k]])
            return y - (diag[:, None] * y - z) / lam

        return T, d


def _f32(values):
    return [float(np.float32(v)) for v in values]


def _bank64(g, G, ks, alphas, chain=None):
    T, _ = chain or g.operator()
    Y, out = g.signal(G), 0
    for j in range(max(ks) + 1):
        Y = T(Y) if j else Y
        out = out + sum(a for k, a in zip(ks, _f32(alphas)) if k == j) * Y[:g.n]
    out[g.fixed] = G[g.fixed]
    return out


def _mlp64(P, F):
    """Activations of the network with its bfloat16 rounding points, otherwise in 64 bits."""
    q = lambda t: t.float().bfloat16().double()
    W1, b1, W2, b2, w3, b3 = torch.split(P.double(), [512, 64, 4096, 64, 64, 1])
    x, W1, W2, w3 = q(F), q(W1).view(64, 8), q(W2).view(64, 64), q(w3)
    z1 = x @ W1.T + b1
    a1 = q(z1.clamp(min=0))
    z2 = a1 @ W2.T + b2
    a2 = q(z2.clamp(min=0))
    return x, z1, a1, z2, a2, W2, w3, a2 @ w3 + b3


def _learned64(g, G):
    with open(MODEL) as f:
        model = json.load(f)
    params = torch.tensor(model["params"], dtype=torch.float32, device=DEV)
    T, d = g.operator()
    h = [g.signal(G)]
    for _ in range(3):
        h.append(T(h[-1]))
    h, d = [y[:g.n] for y in h], d[:g.n, None]
    mov = ~g.fixed
    hsum = g.sum(g.hr, g.hw)[:g.n, None]
    mean, dev = h[3][mov].mean(0), h[3][mov].std(0, correction=0)
    rms = (h[0] - h[3])[mov].square().mean(0).sqrt()
    full = lambda t: t.expand(g.n, G.shape[1])
    F = torch.stack([(h[0] - h[3]) / rms, (h[1] - h[3]) / rms, (h[2] - h[3]) / rms, (h[3] - mean) / dev,
                     full(torch.log1p(d)), full(torch.where(d > 0, hsum / d.clamp(min=1e-300), 0.0)),
                     full(torch.log(dev / rms)), full(torch.zeros_like(d))], 2)
    o = torch.cat([_mlp64(params, f)[-1] for f in torch.split(F.view(-1, 8), 1 << 20)])
    y = sum(b * v for b, v in zip(_f32(model["beta"]), h)) + rms * o.view(g.n, -1)
    y[g.fixed] = G[g.fixed]
    return y


def _train64(case, seed):
    F, R, P, m, v = _training(case, seed)
    grad = torch.zeros(P.numel(), dtype=F64, device=DEV)
    for f, t in zip(torch.split(F, 1 << 19), torch.split(R, 1 << 19)):
        x, z1, a1, z2, a2, W2, w3, o = _mlp64(P, f)
        do = 2 * (o - t.double()) / F.shape[0]
        dz2 = do[:, None] * w3 * (z2 > 0)
        dz1 = (dz2 @ W2) * (z1 > 0)
        grad += torch.cat([(dz1.T @ x).ravel(), dz1.sum(0), (dz2.T @ a1).ravel(), dz2.sum(0), a2.T @ do,
                           do.sum()[None]])
    b1, b2, eps, lr = _f32([0.9, 0.999, 1e-8, 1e-3])
    m, v = b1 * m.double() + (1 - b1) * grad, b2 * v.double() + (1 - b2) * grad ** 2
    step = lr * (m / (1 - b1 ** 500)) / ((v / (1 - b2 ** 500)).sqrt() + eps)
    return dict(grad=grad, params=P.double() - step, m=m, v=v)


def _nets64(nl):
    """Pins of the non-empty nets: (net of every pin, number of nets, node, offset)."""
    deg = nl["net_ptr"][1:] - nl["net_ptr"][:-1]
    deg = deg[deg > 0]
    return torch.repeat_interleave(torch.arange(deg.numel(), device=DEV), deg), deg.numel(), nl["pin_node"], \
        nl["pin_off"].double()


def _extreme(x, net, n, how):
    return torch.zeros(n, dtype=F64, device=DEV).scatter_reduce_(0, net, x, how, include_self=False)


def _hpwl64(nl, G):
    net, n, node, off = _nets64(nl)
    out = torch.zeros(G.shape[1] // 2, dtype=F64, device=DEV)
    for c in range(G.shape[1]):
        x = G[node, c] + off[:, c % 2]
        out[c // 2] += (_extreme(x, net, n, "amax") - _extreme(x, net, n, "amin")).sum()
    return out


def _wa64(nl, G, gamma):
    net, n, node, off = _nets64(nl)
    total, grad = torch.zeros(G.shape[1] // 2, dtype=F64, device=DEV), torch.zeros_like(G)
    for c in range(G.shape[1]):
        x = G[node, c] + off[:, c % 2]
        for sign, how in ((1.0, "amax"), (-1.0, "amin")):
            e = torch.exp(sign * (x - _extreme(x, net, n, how)[net]) / gamma)
            add = lambda t: torch.zeros(n, dtype=F64, device=DEV).index_add_(0, net, t)
            s = add(e)
            mean = add(e * x) / s
            total[c // 2] += sign * mean.sum()
            grad[:, c].index_add_(0, node, sign * e / s[net] * (1 + sign * (x - mean[net]) / gamma))
    return total, grad


def _charge64(case, nl):
    """Macro charge per bin of the models whose bin integral is a product of one-dimensional ones,
    with the binding's default schedule constants (300 iterations)."""
    a, nb = case["t"] / 300, case["bins"]
    factor, r0, r1, beta0, beta1, a0, a1 = _f32([0.005, 1e-3, 0.9, 0.1, 1.0, 0.2, 0.8])
    if case["model"] == A.CHARGE_EXP:
        param = -factor * 300 * math.log(1 - a)
    else:
        z = min(1.0, max(0.0, (a - a0) / (a1 - a0)))
        mix = 3 * z * z - 2 * z ** 3
        param = ((math.sqrt(2 * math.log(2)) / (beta0 + (beta1 - beta0) * a)) ** (1 - mix)
                 * math.sqrt(-2 * ((1 - a) * math.log(r0) + a * math.log(r1))) ** mix)
    m = torch.nonzero((nl["node_flags"].long() & 2) > 0).ravel()
    pos, size, lo = nl["g0"].double()[m], nl["node_size"].double()[m], float(np.float32(nl["die"][0]))
    edge = lo + torch.arange(nb + 1, device=DEV, dtype=F64) * (-2 * lo / nb)
    node, wt = (torch.tensor(t, device=DEV) for t in np.polynomial.legendre.leggauss(48))

    def axis(k):
        L = size[:, k:k + 1]
        x = torch.minimum(torch.maximum(edge - pos[:, k:k + 1], -L / 2), L / 2)
        if case["model"] == A.CHARGE_GAUSSIAN:
            q = math.sqrt(2) * param / L
            return (math.sqrt(math.pi) / (2 * q) * torch.diff(torch.erf(q * x)))
        total = torch.zeros(x.shape[0], nb, dtype=F64, device=DEV)
        for part in range(8):       # each bin's part in eight pieces, split at the macro's centre
            for y in (x.clamp(max=0), x.clamp(min=0)):
                a, b = y[:, :-1], y[:, 1:]
                u, h = a + (b - a) * part / 8, (b - a) / 16
                t = torch.tan(math.pi * (u + h)[..., None].add(h[..., None] * node) / L[..., None])
                total += (torch.exp(-t * t / (2 * param * param)) * wt).sum(-1) * h
        return total

    scale = 1.0
    if case["model"] == A.CHARGE_GAUSSIAN:
        scale = 2 * param ** 2 / (math.pi * math.erf(param / math.sqrt(2)) ** 2)
    return scale * (axis(1).T @ axis(0)).ravel()


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _train64(case, seed)
    if kind == "batch":
        out = []
        for nl in _members(case, seed):
            g = _Graph64(nl, bins=_member_bins(nl["n_inst"]))
            g.set_hints(nl["g0"][:, :2], 0.0)
            out.append(_bank64(g, nl["g0"].double(), *BANK))
        return torch.cat(out)
    nl = _one(case, seed)
    G = nl["g0"].double()
    if kind == "hpwl":
        return _hpwl64(nl, G)
    if kind == "wa":
        return _wa64(nl, G, 4.0)
    if kind == "charge":
        return _charge64(case, nl) if case["model"] in (A.CHARGE_GAUSSIAN, A.CHARGE_EXP) else None
    if kind == "gift":
        g = _Graph64(nl, expand=False, hints=False)
        out = 0
        for sigma in sorted(set(GIFT[1])):
            sel = [(k, a) for k, s, a in zip(*GIFT) if s == sigma]
            out = out + _bank64(g, G, [k for k, _ in sel], [a for _, a in sel], g.operator(sigma, 1.0))
        out[g.fixed] = G[g.fixed]
        return out
    g = _Graph64(nl, bins=case["bins"])
    if kind == "refine":
        for _ in range(case["rounds"]):
            g.set_hints(G[:, :2].float(), case["prune"] and float(np.float32(case["prune"])))
            G = 0.5 * G + 0.5 * _bank64(g, G, *_bands(case))
        return G
    g.set_hints(nl["g0"][:, :2], 0.0)
    return _learned64(g, G) if kind == "learned" else _bank64(g, G, *_bands(case))
