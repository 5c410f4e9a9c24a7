"""What the speed of this library is measured on: calls that a program with a sparse network in hand makes.

A case is a network and a batch.  Three kinds of network:

  challenge  32 connections per neuron, every weight 1/16, one negative bias, binary inputs: the networks of the
             Sparse DNN Challenge.  Columns are uniform over the row, uniform inside a 4096-wide window per 4096
             neurons ("window"), or strided ("strided", the building block of the RadiX-Net topologies).  Half of
             the rows are sparse and die within a few layers, the other half stay alive and grow: the partly dead
             batches that the pruning between two layers is for.
  trained    32 connections per neuron, weights of their own of both signs, real-valued inputs, a few blank rows.
  general    the same, with kmin .. kmax connections per neuron, through the CSR entry point.

and three ways in: infer (inputs resident), static (the library's own work memory, for callers that allocate
nothing) and host (inputs in pinned host memory, in serial batches).

Row densities keep a distance from the edge between dying and surviving, so that which rows survive depends on no
rounding; the networks are shallow enough (or do not saturate) where values are to be told apart from the clip.
"""
import math

import torch

import paper_2007_14152_amd as sp

DEV = "cuda:0"
CLIP = 32.0

# Connections per neuron of a case, the most; a trained or challenge network has exactly 32.
NNZ = 32


def listed():
    c = dict(kind="challenge", pattern="uniform", entry="infer", kmin=NNZ, kmax=NNZ, per=0)
    t = dict(c, kind="trained", bias=-0.02)
    g = dict(t, kind="general")
    return [
        # one input at a time through a small trained network: a serving loop, latency and launches only
        dict(t, name="serve_one_row", N=1024, L=12, batch=1, entry="static"),
        # the benchmark's smallest configuration: 1000 inputs of 1024 features, 120 layers
        dict(c, name="small_net_1000", N=1024, L=120, batch=1000, bias=-0.30),
        # the challenge's smallest network on its whole input set
        dict(c, name="small_net_60000", N=1024, L=120, batch=60000, bias=-0.30),
        # its second size, 60 000 inputs; 24 of the 480 layers
        dict(c, name="mid_net_60000", N=4096, L=24, batch=60000, bias=-0.35),
        # a RadiX-Net-like network on a modest batch: many short layers one behind the other
        dict(c, name="radix_16384_2000", N=16384, L=48, batch=2000, bias=-0.40, pattern="strided"),
        # the third size, columns anywhere in the row, a third of the inputs
        dict(c, name="wide_net_16384", N=16384, L=6, batch=20000, bias=-0.40),
        # the largest size in its locality variant: bound by memory, the benchmark's headline configuration
        dict(c, name="big_net_65536", N=65536, L=6, batch=24000, bias=-0.45, pattern="window"),
        # inputs that stay in host memory and go through the device in serial batches
        dict(c, name="host_inputs_4096", N=4096, L=24, batch=6000, bias=-0.35, entry="host", per=1500),
        # a trained, pruned network whose layers fit one LDS stage; an odd batch
        dict(t, name="trained_4096", N=4096, L=12, batch=10007),
        # the same with rows four stages wide
        dict(t, name="trained_16384", N=16384, L=6, batch=8000),
        # neurons of uneven length, most of them longer than 32 connections
        dict(g, name="general_4096", N=4096, L=6, batch=10000, kmin=16, kmax=64),
        # a small ragged network: odd sizes, some neurons without a connection, some longer than 32
        dict(g, name="ragged_1500", N=1500, L=12, batch=777, kmin=0, kmax=40),
    ]


def draw(rng):
    """One more case of the ranges above."""
    def log(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    kind = rng.choice(["challenge", "challenge", "challenge", "trained", "trained", "general"])
    c = dict(kind=kind, pattern="uniform", entry="infer", kmin=NNZ, kmax=NNZ, per=0)
    if kind == "challenge":
        c["pattern"] = rng.choice(["uniform", "uniform", "window", "strided"])
        if c["pattern"] == "uniform":  # half of them the challenge's own sizes, half any size
            c["N"] = rng.choice([1024, 4096, 16384]) if rng.random() < 0.5 else 4 * round(log(256, 4096))
        else:
            c["N"] = rng.choice([16384, 32768, 65536] if c["pattern"] == "window" else [4096, 16384, 65536])
        c["bias"] = -rng.choice([0.30, 0.35, 0.40, 0.45])
        c["entry"] = rng.choice(["infer", "infer", "infer", "host"])
    else:
        c["N"] = rng.choice([1024, 4096, 16384]) if rng.random() < 0.4 else 4 * round(log(125, 4096 if kind == "trained" else 2048))
        c["bias"] = -0.02
        c["entry"] = "static" if c["N"] <= 1024 and rng.random() < 0.5 else "infer"
        if kind == "general":
            c["kmin"], c["kmax"] = rng.choice([(0, 32), (8, 32), (0, 40), (16, 64), (33, 64), (0, 100)])
    c["L"] = rng.randint(4, 12 if kind != "challenge" else 120 if c["N"] <= 1024 else 48)
    # rows so that no drawn case does more than the largest listed one of its kind
    most = {"challenge": 24000 * 65536 * 6, "trained": 10007 * 4096 * 12, "general": 10000 * 4096 * 4}[kind]
    if c["entry"] == "host":
        most //= 8
    if c["entry"] == "static":  # its work memory is fixed
        most = min(most, c["N"] * c["L"] * 4000)
    least = 16 if kind == "challenge" else 1  # some rows of a challenge batch die: its survivors are the answer
    c["batch"] = max(least, round(log(least, min(60000, most // (c["N"] * c["L"])))))
    if c["entry"] == "host":
        c["per"] = -(-c["batch"] // rng.choice([1, 3, 4, 7]))
    return c


# ---------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------
def _rng(seed, salt):
    return torch.Generator(device=DEV).manual_seed((int(seed) * 1000003 + salt) & ((1 << 62) - 1))


def _columns(g, N, width, base):
    """32 distinct columns per neuron, uniform over the `width` columns from base on, ascending: int64 [N, 32]."""
    c = torch.randint(0, width, (N, NNZ), generator=g, device=DEV).sort(1).values
    while True:
        bad = (c[:, 1:] == c[:, :-1]).any(1).nonzero().flatten()
        if not len(bad):
            return c + base[:, None]
        c[bad] = torch.randint(0, width, (len(bad), NNZ), generator=g, device=DEV).sort(1).values


def _layer(case, seed, l):
    """Layer l: columns int64 [N, K], weights float32 [N, K], connections per neuron int64 [N] (the first of the K)."""
    N, K = case["N"], case["kmax"]
    g = _rng(seed, 17 + l)
    j = torch.arange(N, device=DEV)
    full = torch.full((N,), NNZ, dtype=torch.int64, device=DEV)
    if case["kind"] == "challenge":
        if case["pattern"] == "strided":  # neuron j reads columns j, j + S, ...; S grows through N / 32 and starts again
            stride = [s for s in (1, 32, 1024, 32768) if s * NNZ < N] + [N // NNZ]
            cols = ((j[:, None] + stride[l % len(stride)] * torch.arange(NNZ, device=DEV)) % N).sort(1).values
        elif case["pattern"] == "window":  # the 4096-wide windows of the row, in another order in every layer
            order = torch.randperm(N // 4096, generator=g, device=DEV)
            cols = _columns(g, N, 4096, order[j // 4096] * 4096)
        else:
            cols = _columns(g, N, N, 0 * j)
        return cols, torch.full((N, NNZ), 0.0625, device=DEV), full
    draws = max(1, -(-K // NNZ))
    cols = torch.cat([_columns(g, N, N, 0 * j) for _ in range(draws)], 1)[:, :K].contiguous()
    deg = full if case["kind"] == "trained" else torch.randint(case["kmin"], K + 1, (N,), generator=g, device=DEV)
    # both signs, variance 2 over the neuron's length: the scale of the activations is kept from layer to layer
    w = torch.randn((N, K), generator=g, device=DEV) * (2.0 / deg.clamp(min=1)).sqrt()[:, None]
    return cols, w, deg


def _inputs(case, seed):
    """float32 [batch, N].  challenge: zeros and ones, half of the rows dense enough to live; others: non-negative
    activations, every second one zero, and one row in eight blank."""
    N, B = case["N"], case["batch"]
    g = _rng(seed, 1)
    out = torch.empty((B, N), dtype=torch.float32, device=DEV)
    u = torch.rand((B,), generator=g, device=DEV)
    order = torch.rand((B,), generator=g, device=DEV).argsort()
    first = torch.zeros((B,), dtype=torch.bool, device=DEV)
    if case["kind"] == "challenge":
        first[order[: (B + 1) // 2]] = True
        density = torch.where(first, 0.55 + 0.15 * u, 0.03 + 0.07 * u)
    else:
        first[order[: B // 8]] = True
        density = torch.where(first, 0.0 * u, 0.4 + 0.2 * u)
    step = max(1, (1 << 26) // N)
    for r in range(0, B, step):
        x = out[r:r + step].uniform_(generator=g)
        one = x < density[r:r + step, None]
        if case["kind"] == "challenge":
            x.copy_(one)
        else:  # the surviving draws, spread over (0, 1]
            x.div_(density[r:r + step, None].clamp(min=0.1)).mul_(one)
    return out


def prepare(case, seed):
    """The network as a handle of the library, and the batch."""
    N, L = case["N"], case["L"]
    bias = torch.full((N,), case["bias"], dtype=torch.float32, device=DEV)
    layers = [_layer(case, seed, l) for l in range(L)]
    if case["kind"] == "general":
        ptr, idx, val = [], [], []
        for cols, w, deg in layers:
            keep = torch.arange(cols.shape[1], device=DEV)[None, :] < deg[:, None]
            ptr.append(torch.cat([deg.new_zeros(1), deg.cumsum(0)]).to(torch.int32))
            idx.append(cols[keep].to(torch.int32))
            val.append(w[keep])
        model = sp.Model.from_csr(ptr, idx, val, bias, device=DEV)
    else:
        model = sp.Model([c.to(torch.int32) for c, _, _ in layers], [w for _, w, _ in layers], bias, device=DEV)
    del layers
    y0 = _inputs(case, seed)
    if case["entry"] == "host":
        y0 = torch.empty(y0.shape, dtype=torch.float32, pin_memory=True).copy_(y0)
    return dict(model=model, y0=y0, entry=case["entry"], per=case["per"])


def run(state):
    """(rows that survive, their numbers, their outputs)"""
    m = state["model"]
    if state["entry"] == "static":
        return m.infer_static(state["y0"])
    if state["entry"] == "host":
        return m.infer_batched(state["y0"], state["per"])
    return m.infer(state["y0"])


# ---------------------------------------------------------------------------
# what a pass cannot do without, and what it has to give
# ---------------------------------------------------------------------------
def _alive(case):
    """Rows that go through the whole network; the others die in its first layers."""
    return (case["batch"] + 1) // 2 if case["kind"] == "challenge" else case["batch"] - case["batch"] // 8


def work(case):
    """The inputs and the connections read once, the surviving rows written once; a multiply and an add for every
    connection of every neuron of the surviving rows, and of all rows in the first layer.  Feature maps between
    layers are not counted: rows are independent, so a batch can go through them in pieces that stay on the chip."""
    N, L, B, live = case["N"], case["L"], case["batch"], _alive(case)
    nnz = N * (case["kmin"] + case["kmax"]) / 2
    weight = 2 if case["kind"] == "challenge" else 6  # 16-bit column, 32-bit weight where there is more than one
    return dict(bytes=4.0 * N * B + 4.0 * N * live + weight * nnz * L + 4.0 * live,
                flops=2.0 * nnz * (B + live * (L - 1)))


def tolerance(case):
    """32-bit sums of at most a hundred terms per layer, in any order, carried through the layers: about four times
    what the library was seen to be off the 64-bit result (up to 6.5e-7)."""
    return dict(rel=2.5e-6, max=4e-5)


def exact(case, seed):
    """The layers one by one in 64 bits, a few thousand rows at a time, rows without a positive output dropped."""
    N, L = case["N"], case["L"]
    b = torch.full((N, 1), case["bias"], dtype=torch.float32, device=DEV).double()
    y0 = _inputs(case, seed)
    rows, outs = [], []
    layers = [_layer(case, seed, l) for l in range(L)]
    step = max(1, (1 << 28) // N)
    for r in range(0, case["batch"], step):
        y = y0[r:r + step].double().t().contiguous()  # a column of the batch side by side
        ids = torch.arange(r, r + y.shape[1], device=DEV)
        for cols, w, deg in layers:
            if not y.shape[1]:
                break
            s = b.expand(-1, y.shape[1]).clone()
            for k in range(cols.shape[1]):
                wk = torch.where(deg > k, w[:, k], torch.zeros_like(w[:, k])).double()
                s.addcmul_(y.index_select(0, cols[:, k]), wk[:, None])
            y = s.clamp_(0.0, CLIP)
            live = (y > 0).any(0)
            if not bool(live.all()):
                y, ids = y[:, live], ids[live]
        rows.append(ids)
        outs.append(y.t().contiguous())
    rows = torch.cat(rows)
    return int(len(rows)), rows.to(torch.int32), torch.cat(outs)
