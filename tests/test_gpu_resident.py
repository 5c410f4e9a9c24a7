"""Networks of at most 4096 neurons: the rows stay in LDS from layer to layer (resident_kernel).  One case per shape the
kernel takes -- one to four output blocks, ragged last blocks, one weight or many, a share of one quad of rows, of one
pass, of several passes, batches that are compacted between launches -- with rows that die on the way, so that passes
lose planes and rows move together.  Checked against the oracle: survivors, values, and rows alive on entry to every layer."""
import numpy as np
import pytest

import oracle
import synth
from parity_util import check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,batch,L,uniform", [
    (32, 9000, 5, False),     # one group of 64 lanes, half of them without a neuron
    (100, 36000, 4, True),    # small rows, several workgroups per CU; more rows than one launch takes
    (1000, 4100, 6, False),   # last group ragged; two launches' worth of passes in one launch
    (1024, 1021, 7, True),    # one quad of rows per workgroup, a wave per group of 64 neurons
    (1024, 9001, 7, False),   # two groups per wave, several passes per share
    (1028, 3000, 4, True),    # a second block of four neurons
    (1500, 1100, 4, False),
    (2048, 5000, 4, True),    # four planes
    (2052, 1500, 3, False),   # three blocks: two planes
    (3072, 2500, 3, True),
    (4092, 700, 3, False),
    (4096, 2100, 4, True),    # eight rows per pass, two launches
    (4096, 2600, 11, False),  # ... and three
])
def test_rows_stay_on_chip_through_the_layers(N, batch, L, uniform):
    import torch
    import paper_2007_14152_amd as sp
    rng = np.random.default_rng(N + batch + L)
    idx = [np.sort(rng.integers(0, N, size=(N, 32)), axis=1).astype(np.int32) for _ in range(L)]
    val = [np.full((N, 32), 0.0625, np.float32) if uniform else rng.uniform(0.02, 0.11, size=(N, 32)).astype(np.float32)
           for _ in range(L)]
    bias = -rng.uniform(0.0, 0.5, size=N).astype(np.float32)
    Y0 = synth.gen_y0(batch, N, 23, density="mixed")
    Y0[3] = 0
    sample = batch if batch <= 3000 else 1500   # the oracle on the first rows and the last
    ids = np.arange(batch) if sample == batch else np.r_[0:sample // 2, batch - sample // 2:batch]
    ref = oracle.infer(idx, val, bias, Y0[ids])
    m = sp.Model(idx, val, bias)
    m.set_profiling(True)
    n, rows, Y = m.infer(torch.from_numpy(Y0).to("cuda:0"))
    run, rows_in, ms = m.profile()
    m.close()
    rows, Y = rows.cpu().numpy(), Y.cpu().numpy()
    assert n == len(rows) and 0 < n < batch and np.all(np.diff(rows) > 0)
    mine = np.isin(rows, ids)
    common, _ = check_against_oracle(ref, int(mine.sum()), rows[mine], Y[mine], row_ids=ids, what="N=%d" % N)
    assert common > 0
    assert run == L and int(rows_in[0]) == batch and np.all(np.diff(rows_in[:L]) <= 0) and int(rows_in[L - 1]) >= n
    if sample == batch and not (ref.fragile_layer >= 0).any():
        assert [int(x) for x in rows_in[:L]] == [int(x) for x in ref.active_per_layer[:L]]
    # the same call without the measurement: same bits
    m = sp.Model(idx, val, bias)
    n2, rows2, Y2 = m.infer(torch.from_numpy(Y0).to("cuda:0"))
    m.close()
    assert n2 == n and np.array_equal(rows2.cpu().numpy(), rows) and np.array_equal(Y2.cpu().numpy(), Y)


@pytest.mark.parametrize("N,batch,L,kmin,kmax", [
    (64, 3000, 3, 0, 300),      # ten parts of 32 connections per neuron, one group of lanes
    (100, 1100, 4, 0, 9),       # two chunks at most; a ragged last group
    (1024, 4500, 3, 0, 100),    # several passes per share, uneven neurons
    (1500, 700, 4, 0, 40),
    (1028, 2500, 3, 33, 64),    # two parts everywhere
    (2052, 1300, 3, 1, 32),     # one part, three blocks
    (4096, 2300, 4, 16, 64),    # two launches
])
def test_neurons_of_any_length_stay_on_chip(N, batch, L, kmin, kmax):
    """The same for general layers: neurons sorted by length, as many chunks of connections as a group's longest needs."""
    import torch
    import paper_2007_14152_amd as sp
    rng = np.random.default_rng(N + kmax)
    ptr, idx, val = [], [], []
    for l in range(L):
        deg = rng.integers(kmin, kmax + 1, size=N)
        if kmin == 0:
            deg[: 70] = 0                    # a whole group of lanes without a connection, where there are that many
        p = np.zeros(N + 1, dtype=np.int32)
        np.cumsum(deg, out=p[1:])
        ptr.append(p)
        idx.append(rng.integers(0, N, size=int(p[N])).astype(np.int32))
        val.append((rng.uniform(0.5, 1.5, size=int(p[N])) * np.repeat(2.0 / np.maximum(deg, 1), deg)).astype(np.float32))
    bias = -rng.uniform(0.0, 0.3, size=N).astype(np.float32)
    Y0 = synth.gen_y0(batch, N, 29, density="mixed")
    Y0[1] = 0
    ref = oracle.infer(idx, val, bias, Y0, ptr=ptr)
    m = sp.Model.from_csr(ptr, idx, val, bias)
    n, rows, Y = m.infer(torch.from_numpy(Y0).to("cuda:0"))
    m.close()
    check_against_oracle(ref, n, rows.cpu().numpy(), Y.cpu().numpy(), what="general N=%d" % N)
    assert n == 0 or n < batch


@pytest.mark.parametrize("N,batch,L,general,order", [
    (100, 70000, 12, False, "mixed"),    # one group of lanes; several workgroups per CU
    (1024, 9001, 12, False, "mixed"),    # one launch, passes stopped at the second layer
    (1024, 41003, 16, False, "sorted"),  # sixteen rows per pass, two launches
    (1028, 22001, 12, True, "mixed"),    # neurons by length
    (2048, 20002, 12, False, "sorted"),
    (3072, 9003, 12, False, "mixed"),    # eight rows per pass
    (4096, 13001, 18, False, "mixed"),
    (4096, 13001, 18, False, "sorted"),
    (4096, 11001, 12, True, "late"),
    (4096, 9001, 30, False, "late"),
    (4096, 17001, 12, False, "mixed"),   # the first two layers one by one, two neurons per lane
    (1500, 49300, 7, False, "sorted"),   # ... one neuron per lane
])
def test_rows_that_die_late(N, batch, L, general, order):
    """Passes that lose half their rows on the way are stopped and merged, more than once.  Row r holds the integer v_r
    in every column, a layer turns v into v - 1, exactly; most die in layers 3, 5, 8 and 9, some in every layer.  Sorted:
    the first rows of the batch die first."""
    import torch
    import paper_2007_14152_amd as sp
    dev = "cuda:0"
    rng = np.random.default_rng(N + L)
    top = L + 2   # the first layer's outputs stay below the clip
    u = rng.uniform(size=batch)
    if order == "late":
        v = np.where(u < 0.6, L - 6, np.where(u < 0.9, L - 3, top))
    else:
        v = np.select([u < 0.55, u < 0.75, u < 0.9, u < 0.93], [3, 5, 8, 9], top)
    odd = rng.uniform(size=batch) < 0.05
    v[odd] = rng.integers(1, top + 1, size=int(odd.sum()))
    if order == "sorted":
        v.sort()
    ptr, idx, val = [], [], []
    for l in range(L):
        deg = rng.choice([8, 16, 64], size=N) if general else np.full(N, 32)
        p = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
        ptr.append(p)
        idx.append(rng.integers(0, N, size=int(p[N])).astype(np.int32))
        val.append(np.repeat(1.0 / deg, deg).astype(np.float32))
    bias = np.full(N, -1.0, np.float32)
    if general:
        m = sp.Model.from_csr(ptr, idx, val, bias)
    else:
        m = sp.Model([a.reshape(N, 32) for a in idx], [a.reshape(N, 32) for a in val], bias)
    y0 = torch.from_numpy(v.astype(np.float32)).to(dev)[:, None].expand(batch, N).contiguous()
    alive = np.nonzero(v > L)[0]
    m.set_profiling(True)
    for _ in range(2):
        n, rows, Y = m.infer(y0)
        assert n == len(alive) and np.array_equal(rows.cpu().numpy(), alive)
        assert bool((Y == torch.from_numpy((v[alive] - L).astype(np.float32)).to(dev)[:, None]).all())
        run, rows_in, _ = m.profile()
        want = [int((v > l).sum()) for l in range(L)]
        assert [int(x) for x in rows_in[:run]] == want[:run] and not any(want[run:])
    assert m.launches()[1] > 0
    m.close()


@pytest.mark.parametrize("N,batch,L,kind", [
    (100, 60000, 9, "weights"), (1024, 20001, 14, "uniform"), (1024, 41003, 12, "weights"), (1028, 21001, 10, "general"),
    (2048, 20002, 12, "weights"), (3072, 9003, 11, "uniform"), (4096, 13001, 18, "weights"), (4096, 13001, 12, "uniform"),
    (4092, 9001, 10, "general"), (4096, 17001, 9, "uniform"),
])
def test_rows_that_die_late_keep_their_columns(N, batch, L, kind):
    """Rows that wait while their pass is stopped go to memory in one layer's layout and come back in another's.  Values
    differ from column to column here, rows die in every layer, and each row must come out with the bits that it has in
    a batch of a thousand, whose passes never stop."""
    import torch
    import paper_2007_14152_amd as sp
    dev = "cuda:0"
    rng = np.random.default_rng(N + L)
    ptr, idx, val = [], [], []
    for l in range(L):
        deg = rng.integers(4, 61, size=N) if kind == "general" else np.full(N, 32)
        p = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
        w = np.full(p[N], 1.0) if kind == "uniform" else rng.uniform(0.5, 1.5, size=p[N])
        ptr.append(p)
        idx.append(rng.integers(0, N, size=p[N]).astype(np.int32))
        val.append((w / np.repeat(deg, deg)).astype(np.float32))
    bias = -rng.uniform(0.8, 1.2, size=N).astype(np.float32)   # a layer takes about one off
    if kind == "general":
        m = sp.Model.from_csr(ptr, idx, val, bias)
    else:
        m = sp.Model([a.reshape(N, 32) for a in idx], [a.reshape(N, 32) for a in val], bias)
    g = torch.Generator(device=dev).manual_seed(N + L)
    v = 1.5 + torch.rand((batch, 1), generator=g, device=dev) * (1.1 * L)
    v[: batch // 5] = L / 2      # the first fifth of the batch dies together
    y0 = v * (0.9 + 0.2 * torch.rand((batch, N), generator=g, device=dev))
    n, rows, Y = m.infer(y0)
    assert m.launches()[1] > 0 and 0 < n < batch
    assert bool((Y.max(1).values > Y.min(1).values).all())
    step = 1000
    for r in (0, batch // 5 - 500, batch // 2, batch - step):
        ns, rs, Ys = m.infer(y0[r:r + step].contiguous())
        assert m.launches() == (1, 1)
        mine = (rows >= r) & (rows < r + step)
        assert ns == int(mine.sum()) and torch.equal(rows[mine] - r, rs) and torch.equal(Y[mine], Ys)
    m.close()


@pytest.mark.parametrize("N,batch,L,uniform,one_by_one", [
    (516, 40000, 1, False, 1), (512, 40000, 1, False, 0), (1028, 9000, 1, True, 1), (2048, 9000, 1, False, 1),
    (2048, 21000, 2, True, 2), (2048, 9000, 2, True, 0), (4096, 17000, 3, True, 3), (4096, 9000, 4, False, 0),
    (4096, 25000, 4, False, 4), (1500, 50000, 3, False, 3), (4092, 25000, 2, False, 0), (3072, 20000, 1, True, 0),
    (4096, 17000, 5, True, 2), (2048, 50000, 5, False, 2), (4096, 25000, 5, False, 0),
])
def test_few_layers_on_many_rows_run_one_by_one(N, batch, L, uniform, one_by_one):
    """Layers that are not worth a launch that keeps rows in LDS: a launch each, and the same bits as the same rows get
    on the chip, in batches small enough for one launch."""
    import torch
    import paper_2007_14152_amd as sp
    dev = "cuda:0"
    g = torch.Generator(device=dev).manual_seed(N + batch + L)
    rng = np.random.default_rng(N + batch + L)
    idx = [np.sort(rng.integers(0, N, size=(N, 32)), axis=1).astype(np.int32) for _ in range(L)]
    val = [np.full((N, 32), 0.0625, np.float32) if uniform else rng.uniform(0.02, 0.11, size=(N, 32)).astype(np.float32)
           for _ in range(L)]
    m = sp.Model(idx, val, -rng.uniform(0.0, 0.5, size=N).astype(np.float32))
    density = torch.rand((batch, 1), generator=g, device=dev) * 0.5
    y0 = (torch.rand((batch, N), generator=g, device=dev) < density).float()
    y0[::97] = 0
    m.set_profiling(True)
    n, rows, Y = m.infer(y0)
    launches, resident = m.launches()
    assert launches - resident == one_by_one and (resident > 0) == (one_by_one < L)
    run, rows_in, ms = m.profile()
    assert run == L and rows_in[0] == batch and np.all(np.diff(rows_in) <= 0) and n <= rows_in[L - 1] and np.all(ms > 0)
    assert 0 < n < batch
    step = 1000
    for r in (0, batch // 2 // step * step, batch - step):
        ns, rs, Ys = m.infer(y0[r:r + step].contiguous())
        assert m.launches() == (1, 1)
        mine = (rows >= r) & (rows < r + step)
        assert ns == int(mine.sum()) and torch.equal(rows[mine] - r, rs) and torch.equal(Y[mine], Ys)
    m.close()


@pytest.mark.parametrize("N,stride,uniform", [(1024, 8, True), (1500, 20, False), (2048, 24, True), (2048, 24, False),
                                              (3072, 40, False), (4096, 16, True), (4096, 64, False), (4092, 50, False)])
def test_windows_inside_the_row(N, stride, uniform):
    """Layers whose blocks read a part of the row only, over the row end in the last blocks: the kernels of single layers
    stage that part (weights in host memory; single layers on many rows) in the layout of the whole row, with the same
    sums as on the chip; against the oracle."""
    import torch
    import paper_2007_14152_amd as sp
    rng = np.random.default_rng(N + stride)
    L = 3
    j, k = np.arange(N, dtype=np.int64)[:, None], np.arange(32, dtype=np.int64)[None, :]
    idx = [np.sort((j + 300 * l + k * stride + rng.integers(0, 4, size=(N, 32))) % N, axis=1).astype(np.int32) for l in range(L)]
    val = [np.full((N, 32), 0.0625, np.float32) if uniform else rng.uniform(0.02, 0.11, size=(N, 32)).astype(np.float32)
           for _ in range(L)]
    bias = -rng.uniform(0.0, 0.4, size=N).astype(np.float32)
    Y0 = synth.gen_y0(600, N, 37, density="mixed")
    Y0[7] = 0
    ref = oracle.infer(idx, val, bias, Y0)
    y0 = torch.from_numpy(Y0).to("cuda:0")
    got = []
    for ooc in (False, True):
        m = sp.Model(idx, val, bias, out_of_core=ooc)
        got.append(m.infer(y0))
        assert m.launches() == ((L, 0) if ooc else (1, 1))
        m.close()
    assert got[0][0] == got[1][0] and torch.equal(got[0][1], got[1][1]) and torch.equal(got[0][2], got[1][2])
    common, _ = check_against_oracle(ref, got[0][0], got[0][1].cpu().numpy(), got[0][2].cpu().numpy(), what="windows N=%d" % N)
    assert 0 < common < 600
    # one layer, many rows
    m = sp.Model(idx[:1], val[:1], bias)
    big = y0.repeat(30, 1)
    n, rows, Y = m.infer(big)
    one = m.infer(y0)
    m.close()
    keep = rows < 600
    assert n == 30 * one[0] and torch.equal(rows[keep], one[1]) and torch.equal(Y[keep], one[2])


@pytest.mark.parametrize("N,batch,L,die", [
    (4096, 1600, 9, True),     # rows in LDS, two launches
    (4096, 1600, 9, False),
    (8192, 700, 5, True),      # a launch per layer
    (8192, 700, 5, False),
])
def test_last_layer_writes_to_the_callers_array(N, batch, L, die):
    """When no row has died lately, the last launch writes its rows where the caller wants them; those that die in the
    very last layer leave gaps, which the survivors close.  Row r holds the integer v_r in every column, a layer turns v
    into v - 1, exactly."""
    import torch
    import paper_2007_14152_amd as sp
    dev = "cuda:0"
    rng = np.random.default_rng(N + die)
    v = rng.integers(L + 1, L + 9, size=batch)
    if die:
        v[rng.uniform(size=batch) < 0.3] = L
        v[[0, batch - 1]] = L
    idx = [torch.from_numpy(np.sort(rng.integers(0, N, size=(N, 32)), axis=1).astype(np.int32)).to(dev) for _ in range(L)]
    val = torch.full((N, 32), 1.0 / 32, dtype=torch.float32, device=dev)
    m = sp.Model(idx, [val] * L, torch.full((N,), -1.0, device=dev), device=dev)
    y0 = torch.from_numpy(v.astype(np.float32)).to(dev)[:, None].expand(batch, N).contiguous()
    for _ in range(2):
        n, rows, Y = m.infer(y0)
        alive = np.nonzero(v > L)[0]
        assert n == len(alive) and np.array_equal(rows.cpu().numpy(), alive)
        assert bool((Y == torch.from_numpy((v[alive] - L).astype(np.float32)).to(dev)[:, None]).all())
    m.close()


@pytest.mark.parametrize("N,batch,uniform", [
    (4100, 37, False),     # four rows per tile, units of 33 groups of 64 neurons, a ragged last one
    (4864, 1030, True),    # the widest rows of four per tile; more tiles than workgroups
    (4868, 700, False),    # three rows per tile
    (6656, 95, True),
    (6660, 501, False),    # two
    (9984, 130, True),
    (9988, 260, False),    # one
    (13000, 67, True),
    (16384, 515, False),   # the widest row there is
])
def test_whole_rows_in_lds(N, batch, uniform):
    """Rows of 4097 to 16384 columns read from anywhere (fused_flat_kernel): one to four rows per tile, ragged ends."""
    import torch
    import paper_2007_14152_amd as sp
    rng = np.random.default_rng(N)
    L = 2
    idx = [np.sort(rng.integers(0, N, size=(N, 32)), axis=1).astype(np.int32) for _ in range(L)]
    val = [np.full((N, 32), 0.0625, np.float32) if uniform else rng.uniform(0.02, 0.11, size=(N, 32)).astype(np.float32)
           for _ in range(L)]
    bias = -rng.uniform(0.0, 0.4, size=N).astype(np.float32)
    Y0 = synth.gen_y0(batch, N, 31, density="mixed")
    Y0[5] = 0
    ids = np.arange(batch) if batch <= 300 else np.r_[0:100, batch - 100:batch]
    ref = oracle.infer(idx, val, bias, Y0[ids])
    m = sp.Model(idx, val, bias)
    n, rows, Y = m.infer(torch.from_numpy(Y0).to("cuda:0"))
    m.close()
    rows, Y = rows.cpu().numpy(), Y.cpu().numpy()
    mine = np.isin(rows, ids)
    common, _ = check_against_oracle(ref, int(mine.sum()), rows[mine], Y[mine], row_ids=ids, what="whole rows N=%d" % N)
    assert common > 0 and n == len(rows) < batch
