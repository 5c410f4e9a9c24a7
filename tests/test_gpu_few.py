"""Networks of at most 4096 neurons on few rows (few_kernel): one to four rows per workgroup, ragged last workgroups, one
to four groups of 64 neurons per wave, connections of all three kinds, a deep network shared out anew behind two layers, and a
single row, which one launch finishes.  The bits are those of the same rows in a batch that resident_kernel takes; values
against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from parity_util import check_against_oracle

pytestmark = pytest.mark.gpu


def network(kind, N, L, rng):
    if kind == "general":
        ptr, idx, val = [], [], []
        for l in range(L):
            deg = rng.integers(0, 70, size=N)
            p = np.zeros(N + 1, dtype=np.int32)
            np.cumsum(deg, out=p[1:])
            ptr.append(p)
            idx.append(rng.integers(0, N, size=int(p[N])).astype(np.int32))
            val.append((rng.uniform(0.5, 1.5, size=int(p[N])) * np.repeat(2.0 / np.maximum(deg, 1), deg)).astype(np.float32))
        return ptr, idx, val
    idx = [np.sort(rng.integers(0, N, size=(N, 32)), axis=1).astype(np.int32) for _ in range(L)]
    val = [np.full((N, 32), 0.0625, np.float32) if kind == "uniform" else rng.uniform(0.02, 0.11, size=(N, 32)).astype(np.float32)
           for _ in range(L)]
    return None, idx, val


@pytest.mark.parametrize("kind", ["uniform", "weights", "general"])
@pytest.mark.parametrize("N,L", [(32, 3), (100, 3), (256, 1), (1024, 4), (1028, 3), (2052, 3), (2560, 2), (4096, 3)])
def test_few_rows(kind, N, L):
    import torch
    import paper_2007_14152_amd as sp
    rng = np.random.default_rng(N + L + len(kind))
    ptr, idx, val = network(kind, N, L, rng)
    bias = -rng.uniform(0.0, 0.4, size=N).astype(np.float32)
    many = 1100                                        # more than few_kernel takes
    Y0 = synth.gen_y0(many, N, 51, density="mixed")
    Y0[2] = 0
    ref = oracle.infer(idx, val, bias, Y0, ptr=ptr)
    m = sp.Model.from_csr(ptr, idx, val, bias) if ptr else sp.Model(idx, val, bias)
    y0 = torch.from_numpy(Y0).to("cuda:0")
    n, rows, Y = m.infer(y0)
    assert m.row_kernel() == sp.SPDNN_ROWS_RESIDENT
    check_against_oracle(ref, n, rows.cpu().numpy(), Y.cpu().numpy(), what="%s N=%d" % (kind, N))
    for first, batch in ((0, 1024), (3, 769), (4, 768), (2, 513), (1, 512), (0, 257), (0, 256), (5, 7), (0, 3), (1, 1), (2, 1)):
        m.set_profiling(batch in (1, 512, 513, 1024))
        n2, rows2, Y2 = m.infer(y0[first:first + batch].contiguous())
        few = batch <= (1024 if N <= 2048 else 512) and not (kind == "general" and N > 2560)
        assert m.one_launch(batch) and m.launches() == (1, 1) and m.row_kernel() == (sp.SPDNN_ROWS_FEW if few else sp.SPDNN_ROWS_RESIDENT)
        keep = (rows >= first) & (rows < first + batch)
        assert n2 == int(keep.sum()) and torch.equal(rows2, rows[keep] - first) and torch.equal(Y2, Y[keep]), (first, batch)
        if batch in (512, 513, 1024) and not (ref.fragile_layer >= 0).any():
            want = oracle.infer(idx, val, bias, Y0[first:first + batch], ptr=ptr)
            run, rows_in, _ = m.profile()
            assert [int(x) for x in rows_in[:run]] == [int(x) for x in want.active_per_layer[:run]]
    m.set_profiling(False)
    n3, rows3, _ = m.infer(y0[1:2].contiguous(), want_Y=False)
    assert n3 == int((rows == 1).sum()) and len(rows3) == n3
    m.close()


@pytest.mark.parametrize("N,kind", [(64, "uniform"), (1024, "weights"), (1500, "uniform")])
def test_deep_networks_are_shared_out_anew(N, kind):
    """64 layers and more on more rows than workgroups: two launches, the second on the rows that are left -- three in four,
    half, fewer than workgroups, none; one to four per workgroup, and just above the edges between them."""
    import torch
    import paper_2007_14152_amd as sp
    L = 64
    rng = np.random.default_rng(N)
    _, idx, val = network(kind, N, L, rng)
    val = [v / (2 * v.sum(axis=1, keepdims=True)) * 2.2 for v in val]
    val = [np.full((N, 32), 0.04, np.float32) if kind == "uniform" else v.astype(np.float32) for v in val]
    bias = np.full(N, -0.05, np.float32)
    m = sp.Model(idx, val, bias)
    for batch, alive in ((1000, 0.75), (1024, 0.5), (700, 0.2), (300, 0.0)):
        live = rng.uniform(size=batch) < alive
        y0 = torch.from_numpy(np.where(live, 0.9, 0.04).astype(np.float32)).to("cuda:0")[:, None].expand(batch, N).contiguous()
        assert not m.one_launch(batch)
        n, rows, Y = m.infer(y0)
        assert m.launches() == (2, 2) and m.row_kernel() == sp.SPDNN_ROWS_FEW
        ids = np.nonzero(live)[0]
        assert n == len(ids) and np.array_equal(rows.cpu().numpy(), ids)
        if n:
            one = m.infer(y0[int(ids[0]):int(ids[0]) + 1].contiguous())[2]
            assert bool((Y == one).all())
    m.close()


@pytest.mark.parametrize("kind,N", [("uniform", 96), ("weights", 1024), ("uniform", 1500), ("general", 500)])
def test_rows_keep_their_values_when_they_are_shared_out_anew(kind, N):
    """Rows of different values, some of them blank: every row gives the bits that it gives in a batch that resident_kernel takes,
    whichever of one to four places of a workgroup of the second launch it comes to, and the layers' counts are the survivors'."""
    import torch
    import paper_2007_14152_amd as sp
    L = 64
    rng = np.random.default_rng(7 * N)
    ptr, idx, val = network(kind, N, L, rng)
    if kind == "general":   # weights that sum to 1 per neuron, as below
        val = [(v / np.maximum(np.repeat(np.add.reduceat(np.r_[v, 0], p[:-1]) * (np.diff(p) > 0) + (np.diff(p) == 0), np.diff(p)), 1e-9)).astype(np.float32)
               for v, p in zip(val, ptr)]
    else:
        val = [np.full((N, 32), 1 / 32, np.float32) if kind == "uniform" else (v / v.sum(axis=1, keepdims=True)).astype(np.float32) for v in val]
    bias = np.zeros(N, np.float32)          # averages of the row's values: they neither die nor reach the clip, and differ from row to row
    m = sp.Model.from_csr(ptr, idx, val, bias) if ptr else sp.Model(idx, val, bias)
    many = 1300                             # more than few_kernel takes
    Y0 = rng.uniform(0.0, 1.0, size=(many, N)).astype(np.float32) * rng.uniform(0.5, 20.0, size=(many, 1)).astype(np.float32)
    blank = rng.uniform(size=many) < 0.35
    Y0[blank] = 0
    y0 = torch.from_numpy(Y0).to("cuda:0")
    n, rows, Y = m.infer(y0)
    assert m.row_kernel() == sp.SPDNN_ROWS_RESIDENT and n == int((~blank).sum())
    assert len(torch.unique(Y[:, 0])) > 0.9 * n
    live = np.nonzero(~blank)[0]
    dead = np.nonzero(blank)[0]
    m.set_profiling(True)
    for alive, batch in ((600, 800), (513, 700), (512, 700), (257, 500), (256, 400), (3, 300), (768, 1024), (769, 1024)):
        ids = np.sort(np.r_[live[:alive], dead[:batch - alive]])
        n2, rows2, Y2 = m.infer(y0[torch.from_numpy(ids).to("cuda:0")].contiguous())
        assert m.launches() == (2, 2) and m.row_kernel() == sp.SPDNN_ROWS_FEW
        kept = np.nonzero(~blank[ids])[0]
        assert n2 == len(kept) and np.array_equal(rows2.cpu().numpy(), kept)
        at = torch.from_numpy(np.searchsorted(live, ids[kept])).to("cuda:0")
        assert torch.equal(Y2, Y[at]), (alive, batch)
        run, rows_in, _ = m.profile()
        assert len(ids) == batch and run == L and [int(x) for x in rows_in] == [batch] + [alive] * (L - 1)
    m.close()
