"""Inputs in host memory whose last batch is large enough to be copied and inferred in pieces (spdnn_infer_host): the same
survivors, numbers and bits as one spdnn_infer over all rows, for one batch and for several, at the size where a batch is
first cut, and in a network too deep for it.  Inputs in pageable memory go through in whole batches."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,batch,per,L,pieces", [
    (4096, 5001, 5001, 3, 4),    # one batch of 82 MB: four pieces
    (4096, 3100, 1030, 3, 4),    # four batches, the last of ten rows
    (4096, 4096, 1024, 3, 5),    # 16 MB each: two pieces of the last
    (4096, 2047, 1024, 3, 2),    # one row less: one
    (16384, 700, 300, 2, 3),     # a ragged last batch of 6 MB
    (16384, 601, 301, 2, 3),     # of 20 MB
    (1024, 9000, 9000, 50, 1),    # fifty layers: whole
])
def test_pieces_of_the_last_batch(N, batch, per, L, pieces):
    import torch
    import paper_2007_14152_amd as sp
    rng = np.random.default_rng(N + batch)
    idx = [np.sort(rng.integers(0, N, size=(N, 32)), axis=1).astype(np.int32) for _ in range(L)]
    val = [np.full((N, 32), 0.0625, np.float32)] * L
    m = sp.Model(idx, val, np.full(N, -0.3, np.float32))
    Y0 = torch.from_numpy(synth.gen_y0(batch, N, 61, density="mixed"))
    want = m.infer(Y0.to("cuda:0"))
    assert 0 < want[0] < batch
    batches = range(0, batch, per)
    launches = 0
    for lo in batches:
        m.infer(Y0[lo:lo + per].to("cuda:0"))
        launches += m.launches()[0]
    host = Y0.pin_memory()
    for src in (host, Y0):
        n, rows, Y = m.infer_batched(src, per)
        assert n == want[0] and torch.equal(rows, want[1]) and torch.equal(Y, want[2])
        if src is Y0 or pieces == len(batches):
            assert m.launches()[0] == launches
        else:   # (three layers or fewer, and fewer in a piece than in a batch: a launch for each piece, or one for each of its layers)
            assert m.launches()[0] == pieces * (1 if N <= 4096 else L)
    m.close()


@pytest.mark.parametrize("N,batch,per,L,pieces", [
    (4096, 2560, 2560, 3, 2),    # 40 MB: cut in two
    (4096, 2559, 2559, 3, 1),    # a row less
    (16384, 1700, 1700, 3, 3),   # 106 MB: one half, a quarter, and the rest
    (16384, 1200, 400, 3, 3),    # batches of 25 MB
    (4096, 3072, 3072, 180, 1),  # 180 layers: from 56 MB on
])
def test_pieces_of_networks_of_strided_sums(N, batch, per, L, pieces):
    import torch
    import paper_2007_14152_amd as sp
    idx = [synth.gen_layer_strided(N, (1, N // 32, 3)[l % 3]) for l in range(min(L, 3))]
    idx = [idx[l % len(idx)] for l in range(L)]
    m = sp.Model(idx, [np.full((N, 32), 0.0625, np.float32)] * L, np.full(N, -0.3, np.float32))
    Y0 = torch.from_numpy(synth.gen_y0(batch, N, 61, density="mixed"))
    want = m.infer(Y0.to("cuda:0"))
    assert 0 < want[0] < batch
    n, rows, Y = m.infer_batched(Y0.pin_memory(), per)
    assert m.row_kernel() == sp.SPDNN_ROWS_STRIDED and (L > 3 or m.launches()[0] == pieces)
    assert n == want[0] and torch.equal(rows, want[1]) and torch.equal(Y, want[2])
    if L > 3:    # several launches for a batch: as many as in one call
        m.infer(Y0.to("cuda:0"))
        one = m.launches()
        m.infer_batched(Y0.pin_memory(), per)
        assert m.launches() == one
    m.close()
