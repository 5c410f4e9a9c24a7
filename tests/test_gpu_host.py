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
