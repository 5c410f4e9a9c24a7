"""Inputs in host memory whose last batch is large enough to be copied and inferred in pieces (spdnn_infer_host): the same
survivors, numbers and bits as one spdnn_infer over all rows, for one batch and for several, at the size where a batch is
first cut, and in a network too deep for it."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,batch,per,L", [
    (4096, 5001, 5001, 3),      # one batch of 82 MB: four pieces
    (4096, 3100, 1030, 3),      # four batches, the last of ten rows
    (4096, 4096, 1024, 3),      # 16 MB each: two pieces of the last
    (4096, 2047, 1024, 3),      # one row less: one
    (16384, 700, 300, 2),       # a ragged last batch of 6 MB
    (16384, 601, 301, 2),       # of 20 MB
    (1024, 9000, 9000, 50),     # fifty layers: whole
])
def test_pieces_of_the_last_batch(N, batch, per, L):
    import torch
    import paper_2007_14152_amd as sp
    rng = np.random.default_rng(N + batch)
    idx = [np.sort(rng.integers(0, N, size=(N, 32)), axis=1).astype(np.int32) for _ in range(L)]
    val = [np.full((N, 32), 0.0625, np.float32)] * L
    m = sp.Model(idx, val, np.full(N, -0.3, np.float32))
    Y0 = torch.from_numpy(synth.gen_y0(batch, N, 61, density="mixed"))
    want = m.infer(Y0.to("cuda:0"))
    assert 0 < want[0] < batch
    host = Y0.pin_memory()
    for src in (host, Y0):
        n, rows, Y = m.infer_batched(src, per)
        assert n == want[0] and torch.equal(rows, want[1]) and torch.equal(Y, want[2])
    m.close()
