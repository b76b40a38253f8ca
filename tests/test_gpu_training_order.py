"""The order of the training step's sums depends on the batch alone, so a seeded training
run repeats bit for bit: whatever the launch, and as the layer-by-layer step did it."""
from __future__ import annotations

import hashlib

import numpy as np
import pytest

from helpers import say
from paper_1409_4923_amd import bmotor as B
from paper_1409_4923_amd import workloads as W

pytestmark = pytest.mark.gpu
W2, B2, W3, B3, END = 1536, 67072, 67328, 132864, 133120      # offsets in a member's parameters
ROWS = 6000


def inputs(members, batch):
    x = W.surrogate_queries(ROWS, seed=31)
    t = (0.25 * x[:, 2] / x[:, 4] + 0.01 * x[:, 0]).astype(np.float32)
    idx = np.random.default_rng(32).integers(0, ROWS, (members, batch)).astype(np.int32)
    return x, t, idx


def training_digest(B, members, batch, steps=5):
    """Digests of the losses and gradients of every step and of what they leave behind."""
    import torch
    x, t, idx = (torch.tensor(v, device="cuda") for v in inputs(members, batch))
    s = B.Surrogate(members, params=W.mlp_params(members, seed=33))
    h = hashlib.sha256()
    for _ in range(steps):
        loss = s.backward(x, t, idx)
        h.update(loss.cpu().numpy().tobytes())
        h.update(s.grad.cpu().numpy().tobytes())
        s.adam(2e-3)
    h.update(s.params.cpu().numpy().tobytes())
    h.update(s.wbf.cpu().numpy().tobytes())
    return h.hexdigest()[:32]


# what the step gave when every layer and direction was a launch of its own
LAYER_BY_LAYER = {
    (1, 64): "a6ce1de072303e161ab231ed90923f6f",
    (4, 448): "1e8bc9c1614aed53c92f003f11b34a2f",
    (5, 1024): "0b5607a5a3d86704ee196320bc79d759",
    (3, 1088): "193a748beb6fef6ce6e70d5be6a2bf04",
    (2, 2752): "ab614794f50ed7ee86332fb3fa54d480",
    (5, 4096): "a26d40d9c8b9af964b76753c2f2e0b21",
    (5, 576): "0c1899d92aff5473f0b30a2b37040fe3",
    (5, 4032): "0b7dd51cf76f99c67f8c6e53836f4133",
    (6, 2112): "d32f39f25a4b3b190808b3887a082e71",
}


@pytest.mark.parametrize("members,batch", sorted(LAYER_BY_LAYER))
def test_training_run_repeats(members, batch):
    """One and several chunks of rows, of 128-row tiles and not, in weight tiles of 32 rows and
    of 64, partial sums of the input layer that begin inside eight rows; five steps, every
    output."""
    say("training run", members, batch)
    assert training_digest(B, members, batch) == LAYER_BY_LAYER[members, batch]


@pytest.mark.parametrize("batch,chunks", [(512, 2), (1024, 4), (1536, 4), (2048, 8), (2560, 8)])
def test_chunks_are_added_in_order(batch, chunks):
    """The 256 x 256 layers' gradients are their chunks' gradients added one after another:
    a batch of one chunk gives that chunk's sum, times a power of two (the mean's divisor)."""
    import torch
    x, t, idx = inputs(2, batch)
    say("chunks", batch, chunks)
    s = B.Surrogate(2, params=W.mlp_params(2, seed=33))
    xd, td = torch.tensor(x, device="cuda"), torch.tensor(t, device="cuda")

    def gradient(rows):
        s.backward(xd, td, torch.tensor(np.ascontiguousarray(rows), device="cuda"))
        return s.grad.cpu().numpy()[:, W2:END]

    want = np.zeros((2, END - W2), dtype=np.float32)
    for k in range(chunks):
        n = batch // chunks
        want += gradient(idx[:, k * n:(k + 1) * n]) / np.float32(chunks)
    assert np.array_equal(gradient(idx), want)
