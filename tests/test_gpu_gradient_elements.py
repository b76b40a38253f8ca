"""Every single element of the training gradients.  The kernels hand the BF16 operands of the
weight gradients over in a layout of their own, where one misplaced element, or one in a row,
does not show in a norm over a parameter group.  Here the operands are read back from the
workspace and checked in place, and the gradients are those operands' sums in 64 bits, within
the bound of an FP32 sum."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import say
from oracle import mlp as M
from paper_1409_4923_amd import bmotor as B
from paper_1409_4923_amd import workloads as W

H, IN = 256, 5


def fragments(raw, at, members, batch):
    """BF16 operand [member][batch / 32][16 feature tiles][4 eights of rows][16 features][8 rows]
    at byte `at` of the workspace, as FP64 [member][row][feature]; and where the next begins."""
    n = members * batch * H
    v = (raw[at:at + 2 * n].view(np.uint16).astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    v = v.reshape(members, batch // 32, 16, 4, 16, 8).transpose(0, 1, 3, 5, 2, 4)
    return v.reshape(members, batch, H), at + (2 * n + 255) // 256 * 256


def sums(ops, m):
    """Gradients of the summed layers of member m, and sum |dz a| of every element."""
    one = np.ones((ops["u"].shape[1], 1))
    g, mag = {}, {}
    for name, d, a in (("W1", "dz1", "u"), ("b1", "dz1", None), ("W2", "dz2", "a1"), ("b2", "dz2", None),
                       ("W3", "dz3", "a2"), ("b3", "dz3", None)):
        d, a = ops[d][m], one if a is None else ops[a][m]
        g[name], mag[name] = (d.T @ a).reshape(-1), (np.abs(d).T @ np.abs(a)).reshape(-1)
    return g, mag


def bound(batch):
    """Of an FP32 sum over the batch, relative to sum |dz a|: products of two BF16 are exact,
    each addition rounds to 2^-24 or cuts off 2^-23, and none follows more others than the
    rows of a chunk (the batch in 1, 2, 4 or 8) and the partial sums added after it."""
    split = 1
    while split < 8 and 512 * split <= batch and batch % (64 * split) == 0:
        split *= 2
    return min(batch, batch // split + 72) * 2.0 ** -23


def offsets():
    at = np.cumsum([0] + [int(np.prod(sh)) for _, sh in M.SIZES])
    return {name: slice(at[k], at[k + 1]) for k, (name, _) in enumerate(M.SIZES)}


@pytest.mark.parametrize("batch", [64, 4096])
def test_the_bound_sees_one_element(batch):
    """Planted in the sums: an element that holds its neighbour's value, and one whose sum
    misses 32 rows, leave the bound nearly everywhere."""
    rng = np.random.default_rng(44)
    ops = {k: rng.standard_normal((1, batch, IN if k == "u" else H)) for k in ("u", "a1", "a2", "dz1", "dz2", "dz3")}
    g, mag = sums(ops, 0)
    part, _ = sums({k: v[:, :-32] for k, v in ops.items()}, 0)
    for name in ("W2", "W3", "W1"):
        for wrong in (np.roll(g[name], 1), part[name]):
            assert np.mean(np.abs(wrong - g[name]) > bound(batch) * mag[name]) > 0.9


@pytest.mark.gpu
@pytest.mark.parametrize("members,batch", [(1, 64), (16, 128), (3, 512), (2, 1088), (5, 1024), (2, 2752), (5, 2752), (2, 4096)])
def test_every_element_of_the_gradients(members, batch):
    import torch
    p = W.mlp_params(members, seed=43)
    x = W.surrogate_queries(3000, seed=41)
    t = (0.3 * np.sin(x[:, 0]) + 0.5 * x[:, 2]).astype(np.float32)
    idx = np.random.default_rng(42).integers(0, 3000, (members, batch)).astype(np.int32)
    say("gradient elements", members, batch)
    s = B.Surrogate(members, params=p)
    s.backward(*(torch.tensor(v, device="cuda") for v in (x, t, idx)))
    grad = s.grad.cpu().numpy().astype(np.float64)
    raw = s._ws[batch, True].cpu().numpy()
    ops, at = {}, 0
    for name in ("a1", "a2", "dz1", "dz2", "dz3"):
        ops[name], at = fragments(raw, at, members, batch)
    ops["u"] = raw[at:at + 4 * members * batch * IN].view(np.float32).astype(np.float64).reshape(members, batch, IN)
    for m in sorted({0, members - 1}):
        # the operands in their places: BF16 roundings move a value by 2^-8 of its row's
        # largest at each of at most five layers, the flips they cause by less
        _, c = M.forward(p[m].astype(np.float64), x[idx[m]].astype(np.float64), bf16_weights=True)
        assert np.max(np.abs(ops["u"][m] - c["u"])) <= 1e-5
        dy = 2.0 * (c["a3"] @ c["W"]["W4"] + p[m][-1] - t[idx[m]]) / batch
        dz3 = np.outer(dy, c["W"]["W4"]) * M.gelu_grad(c["z3"])
        dz2 = (dz3 @ c["W"]["W3"]) * M.gelu_grad(c["z2"])
        want = {"a1": c["a1"], "a2": c["a2"], "dz3": dz3, "dz2": dz2,
                "dz1": (dz2 @ c["W"]["W2"]) * M.gelu_grad(c["z1"])}
        scale = np.maximum(np.abs(dy), np.max(np.abs(dy)) / 16)[:, None]     # dy itself is a difference
        for name, v in want.items():
            size = np.max(np.abs(v / scale)) * scale if name[0] == "d" else np.max(np.abs(v), axis=1, keepdims=True)
            assert np.all(np.abs(ops[name][m] - v) <= 2.0 ** -4 * size), (m, name)
        g, mag = sums(ops, m)
        for name, part in offsets().items():
            if name in g:
                err = np.abs(grad[m, part] - g[name])
                assert np.all(err <= bound(batch) * mag[name]), (m, name, int(np.argmax(err / mag[name])))
