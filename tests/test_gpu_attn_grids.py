"""Attention launches of more workgroups than one grid is given (2^20): the second
launch takes up where the first ends."""

import pytest
import torch

from gpu_helpers import require_gpu, say

import paper_2609_19868_amd as Z

pytestmark = pytest.mark.gpu


def test_f32_more_groups_than_a_grid():
    """One key a row: its weight is 1, so the output is its value, bit for bit."""
    dev = require_gpu()
    B, H, D = (1 << 17) + 3, 8, 64
    g = torch.Generator(device=dev).manual_seed(7)
    q, k, v = (torch.randn((B, H, 1, D), generator=g, device=dev) for _ in range(3))
    say(f"slot_attn f32 {B * H} groups of one row and key")
    out, lse = Z.slot_attn(q, None, None, k, v, 1, 1)
    torch.cuda.synchronize()
    assert torch.equal(out, v)
    ref = (q.double() * k.double()).sum(-1) / 8
    # 64 products and sums of float32: 64 * 2^-24 of at most |score| + |q||k| / 8, below 16 here
    assert (lse - ref).abs().max() <= 64 * 2.0**-24 * 16


def test_merge_of_more_rows_than_a_grid():
    """Nine splits of 2.1 million rows (two a workgroup of the merge) against one
    split, which needs no merge.  Probabilities are rounded to bf16 against another
    running maximum in each (2^-9 of each term) and the outputs to bf16: 1e-2."""
    dev = require_gpu()
    T, D, P = (1 << 21) + 5, 128, 9 * 64
    g = torch.Generator(device=dev).manual_seed(8)
    q, ks, vs = (torch.randn((1, 1, T, D), generator=g, device=dev, dtype=torch.bfloat16) for _ in range(3))
    kc, vc = (torch.randn((1, 1, P, D), generator=g, device=dev, dtype=torch.bfloat16) for _ in range(2))
    res = []
    for n in (1, 9):
        say(f"slot_attn bf16 {T} rows, {n} splits")
        res.append(Z.slot_attn(q, kc, vc, ks, vs, T, 1, prefix_splits=n))
        torch.cuda.synchronize()
    for t in (slice(0, T), slice(T - 40, T), slice((1 << 21) - 8, (1 << 21) + 5)):
        a, b = res[0][0][:, :, t].float(), res[1][0][:, :, t].float()
        assert (a - b).norm() <= 1e-2 * a.norm()
        assert (res[0][1][:, :, t] - res[1][1][:, :, t]).abs().max() <= 1e-3
