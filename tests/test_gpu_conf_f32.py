"""Float32 LM-head reduction (MFMA tiles of 128 ids x 32 or 64 rows) against
the float64 oracle at the edges of its tiles: row tiles, vocabulary blocks and
groups, contraction tails, rows that are not 16-byte aligned.

Tolerance: a logit is a float32 running sum of H products; each addition rounds
by up to 2^-24 of the partial sum (at most about the row's largest logit, and
the log-sum-exp is no smaller where it matters), and H independent roundings
add up to sqrt(H) of one.  lse is checked to that, sqrt(H) * 2^-24 * |lse|, plus
2e-6 for its own rounding and logarithm; everything also to the 1e-4 of the
other float32 checks."""

import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import check_conf, require_gpu, say

import paper_2609_19868_amd as Z

pytestmark = pytest.mark.gpu

# rows, hidden, vocab, offset of the hidden and of the W pointer in floats
SHAPES = [
    (1, 1, 1, 0, 0), (2, 3, 129, 0, 0), (31, 30, 33, 0, 0), (32, 32, 4096, 0, 0), (33, 36, 4100, 0, 0),
    (64, 64, 33000, 0, 0), (65, 100, 5000, 0, 0), (130, 775, 2500, 0, 0), (7, 1030, 70001, 0, 0),
    (16, 128, 9001, 1, 0), (40, 256, 3000, 0, 2), (300, 68, 300, 0, 0), (64, 2052, 1000, 0, 0),
]


def _tensors(M, H, V, off_x, off_w, dev):
    rng = np.random.default_rng(M * 7919 + H * 31 + V)
    h = rng.standard_normal((M, H)).astype(np.float32)
    w = (rng.standard_normal((V, H)) * 0.1).astype(np.float32)

    def at(x, off):
        t = torch.empty(x.size + off, dtype=torch.float32, device=dev)[off:].view(x.shape)
        t.copy_(torch.from_numpy(x))
        return t

    return h, w, at(h, off_x), at(w, off_w), rng


@pytest.mark.parametrize("M,H,V,off_x,off_w", SHAPES)
def test_f32_tile_edges(M, H, V, off_x, off_w):
    dev = require_gpu()
    h, w, hd, wd, rng = _tensors(M, H, V, off_x, off_w, dev)
    targets = rng.integers(0, V, M).astype(np.int32)
    say(f"slot_confidence f32 M={M} H={H} V={V} offsets {off_x} {off_w}")
    res = Z.slot_confidence(hd, wd, target_ids=torch.from_numpy(targets).to(dev))
    torch.cuda.synchronize()
    hf, wf = h.astype(np.float64), w.astype(np.float64)
    ref = oracle.slot_confidence(hf, wf, target_ids=targets)
    check_conf(res, ref, what=f"{M}x{H}x{V}", f32=True, logit_of=lambda i, v: float(hf[i] @ wf[v]))
    bound = 2e-6 + np.sqrt(H) * 2.0**-24 * np.maximum(1.0, np.abs(ref["lse"]))
    assert np.all(np.abs(res["lse"].cpu().numpy() - ref["lse"]) <= bound)

    say(f"slot_sample f32 M={M} H={H} V={V} (rows gathered)")
    rows = rng.integers(0, M, M + 3).astype(np.int32)
    got = Z.slot_sample(hd, wd, 0.8, 12345, 7, rows=torch.from_numpy(rows).to(dev))
    torch.cuda.synchronize()
    ref = oracle.slot_sample(hf[rows], wf, 0.8, 12345, 7, row_ids=np.arange(M + 3))
    decided = ref["score_gap"] >= 1e-3 / 0.8
    sid = got["sample_id"].cpu().numpy()
    assert np.array_equal(sid[decided], ref["sample_id"][decided])
    p = np.exp(np.einsum("ih,ih->i", hf[rows], wf[sid]) - ref["lse"])
    assert np.abs(got["sample_prob"].cpu().numpy() - p).max() <= 1e-4 * max(1e-3, p.max())


@pytest.mark.parametrize("M,V", [(5, 300), (64, 5001)])
@pytest.mark.parametrize("top", [20.0, 300.0, 1000.0, -700.0])
def test_f32_dominant_logits(top, M, V):
    """A few logits at and just below a large maximum, the rest far away.  Every
    logit is exact (integers times 2^-3, below 2^24 of them), so max_prob carries
    only the rounding of the exponentials: (x - m) * log2e to 2^-24 of up to 6 log2
    units (2.5e-7 of the term), the instruction's and the sums' few 2^-24."""
    dev = require_gpu()
    rng = np.random.default_rng(int(abs(top)) + V)
    H = 36
    w = np.zeros((V, H), np.float32)
    w[:, 0] = 8 * (top - 100 - rng.integers(0, 400, V) / 8)
    w[rng.choice(V, 6, replace=False), 0] = 8 * (top - np.array([0.0, 0.125, 0.5, 1.25, 2.5, 4.0]))
    w[:, 1:] = rng.integers(-3, 4, (V, H - 1))
    h = np.zeros((M, H), np.float32)
    h[:, 0] = 0.125
    say(f"slot_confidence f32 M={M} V={V} dominant logit {top}")
    res = Z.slot_confidence(torch.from_numpy(h).to(dev), torch.from_numpy(w).to(dev))
    torch.cuda.synchronize()
    ref = oracle.slot_confidence(h.astype(np.float64), w.astype(np.float64))
    p = res["max_prob"].cpu().numpy().astype(np.float64)
    assert p.max() <= 1.0
    assert np.abs(p / ref["max_prob"] - 1).max() <= 1e-6
    assert np.array_equal(res["argmax"].cpu().numpy(), ref["argmax"])
