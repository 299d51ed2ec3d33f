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
