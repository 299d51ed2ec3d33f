"""bf16 LM-head reduction where its stages and vocabulary tiles can go wrong: one
stage a tile, a partial last stage, a last tile that fills one vocabulary half,
rows of W that do not start on 128-byte lines; the few-row and the 256-row tile.
Against the float64 oracle, tolerances of the other bf16 checks."""

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_helpers import check_conf, require_gpu, say

import paper_2609_19868_amd as Z

pytestmark = pytest.mark.gpu

# hidden, vocab, offset of the W pointer in elements
SHAPES = [
    (64, 70001, 0),    # one stage a tile; groups of two tiles, the last of few ids
    (72, 300, 0),      # two stages, the second of 8 columns; one short tile a group
    (128, 41000, 8),   # two whole stages, W 16 bytes past a line
    (200, 70001, 0),   # rows of 400 bytes
    (192, 140000, 0),  # three stages, whole lines
]


@pytest.mark.parametrize("M", [25, 65, 300])
@pytest.mark.parametrize("H,V,off", SHAPES)
def test_bf16_stage_edges(M, H, V, off):
    dev = require_gpu()
    rng = np.random.default_rng(M * 7919 + H * 31 + V)
    hb = W.bf16_bits(rng.standard_normal((M, H)).astype(np.float32))
    wb = W.bf16_bits((rng.standard_normal((V, H)) * 0.1).astype(np.float32))
    targets = rng.integers(0, V, M).astype(np.int32)

    def at(bits, o):
        t = torch.empty(bits.size + o, dtype=torch.bfloat16, device=dev)[o:].view(bits.shape)
        t.copy_(torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16))
        return t

    hd, wd = at(hb, 0), at(wb, off)
    say(f"slot_confidence M={M} H={H} V={V} offset {off}")
    res = Z.slot_confidence(hd, wd, target_ids=torch.from_numpy(targets).to(dev))
    torch.cuda.synchronize()
    hf, wf = W.as_f64(hb, "bf16"), W.as_f64(wb, "bf16")
    ref = oracle.slot_confidence(hf, wf, target_ids=targets)
    check_conf(res, ref, what=f"{M}x{H}x{V}", logit_of=lambda i, v: float(hf[i] @ wf[v]))
    say(f"slot_sample M={M} H={H} V={V} offset {off}")
    got = Z.slot_sample(hd, wd, 0.9, 4321, 3)
    torch.cuda.synchronize()
    # the sampled reduction accumulates the same statistics
    assert torch.equal(got["max_prob"], res["max_prob"]) and torch.equal(got["lse"], res["lse"])
    ids = got["sample_id"].cpu().numpy()
    z = np.einsum("ij,ij->i", hf, wf[ids])
    np.testing.assert_allclose(got["sample_prob"].cpu().numpy(), np.exp(z - ref["lse"]), rtol=1e-3)
    # the draws themselves, on rows at the edges of the row tiles and blocks: the
    # best score is decided where it leads by more than the logits' rounding
    rows = np.unique(np.minimum([0, 1, 24, 31, 32, 63, 64, 127, 128, 255, 256, 299], M - 1))
    draw = oracle.slot_sample(hf[rows], wf, 0.9, 4321, 3, row_ids=rows)
    decided = draw["score_gap"] >= 1e-3 / 0.9
    assert decided.sum() >= 0.9 * len(rows)
    assert np.array_equal(ids[rows][decided], draw["sample_id"][decided])
