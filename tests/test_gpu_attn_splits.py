"""The merge of many prefix splits (more than eight: four waves share a row's
splits) against the float64 oracle, with split counts that do not divide by
four, splits that hold no key of a row, and the planner's own choice for one
long sequence.  Tolerances as in test_gpu_slot_attn.py."""

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_helpers import attn_inputs_dev, check_attn, require_gpu, say, to_f64

import paper_2609_19868_amd as Z

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("splits", [0, 9, 13, 32, 64])
def test_many_splits(splits, head_dim):
    dev = require_gpu()
    wl = W.WORKLOADS["qwen0.6b"].replace(batch=2, n_q_heads=3, n_kv_heads=1, head_dim=head_dim, prefix_len=4150,
                                         n_slots=3, slot_len=5, hidden=0, vocab=0, seed=93)
    xd, xf = attn_inputs_dev(wl, dev)
    plens = np.array([4150, 70], dtype=np.int32)  # the second row leaves most splits without a key
    say(f"slot_attn {splits} splits D={head_dim}")
    out, lse = Z.slot_attn(xd["q"], xd["k_cache"], xd["v_cache"], xd["k_slot"], xd["v_slot"], wl.n_slots, wl.slot_len,
                           prefix_len=wl.prefix_len, prefix_splits=splits, prefix_lens=torch.from_numpy(plens).to(dev))
    torch.cuda.synchronize()
    O, L = oracle.slot_attention(xf["q"], xf["k_cache"], xf["v_cache"], xf["k_slot"], xf["v_slot"], plens, wl.n_slots,
                                 wl.slot_len, wl.scale, oracle.PASS_DIFFUSION)
    check_attn(to_f64(out), to_f64(lse), O, L, "bf16", f"splits {splits}")


@pytest.mark.parametrize("prefix", [4096, 8192])
def test_few_wide_blocks_give_the_result_of_eight_splits(prefix):
    """One sequence whose 256-row blocks are few: the planner halves the blocks
    instead of doubling the splits, which leaves every bit as eight splits of
    256-row blocks have it (a call that names its splits keeps those blocks)."""
    dev = require_gpu()
    wl = W.WORKLOADS["qwen4b"].replace(batch=1, prefix_len=prefix, hidden=0, vocab=0, seed=94)
    xd, _ = attn_inputs_dev(wl, dev)
    rows = [Z._lib.slot_attn_plan(Z.slot_attn_desc(xd["q"], xd["k_cache"], xd["k_slot"], wl.n_slots, wl.slot_len,
                                                   prefix_splits=n))["rows_per_workgroup"] for n in (0, 8)]
    assert rows == [128, 256]
    say(f"slot_attn one sequence, {prefix} keys, planner's splits and eight")
    got = [Z.slot_attn(xd["q"], xd["k_cache"], xd["v_cache"], xd["k_slot"], xd["v_slot"], wl.n_slots, wl.slot_len,
                       prefix_len=wl.prefix_len, prefix_splits=n) for n in (0, 8)]
    torch.cuda.synchronize()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
