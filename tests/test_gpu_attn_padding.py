"""Row blocks that are only partly filled: waves without a row, which only load,
with and without the heaviest-first order, against the float64 oracle.
Tolerances as in test_gpu_slot_attn.py."""

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_helpers import attn_inputs_dev, check_attn, require_gpu, say, to_f64

import paper_2609_19868_amd as Z

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prefix_len", [0, 40, 700])
@pytest.mark.parametrize("heads,n_slots,slot_len", [
    ((8, 4), 66, 1),    # 132 rows: a last block of 4, one wave
    ((8, 4), 10, 16),   # 320 rows: a last block of 64, two waves
    ((8, 4), 97, 1),    # 194 rows: a last block of 66, three waves
    ((16, 4), 5, 8),    # 160 rows: 256-row block with three empty waves, or a last block of 32
    ((12, 4), 1, 11),   # 33 rows: one block, two waves
])
def test_partly_filled_blocks(heads, n_slots, slot_len, prefix_len):
    dev = require_gpu()
    wl = W.WORKLOADS["qwen0.6b"].replace(batch=2, n_q_heads=heads[0], n_kv_heads=heads[1], prefix_len=prefix_len,
                                         n_slots=n_slots, slot_len=slot_len, hidden=0, vocab=0, seed=94)
    xd, xf = attn_inputs_dev(wl, dev)
    for cross, pass_ in ((Z.CROSS_SLOT_CAUSAL, Z.PASS_AR_INFILL), (Z.CROSS_SLOT_NONE, Z.PASS_DIFFUSION)):
        say(f"slot_attn heads {heads} S={n_slots} L={slot_len} P={prefix_len} cross={cross}")
        out, lse = Z.slot_attn(xd["q"], xd["k_cache"], xd["v_cache"], xd["k_slot"], xd["v_slot"], n_slots, slot_len,
                               pass_=pass_, cross_slot=cross, prefix_len=prefix_len, prefix_splits=1)
        torch.cuda.synchronize()
        O, L = oracle.slot_attention(xf["q"], xf["k_cache"], xf["v_cache"], xf["k_slot"], xf["v_slot"], prefix_len,
                                     n_slots, slot_len, wl.scale, pass_, cross_slot=cross)
        check_attn(to_f64(out), to_f64(lse), O, L, "bf16", f"cross {cross}")


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("n_slots,slot_len", [
    (5, 8),    # 160 rows: a 256-row block with three empty waves
    (8, 8),    # 256 rows: one full block
    (11, 5),   # 220 rows: a wave of 28
    (17, 7),   # 476 rows: a last block with one empty wave
])
def test_partly_filled_wide_blocks(n_slots, slot_len, head_dim):
    """256-row blocks, of which the planner's own splits take 17 or more: ragged
    prefixes, the planner's splits, one and three."""
    dev = require_gpu()
    wl = W.WORKLOADS["qwen0.6b"].replace(batch=9, n_q_heads=8, n_kv_heads=2, head_dim=head_dim, prefix_len=330,
                                         n_slots=n_slots, slot_len=slot_len, hidden=0, vocab=0, seed=97)
    xd, xf = attn_inputs_dev(wl, dev)
    plan = Z._lib.slot_attn_plan(Z.slot_attn_desc(xd["q"], xd["k_cache"], xd["k_slot"], n_slots, slot_len, prefix_len=330))
    assert plan["rows_per_workgroup"] == 256
    plens = np.array([330, 329, 0, 64, 65, 1, 200, 128, 320], dtype=np.int32)
    for pass_, splits in ((Z.PASS_DIFFUSION, 0), (Z.PASS_AR_INFILL, 1), (Z.PASS_DIFFUSION, 3)):
        say(f"slot_attn 256-row blocks S={n_slots} L={slot_len} D={head_dim} pass={pass_} splits={splits}")
        out, lse = Z.slot_attn(xd["q"], xd["k_cache"], xd["v_cache"], xd["k_slot"], xd["v_slot"], n_slots, slot_len,
                               pass_=pass_, prefix_len=330, prefix_lens=torch.from_numpy(plens).to(dev),
                               prefix_splits=splits)
        torch.cuda.synchronize()
        O, L = oracle.slot_attention(xf["q"], xf["k_cache"], xf["v_cache"], xf["k_slot"], xf["v_slot"], plens, n_slots,
                                     slot_len, wl.scale, pass_)
        check_attn(to_f64(out), to_f64(lse), O, L, "bf16", f"pass {pass_} splits {splits}")
