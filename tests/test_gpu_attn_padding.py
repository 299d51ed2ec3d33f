"""Row blocks that are only partly filled: waves without a row, which only load,
with and without the heaviest-first order, against the float64 oracle.
Tolerances as in test_gpu_slot_attn.py."""

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
