"""Float32 slot_attn (MFMA tiles of 16 keys split over eight waves) against the
float64 oracle at the sizes where its tiling can go wrong.

Tolerance: relative L2 per (batch, head) 1e-5.  Scores of N(0, 1) inputs carry
about sqrt(D) * 2^-24 = 7e-7 absolute error each, which the softmax turns into
the same relative error per term; the value sums add sqrt(n) * 2^-24."""

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_helpers import attn_inputs_dev, check_attn, require_gpu, say, to_f64

import paper_2609_19868_amd as Z

pytestmark = pytest.mark.gpu

SHAPES = [
    # 16-row workgroups: fewer rows than one tile; one key past a tile; three heads per group
    ("one_row", dict(batch=1, n_q_heads=1, n_kv_heads=1, prefix_len=129, n_slots=1, slot_len=1)),
    ("rows17_p257", dict(batch=1, n_q_heads=1, n_kv_heads=1, prefix_len=257, kv_capacity=300, n_slots=17, slot_len=1)),
    ("g3_odd", dict(batch=2, n_q_heads=6, n_kv_heads=2, prefix_len=500, n_slots=7, slot_len=3)),
    ("d64_slots", dict(batch=1, n_q_heads=4, n_kv_heads=2, head_dim=64, prefix_len=175, n_slots=5, slot_len=9)),
    # 32-row workgroups: few keys, and many row blocks
    ("few_keys", dict(batch=1, n_q_heads=4, n_kv_heads=2, prefix_len=15, n_slots=3, slot_len=11)),
    ("few_keys_d64", dict(batch=1, n_q_heads=3, n_kv_heads=1, head_dim=64, prefix_len=1, n_slots=2, slot_len=17)),
    ("many_rows", dict(batch=8, n_q_heads=16, n_kv_heads=4, prefix_len=100, n_slots=8, slot_len=9)),
    ("many_rows_d64", dict(batch=8, n_q_heads=16, n_kv_heads=4, head_dim=64, prefix_len=100, n_slots=9, slot_len=8)),
    ("no_prefix", dict(batch=1, n_q_heads=2, n_kv_heads=1, prefix_len=0, n_slots=9, slot_len=25)),
]


@pytest.mark.parametrize("cross", [Z.CROSS_SLOT_NONE, Z.CROSS_SLOT_CAUSAL], ids=["none", "causal"])
@pytest.mark.parametrize("name,over", SHAPES, ids=[s[0] for s in SHAPES])
def test_f32_tiles(name, over, cross):
    dev = require_gpu()
    wl = W.WORKLOADS["qwen0.6b"].replace(**over, dtype="f32", hidden=0, vocab=0, seed=91)
    xd, xf = attn_inputs_dev(wl, dev)
    plens = (wl.prefix_len - 3 * np.arange(wl.batch)).clip(0).astype(np.int32)
    lens = torch.from_numpy(plens).to(dev)
    for pass_ in (Z.PASS_DIFFUSION, Z.PASS_AR_INFILL):
        say(f"slot_attn f32 {name} cross={cross} pass={pass_}")
        cache = wl.capacity > 0
        out, lse = Z.slot_attn(xd["q"], xd["k_cache"] if cache else None, xd["v_cache"] if cache else None,
                               xd["k_slot"], xd["v_slot"], wl.n_slots, wl.slot_len, pass_=pass_, cross_slot=cross,
                               prefix_len=wl.prefix_len, prefix_lens=lens)
        torch.cuda.synchronize()
        O, L = oracle.slot_attention(xf["q"], xf["k_cache"], xf["v_cache"], xf["k_slot"], xf["v_slot"], plens,
                                     wl.n_slots, wl.slot_len, wl.scale, pass_, cross_slot=cross)
        assert check_attn(to_f64(out), to_f64(lse), O, L, "f32", f"{name} cross={cross}") <= 1e-5


@pytest.mark.parametrize("batch", [6, 7], ids=["two_workgroups_a_block", "one"])
def test_f32_around_the_shared_block_limit(batch):
    """Five blocks of 16 rows per KV head (75 rows, the last block partly filled):
    120 blocks are shared by two workgroups each, 140 are not."""
    dev = require_gpu()
    wl = W.WORKLOADS["qwen0.6b"].replace(batch=batch, n_q_heads=12, n_kv_heads=4, prefix_len=130, n_slots=5, slot_len=5,
                                         dtype="f32", hidden=0, vocab=0, seed=95)
    xd, xf = attn_inputs_dev(wl, dev)
    plan = Z._lib.slot_attn_plan(Z.slot_attn_desc(xd["q"], xd["k_cache"], xd["k_slot"], 5, 5, prefix_len=130))
    assert plan["rows_per_workgroup"] == 16 and plan["workgroups"] == {6: 240, 7: 140}[batch]
    say(f"slot_attn f32 B={batch}")
    out, lse = Z.slot_attn(xd["q"], xd["k_cache"], xd["v_cache"], xd["k_slot"], xd["v_slot"], 5, 5, prefix_len=130)
    torch.cuda.synchronize()
    O, L = oracle.slot_attention(xf["q"], xf["k_cache"], xf["v_cache"], xf["k_slot"], xf["v_slot"], 130, 5, 5, wl.scale,
                                 oracle.PASS_DIFFUSION)
    assert check_attn(to_f64(out), to_f64(lse), O, L, "f32", f"B={batch}") <= 1e-5


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("prefix_len", [20, 200], ids=["rows32", "rows16"])
def test_f32_values_a_row_does_not_see_do_not_reach_it(head_dim, prefix_len):
    """NaN and infinite keys and values in other slots, and past a row's own
    prefix, leave a row's result as it is without them."""
    dev = require_gpu()
    wl = W.WORKLOADS["qwen0.6b"].replace(batch=1, n_q_heads=2, n_kv_heads=1, head_dim=head_dim, prefix_len=prefix_len,
                                         n_slots=5, slot_len=4, dtype="f32", hidden=0, vocab=0, seed=92)
    xd, _ = attn_inputs_dev(wl, dev)
    lens = torch.tensor([wl.prefix_len - 3], dtype=torch.int32, device=dev)

    def run():
        out, lse = Z.slot_attn(xd["q"], xd["k_cache"], xd["v_cache"], xd["k_slot"], xd["v_slot"], wl.n_slots,
                               wl.slot_len, prefix_len=wl.prefix_len, prefix_lens=lens)
        torch.cuda.synchronize()
        return out, lse

    say(f"slot_attn f32 unseen values D={head_dim} P={prefix_len}")
    clean_out, clean_lse = run()
    for x in (xd["k_cache"], xd["v_cache"]):
        x[:, :, wl.prefix_len - 3:] = float("nan")
    xd["k_slot"][:, :, 8:12, 5] = float("nan")  # slot 2
    xd["v_slot"][:, :, 8:12] = float("inf")
    xd["v_slot"][:, :, 9, 3] = float("nan")
    out, lse = run()
    keep = [t for t in range(20) if not 8 <= t < 12]
    # tiles with such values are summed key by key, in another order: 1e-5 as above
    assert (out[:, :, keep] - clean_out[:, :, keep]).norm() <= 1e-5 * clean_out[:, :, keep].norm()
    assert torch.equal(lse[:, :, keep], clean_lse[:, :, keep])
    assert out[:, :, 8:12].isnan().all()


@pytest.mark.parametrize("name,over,one_wave", [
    ("blocks512_one_tile", dict(batch=64, prefix_len=0, n_slots=3, slot_len=5), True),
    ("blocks512_two_tiles_d64", dict(batch=64, head_dim=64, prefix_len=31, n_slots=1, slot_len=1), True),
    ("blocks512_33_keys", dict(batch=64, prefix_len=32, n_slots=1, slot_len=1), False),
    ("blocks504", dict(batch=63, prefix_len=0, n_slots=1, slot_len=1), False),
    ("blocks1024_causal", dict(batch=64, head_dim=64, prefix_len=80, n_slots=32, slot_len=1), True),
    ("blocks1024_512_keys", dict(batch=128, prefix_len=510, n_slots=2, slot_len=1), True),
    ("blocks1024_513_keys", dict(batch=128, prefix_len=511, n_slots=2, slot_len=1), False),
])
def test_f32_many_blocks_take_one_wave_each(name, over, one_wave):
    """Workgroups of one wave from 1024 blocks of 16 rows (512 with one or two key
    tiles): both sides of the lines, 8/8 heads, ragged prefixes."""
    dev = require_gpu()
    wl = W.WORKLOADS["qwen0.6b"].replace(**over, n_q_heads=8, n_kv_heads=8, dtype="f32", hidden=0, vocab=0, seed=96)
    xd, xf = attn_inputs_dev(wl, dev)
    cross = Z.CROSS_SLOT_CAUSAL if "causal" in name else Z.CROSS_SLOT_NONE
    S, L, P = wl.n_slots, wl.slot_len, wl.prefix_len
    cache = [xd["k_cache"], xd["v_cache"]] if P else [None, None]
    plan = Z._lib.slot_attn_plan(Z.slot_attn_desc(xd["q"], cache[0], xd["k_slot"], S, L, cross_slot=cross, prefix_len=P))
    blocks16 = wl.batch * 8 * -(-S * L // 16)
    assert (plan["rows_per_workgroup"] == 16 and plan["workgroups"] == blocks16) == one_wave
    plens = (P - 7 * np.arange(wl.batch)).clip(0).astype(np.int32)
    say(f"slot_attn f32 {name}")
    out, lse = Z.slot_attn(xd["q"], *cache, xd["k_slot"], xd["v_slot"], S, L, cross_slot=cross, prefix_len=P,
                           prefix_lens=torch.from_numpy(plens).to(dev))
    torch.cuda.synchronize()
    O, Ls = oracle.slot_attention(xf["q"], xf["k_cache"], xf["v_cache"], xf["k_slot"], xf["v_slot"], plens, S, L,
                                  wl.scale, oracle.PASS_DIFFUSION, cross_slot=cross)
    assert check_attn(to_f64(out), to_f64(lse), O, Ls, "f32", name) <= 1e-5
