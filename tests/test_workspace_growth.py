"""Workspace sizes as a call grows: a buffer kept for the largest call (the
longest prefix, the most sequences, the most rows) serves every smaller one."""

import pytest

from paper_2609_19868_amd import _lib


def attn_bytes(B, heads, P, S, L, D=128):
    return _lib.slot_attn_workspace_size(_lib.SlotAttnDesc(
        batch=B, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=D, prefix_len=P, kv_capacity=P, n_slots=S,
        slot_len=L, softmax_scale=0.088, pass_=0, cross_slot=0, dtype=_lib.DTYPE_BF16, prefix_splits=0))


@pytest.mark.parametrize("B,heads,S,L,D", [(1, (16, 8), 8, 8, 128), (1, (32, 8), 8, 16, 128), (3, (16, 8), 8, 16, 128),
                                           (2, (12, 4), 5, 7, 64), (5, (16, 8), 8, 8, 64), (1, (8, 8), 1, 1, 128)])
def test_attention_workspace_serves_every_shorter_prefix(B, heads, S, L, D):
    sizes = [attn_bytes(B, heads, P, S, L, D) for P in range(64, 40001, 64)]
    assert all(a <= b for a, b in zip(sizes, sizes[1:]))


@pytest.mark.parametrize("heads,S,L,P,fewer,more", [
    ((16, 8), 8, 8, 4096, 1, 3), ((16, 8), 8, 8, 16384, 2, 5), ((32, 8), 8, 16, 16384, 1, 3),
    ((32, 8), 8, 16, 30000, 2, 3), ((16, 8), 8, 8, 2048, 8, 9)])
def test_attention_workspace_serves_fewer_sequences(heads, S, L, P, fewer, more):
    assert attn_bytes(more, heads, P, S, L) >= attn_bytes(fewer, heads, P, S, L) > 0


def test_attention_workspace_serves_fewer_draft_tokens():
    # 129 tokens of two heads make three row blocks a head, 128 make one
    assert attn_bytes(1, (16, 8), 16384, 1, 129) >= attn_bytes(1, (16, 8), 16384, 1, 128) > 0


@pytest.mark.parametrize("vocab", [100, 300, 5000, 32000, 151936])
@pytest.mark.parametrize("size", [_lib.slot_confidence_workspace_size, _lib.slot_sample_workspace_size])
def test_float32_head_workspace_serves_fewer_rows(size, vocab):
    sizes = [size(_lib.ConfDesc(n_rows=M, hidden=64, vocab=vocab, dtype=_lib.DTYPE_F32)) for M in range(1, 2000)]
    assert all(a <= b for a, b in zip(sizes, sizes[1:]))
