"""Selection, acceptance, append and reveal at the sizes where their work
splitting can go wrong (slot lengths around the lanes per slot, slot counts
around a wave, reveals around the 512 positions up to which keys are counted and
above which they are sorted): bit-exact against the oracle."""

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_helpers import require_gpu, say, to_dev

import paper_2609_19868_amd as Z

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,L", [(1, 1), (1, 63), (2, 64), (3, 65), (63, 2), (65, 3), (1024, 1), (5, 130), (33, 33)])
def test_commit_sizes(S, L):
    dev = require_gpu()
    rng = np.random.default_rng(100 * S + L)
    B, Hkv, D, C = 3, 2, 64, S * L + 10
    conf = rng.choice(np.array([0.1, 0.5, 0.95, np.nan, -np.inf, np.inf], np.float32), (B, S, L)) if S > 2 else \
        rng.random((B, S, L)).astype(np.float32)
    open_ = (rng.random((B, S)) < 0.8).astype(np.uint8)
    prob = rng.random((B, S, L)).astype(np.float32) ** np.float32(0.2)
    prob[rng.random((B, S, L)) < 0.05] = np.nan
    cd, od, pd = (torch.from_numpy(x).to(dev) for x in (conf, open_, prob))
    for rule, conf_rule in ((Z.SELECT_TOP_K, Z.SLOT_CONF_MEAN), (Z.SELECT_THRESHOLD, Z.SLOT_CONF_FIRST_TOKEN)):
        say(f"select_slots S={S} L={L} rule={rule}")
        got = Z.select_slots(cd, od, conf_rule=conf_rule, rule=rule, threshold=0.9, k=S)
        torch.cuda.synchronize()
        ref = oracle.select_slots(conf, open_, conf_rule=conf_rule, rule=rule, threshold=np.float32(0.9), k=S)
        for g, r in zip(got, ref):
            assert np.array_equal(g.cpu().numpy(), r)
        sel = got[1]
        for accept in (Z.ACCEPT_PREFIX, Z.ACCEPT_PER_TOKEN):
            say(f"verify_accept S={S} L={L} rule={accept}")
            acc = Z.verify_accept(pd, sel, 0.4, accept)
            torch.cuda.synchronize()
            ref = oracle.accept_tokens(prob, sel.cpu().numpy(), np.float32(0.4), accept)
            for g, r in zip(acc, ref):
                assert np.array_equal(g.cpu().numpy(), r)
            bits = [W.bf16_bits(rng.standard_normal(s, dtype=np.float32)) for s in ((B, Hkv, C, D),) * 2 + ((B, Hkv, S * L, D),) * 2]
            kc, vc, ks, vs = (to_dev(x, "bf16", dev) for x in bits)
            lens = torch.tensor([0, 10, C - 1], dtype=torch.int32, device=dev)
            say(f"kv_append S={S} L={L}")
            Z.kv_append(kc, vc, lens, ks, vs, acc[0], sel)
            torch.cuda.synchronize()
            kr, vr, lr = oracle.kv_append(bits[0], bits[1], [0, 10, C - 1], bits[2], bits[3], ref[0], sel.cpu().numpy())
            assert np.array_equal(lens.cpu().numpy(), lr)
            for g, r in ((kc, kr), (vc, vr)):
                assert np.array_equal(g.cpu().view(torch.int16).numpy().view(np.uint16), r)


@pytest.mark.parametrize("N", [1, 2, 3, 64, 127, 128, 129, 256, 257, 511, 512, 513, 1025, 4096, 8192])
def test_reveal_sizes(N):
    dev = require_gpu()
    rng = np.random.default_rng(N)
    B = 3
    conf = rng.random((B, N)).astype(np.float32)
    conf[rng.random((B, N)) < 0.3] = np.float32(0.25)  # ties
    odd = rng.random((B, N)) < 0.3  # NaN counts as -inf, -0 as 0
    conf[odd] = rng.choice(np.array([np.nan, np.inf, -np.inf, 0.0, -0.0], np.float32), odd.sum())
    mask = (rng.random((B, N)) < 0.7).astype(np.uint8)
    mask[0] = 1
    k = np.array([N, max(1, N // 3), 2], np.int32)
    for rule in (Z.REVEAL_CONFIDENCE, Z.REVEAL_RANDOM, Z.REVEAL_LEFTMOST):
        md = torch.from_numpy(mask.copy()).to(dev)
        say(f"mdm_reveal N={N} rule={rule}")
        order, n = Z.mdm_reveal(md, torch.from_numpy(k).to(dev), rule, conf=torch.from_numpy(conf).to(dev), seed=9, offset=4)
        torch.cuda.synchronize()
        ref = oracle.reveal(conf, mask.astype(bool), k, rule, seed=9, offset=4)
        assert np.array_equal(order.cpu().numpy(), ref[0]) and np.array_equal(n.cpu().numpy(), ref[1])
        left = mask.copy()
        for b in range(B):
            left[b, ref[0][b][:ref[1][b]]] = 0
        assert np.array_equal(md.cpu().numpy(), left)


@pytest.mark.parametrize("S,L", [(1, 1), (3, 21), (13, 5), (64, 4), (257, 1), (300, 3), (1024, 2)])
@pytest.mark.parametrize("B", [1023, 1024])
def test_accept_of_many_rows(B, S, L):
    """From 1024 rows a row has at most 256 threads: sizes around a wave, that
    limit and the slots; lists that end early, name ids past S and repeat."""
    dev = require_gpu()
    rng = np.random.default_rng(B + 10 * S + L)
    prob = rng.random((B, S, L)).astype(np.float32) ** np.float32(0.2)
    prob[rng.random((B, S, L)) < 0.05] = np.nan
    sel = rng.integers(-1 if S > 2 else 0, S + 2, (B, S)).astype(np.int32)
    sel[B // 2:][sel[B // 2:] < 0] = 0
    for rule in (Z.ACCEPT_PREFIX, Z.ACCEPT_PER_TOKEN):
        say(f"verify_accept B={B} S={S} L={L} rule={rule}")
        got = Z.verify_accept(torch.from_numpy(prob).to(dev), torch.from_numpy(sel).to(dev), 0.4, rule)
        torch.cuda.synchronize()
        for g, r in zip(got, oracle.accept_tokens(prob, sel, np.float32(0.4), rule)):
            assert np.array_equal(g.cpu().numpy(), r)
