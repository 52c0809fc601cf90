"""A store of two organisations (Sec. 7, fine-grained cache organisation: different chunks may be kept differently): the
first slots of a context hold bf16, the last ``n_slots_8bit`` hold 8-bit codes.  Which chunk goes where is the caller's
choice by slot id; every call must treat each slot by its own format, also when one call names both kinds.

bf16 slots must return their input bit for bit, 8-bit slots the oracle's quantiser; attention over a chunk list that
mixes both must match the oracle's attention over what the slots read back, to the bf16 bar."""
import numpy as np
import pytest
import torch

import oracle
from oracle import kv_fp8
from paper_2601_11553_amd import workloads as wl
from paper_2601_11553_amd.binding import Percache, PercacheError

from gpu_util import DEV, bf16, check_close, host

pytestmark = pytest.mark.gpu


def _ctx(D, C, n_slots, n8, Hkv=2, Hq=None, hidden=256, n_layers=1, max_pos=None):
    return Percache(n_layers=n_layers, hidden=hidden, n_q_heads=Hq or 2 * Hkv, n_kv_heads=Hkv, head_dim=D, n_slots=n_slots,
                    slot_capacity=C, max_pos=max_pos or 8 * C + 512, n_slots_8bit=n8, device=DEV)


def _reads_back(x, is8):
    x = wl.round_bf16(np.asarray(x, np.float32))
    return kv_fp8.round_trip(x) if is8 else x


@pytest.mark.parametrize("D", [64, 128])
def test_each_slot_keeps_its_own_format(D):
    g = np.random.default_rng(70 + D)
    Hkv, C, S, n8 = 2, 128, 6, 2                              # slots 0..3 bf16, slots 4, 5 8-bit
    pc = _ctx(D, C, S, n8, n_layers=2)
    data = {}
    for layer, slot, n in [(0, 1, 128), (0, 4, 100), (1, 5, 65), (1, 0, 7), (0, 5, 128)]:
        k = wl.round_bf16(g.standard_normal((Hkv, n, D)).astype(np.float32) * 3)
        v = wl.round_bf16(g.standard_normal((Hkv, n, D)).astype(np.float32))
        pc.percache_kv_put(layer, slot, bf16(k), bf16(v))
        data[(layer, slot)] = (k, v)
    for (layer, slot), (k, v) in data.items():
        kk, vv = pc.percache_kv_get(layer, slot)
        torch.cuda.synchronize()
        assert np.array_equal(host(kk), _reads_back(k, slot >= S - n8)), (layer, slot)
        assert np.array_equal(host(vv), _reads_back(v, slot >= S - n8)), (layer, slot)
    # one batched put that names slots of both kinds
    kb = wl.round_bf16(g.standard_normal((4, Hkv, 70, D)).astype(np.float32))
    vb = wl.round_bf16(g.standard_normal((4, Hkv, 70, D)).astype(np.float32))
    order = [5, 0, 4, 3]
    pc.percache_kv_put_batch(1, order, bf16(kb), bf16(vb))
    for i, slot in enumerate(order):
        kk, vv = pc.percache_kv_get(1, slot)
        torch.cuda.synchronize()
        assert np.array_equal(host(kk), _reads_back(kb[i], slot >= S - n8)), slot
        assert np.array_equal(host(vv), _reads_back(vb[i], slot >= S - n8)), slot
    # appends: exact on a bf16 slot, the oracle's re-quantisation rule on an 8-bit slot
    extra_k = wl.round_bf16(g.standard_normal((Hkv, 30, D)).astype(np.float32) * 5)
    extra_v = wl.round_bf16(g.standard_normal((Hkv, 30, D)).astype(np.float32))
    for slot in (0, 4):
        before_k, before_v = (host(t) for t in pc.percache_kv_get(1, slot))
        pc.percache_kv_append(1, slot, bf16(extra_k), bf16(extra_v))
        kk, vv = pc.percache_kv_get(1, slot)
        torch.cuda.synchronize()
        if slot >= S - n8:
            assert np.array_equal(host(kk), kv_fp8.append(before_k, extra_k))
            assert np.array_equal(host(vv), kv_fp8.append(before_v, extra_v))
        else:
            assert np.array_equal(host(kk), np.concatenate([before_k, extra_k], axis=1))
            assert np.array_equal(host(vv), np.concatenate([before_v, extra_v], axis=1))
    with pytest.raises(PercacheError) as e:
        pc.percache_kv_put(0, 6, bf16(kb[0]), bf16(vb[0]))
    assert e.value.status == -3
    pc.close()


@pytest.mark.parametrize("D", [64, 128])
def test_many_ragged_pieces_in_one_call(D):
    """More pieces than one launch takes, of 1 token up to a whole slot, at starts of every alignment, some not saved."""
    g = np.random.default_rng(80 + D)
    Hkv, C, S, n8 = 2, 128, 96, 40
    pc = _ctx(D, C, S, n8, max_pos=8192)
    lens = [1, 7, 8, 9, 63, 64, 65, 127, 128] + [int(x) for x in g.integers(1, C + 1, 69)]
    bounds = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(bounds[-1]) + 3
    slots = [int(x) for x in g.permutation(S)[:len(lens)]]
    slots[3] = slots[70] = -1
    k = wl.round_bf16(g.standard_normal((Hkv, T, D)).astype(np.float32) * 3)
    v = wl.round_bf16(g.standard_normal((Hkv, T, D)).astype(np.float32))
    pc.percache_kv_slice(0, bf16(k), bf16(v), bounds, slots)
    for i, slot in enumerate(slots):
        if slot < 0:
            continue
        kk, vv = pc.percache_kv_get(0, slot)
        torch.cuda.synchronize()
        for got, x in ((kk, k), (vv, v)):
            assert np.array_equal(host(got), _reads_back(x[:, bounds[i]:bounds[i + 1]], slot >= S - n8)), (i, lens[i], slot)
    pc.close()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 129])
def test_batches_of_both_formats_equal_batches_of_one(D, n):
    """Lists that name both kinds of slots (one launch for both), put and got, bit for bit what a list of each kind stores and returns."""
    g = torch.Generator(device=DEV)
    g.manual_seed(D + n)
    k, v = (torch.randn((5, 3, n, D), generator=g, device=DEV).bfloat16() for _ in range(2))
    slots = [6, 0, 4, 5, 2]                                   # slots 4 to 6 are 8-bit
    outs = []
    for lists in ([[0, 1, 2, 3, 4]], [[1, 4], [0, 2, 3]]):
        pc = _ctx(D, 192, 7, 3, Hkv=3)
        for i in lists:
            pc.percache_kv_put_batch(0, [slots[j] for j in i], k[i].contiguous(), v[i].contiguous())
        got = [torch.empty_like(k), torch.empty_like(v)]
        for i in lists:
            part = pc.percache_kv_get_batch(0, [slots[j] for j in i], n)
            for o, p in zip(got, part):
                o[i] = p
        torch.cuda.synchronize()
        outs.append(got)
        pc.close()
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    assert torch.equal(outs[0][0][[1, 4]], k[[1, 4]])


def test_config_limits_of_the_two_formats():
    from paper_2601_11553_amd import binding
    import ctypes
    lib = binding.load_library()
    ok = binding.Config(1, 256, 4, 2, 64, 6, 128, 1024, 10000.0, 0, 0, 0, 6)          # every slot 8-bit this way too
    assert lib.percache_arena_bytes(ctypes.byref(ok)) > 0
    for bad in (binding.Config(1, 256, 4, 2, 64, 6, 128, 1024, 10000.0, 0, 0, 0, 7),
                binding.Config(1, 256, 4, 2, 64, 6, 128, 1024, 10000.0, 0, 0, 0, -1),
                binding.Config(1, 256, 4, 2, 64, 6, 128, 1024, 10000.0, 0, 0, 1, 2)):
        assert lib.percache_arena_bytes(ctypes.byref(bad)) == 0


@pytest.mark.parametrize("D,t_fresh,G", [(128, 40, 2), (64, 70, 2), (128, 1, 4), (128, 200, 4)])
def test_attention_over_chunks_of_both_formats(D, t_fresh, G):
    """Chunk lists that interleave bf16 and 8-bit slots, ragged lengths, a fresh part; a query that names only bf16
    slots and one that names only 8-bit slots in the same batch; several key-axis partitions."""
    Hkv, C, S, n8 = 2, 192, 10, 4
    w = wl.make_prefill("mixed", 90 + D + t_fresh, "bf16", 256, G * Hkv, Hkv, D, 3, t_fresh, 4, C, S)
    w.slot_ids[0] = [7, 2, 9, 0]          # 8-bit, bf16, 8-bit, bf16
    w.slot_ids[1] = [1, 3, 4, 5]          # bf16 only
    w.slot_ids[2] = [6, 8, 9, 7]          # 8-bit only
    w.used_len[0] = [192, 100, 1, 65]
    w.used_len[1] = [64, 0, 190, 192]
    w.used_len[2] = [130, 192, 0, 7]
    pc = _ctx(D, C, S, n8, Hkv=Hkv, Hq=G * Hkv, max_pos=w.max_pos)
    store = {}
    for s_ in range(S):
        k, v = w.slot_kv(s_)
        pc.percache_kv_put(0, s_, bf16(k), bf16(v))
        store[s_] = (_reads_back(k, s_ >= S - n8), _reads_back(v, s_ >= S - n8))
    X, W = bf16(w.X), bf16(w.Wqkv)
    for n_splits in (0, 1, 3):
        q, kf, vf = pc.percache_qkv_rope(0, X, W, w.slot_ids, w.used_len)
        out = pc.percache_attention_reuse(0, q, kf, vf, w.slot_ids, w.used_len, n_splits=n_splits)
        torch.cuda.synchronize()
        for b in range(3):
            ids = [int(s_) for s_ in w.slot_ids[b]]
            sk = np.stack([store[s_][0] for s_ in ids])
            sv = np.stack([store[s_][1] for s_ in ids])
            O, _, _, _ = oracle.prefill_reuse(w.X[b], w.Wqkv, w.n_q_heads, w.n_kv_heads, D, w.rope_theta, sk, sv,
                                              np.arange(4, dtype=np.int32), w.used_len[b])
            check_close(host(out[b]), O, f"mixed slots D={D} T={t_fresh} G={G} splits={n_splits} b={b}")
    pc.close()


def test_stack_saves_chunks_into_slots_of_both_formats_and_reuses_them():
    """The population pass cuts the prompt's K/V into a bf16 slot, an 8-bit slot and a bf16 slot; the reuse pass over the
    fresh rows reads them back.  Reference: the oracle's full pass, its chunk K/V put through what each slot keeps."""
    from test_gpu_stack import EPS, check_hidden, dev_layers, oracle_block
    H, Hq, Hkv, D, F, C, n_c, Tf, L = 256, 4, 2, 64, 384, 64, 3, 40, 2
    total = n_c * C + Tf
    h0 = wl.round_bf16(np.random.default_rng(29).standard_normal((total, H)).astype(np.float32))
    Ws = [wl.stack_weights(29, l, H, Hq, Hkv, D, F) for l in range(L)]
    layers = dev_layers(Ws)
    pc = Percache(n_layers=L, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=8, slot_capacity=C, max_pos=total,
                  n_slots_8bit=3, device=DEV)
    slots = [1, 6, 4]                                     # slot 6 is 8-bit (slots 5, 6, 7 are)
    bounds = [c * C for c in range(n_c + 1)] + [total]
    pc.percache_stack_reuse(layers, F, EPS, bf16(h0[None]), save_bounds=bounds, save_slots=[slots + [-1]])
    reuse = pc.percache_stack_reuse(layers, F, EPS, bf16(h0[None, n_c * C:]), [slots])
    torch.cuda.synchronize()
    # oracle: full pass layer by layer keeps each layer's K/V; the reuse pass reads what the slots keep of them
    h_full, h_fresh = h0.copy(), h0[n_c * C:].copy()
    for l, W in enumerate(Ws):
        h_next, K, V = oracle_block(h_full, W, Hq, Hkv, D, 10000.0)
        sk = np.stack([_reads_back(K[:, c * C:(c + 1) * C], slots[c] >= 5) for c in range(n_c)])
        sv = np.stack([_reads_back(V[:, c * C:(c + 1) * C], slots[c] >= 5) for c in range(n_c)])
        h_fresh, _, _ = oracle_block(h_fresh, W, Hq, Hkv, D, 10000.0, sk, sv, np.arange(n_c, dtype=np.int32), [C] * n_c)
        h_full = h_next
    check_hidden(host(reuse[0]), h_fresh, "stack reuse over slots of both formats")
    pc.close()
