"""Decoding steps over [reused chunks ; the prompt's own K/V ; generated tokens] through the slot gather, and the slot
append they rely on, through the C ABI.

There is no language-model head here: the "generated token" fed to step i is a seeded row of hidden state.  The reference
for every step is a plain prefill of the whole sequence so far (GPU, no cache) and, at the last step, the CPU oracle's stack for every query of the batch."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_11553_amd import workloads as wl
from paper_2601_11553_amd.binding import Percache, PercacheError, _host_i32

from gpu_util import DEV, bf16, check_close, host
from test_gpu_stack import EPS, check_hidden, dev_layers, oracle_block

pytestmark = pytest.mark.gpu


def test_kv_append_equals_put_of_the_concatenation():
    Hkv, D, C = 2, 128, 192
    pc = Percache(n_layers=1, hidden=256, n_q_heads=2, n_kv_heads=Hkv, head_dim=D, n_slots=3, slot_capacity=C, max_pos=256, device=DEV)
    g = np.random.default_rng(1)
    k = bf16(g.standard_normal((Hkv, 150, D)))
    v = bf16(g.standard_normal((Hkv, 150, D)))
    pc.percache_kv_put(0, 0, k, v)
    cuts = [0, 37, 38, 64, 65, 129, 150]                      # appends that start / end inside and on block borders
    for lo, hi in zip(cuts[:-1], cuts[1:]):
        pc.percache_kv_append(0, 1, k[:, lo:hi].contiguous(), v[:, lo:hi].contiguous())
        assert pc.percache_kv_len(0, 1) == hi
    ka, va = pc.percache_kv_get(0, 1)
    torch.cuda.synchronize()
    assert torch.equal(ka, k) and torch.equal(va, v)
    with pytest.raises(PercacheError) as e:
        pc.percache_kv_append(0, 1, k[:, :43].contiguous(), v[:, :43].contiguous())   # 150 + 43 > 192
    assert e.value.status == -4 and pc.percache_kv_len(0, 1) == 150
    with pytest.raises(PercacheError) as e:                                           # tensors that are not 16-byte aligned
        pc.percache_kv_append(0, 2, k.reshape(-1)[1:1 + Hkv * 2 * D].view(Hkv, 2, D), v[:, :2].contiguous())
    assert e.value.status == -1 and pc.percache_kv_len(0, 2) == 0
    # attention over the appended slot equals attention over the slot written at once (same padding behaviour)
    q = bf16(g.standard_normal((1, 2, 5, D)))
    kf = bf16(g.standard_normal((1, Hkv, 5, D)))
    vf = bf16(g.standard_normal((1, Hkv, 5, D)))
    a0 = pc.percache_attention_reuse(0, q, kf, vf, [[0]])
    a1 = pc.percache_attention_reuse(0, q, kf, vf, [[1]])
    torch.cuda.synchronize()
    assert torch.equal(a0, a1)


@pytest.mark.parametrize("batch,D,Hq", [(1, 64, 4), (3, 64, 4), (2, 128, 8), (1, 128, 2)])
def test_decode_steps_match_full_prefill(batch, D, Hq):
    _decode_case(batch, D, Hq, 2, 256, 384, 2, 64, 2, 20, 6, 40 + batch, full_slot=True)


@pytest.mark.parametrize("seed", list(range(12)))
def test_seeded_random_decode_shapes(seed):
    """Shapes drawn from a seed: batch, head size, GQA ratio, widths, layers, chunk count (none included) and capacity,
    prompt length, number of steps (the sequence slot ends exactly full in some draws)."""
    g = np.random.default_rng(9000 + seed)
    D = int(g.choice([64, 128]))
    Hkv = int(g.choice([1, 2, 4]))
    Hq = Hkv * int(g.choice([1, 2, 4]))
    while ((Hq + 2 * Hkv) * D) % 128:
        Hq += Hkv
    C = int(g.choice([64, 128]))
    n_steps = int(g.integers(1, 6))
    t_prompt = int(g.choice([1, 2, 31, C - n_steps]))
    _decode_case(int(g.integers(1, 4)), D, Hq, Hkv, int(g.choice([128, 256, 384])), int(g.choice([192, 448])),
                 int(g.integers(1, 3)), C, int(g.integers(0, 4)), t_prompt, n_steps, 9100 + seed, full_slot=False)


def _decode_case(batch, D, Hq, Hkv, H, F, L, C, n_c, t_prompt, n_steps, seed, full_slot):
    Ws = [wl.stack_weights(31, l, H, Hq, Hkv, D, F) for l in range(L)]
    layers = dev_layers(Ws)
    n_slots = batch * (n_c + 1)
    pc = Percache(n_layers=L, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=n_slots, slot_capacity=C,
                  max_pos=n_c * C + C, device=DEV)
    plain = Percache(n_layers=L, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=1, slot_capacity=C,
                     max_pos=n_c * C + C, device=DEV)
    g = np.random.default_rng(seed)
    total = n_c * C + t_prompt + n_steps
    seqs = wl.round_bf16(g.standard_normal((batch, total, H)).astype(np.float32))   # chunks, prompt, then the fed tokens
    chunk_slots = [[b * (n_c + 1) + c for c in range(n_c)] for b in range(batch)]
    seq_slots = [b * (n_c + 1) + n_c for b in range(batch)]
    # population: each query's chunks and prompt are prefilled once; chunk K/V -> chunk slots, prompt K/V -> the sequence slot
    bounds = [c * C for c in range(n_c + 1)] + [n_c * C + t_prompt]
    pc.percache_stack_reuse(layers, F, EPS, bf16(seqs[:, :n_c * C + t_prompt]), save_bounds=bounds,
                            save_slots=[chunk_slots[b] + [seq_slots[b]] for b in range(batch)])
    for step in range(n_steps):
        pos = n_c * C + t_prompt + step
        x = bf16(seqs[:, pos:pos + 1])
        chains = [chunk_slots[b] + [seq_slots[b]] for b in range(batch)]
        out = pc.percache_stack_decode(layers, F, EPS, x, chains, seq_slots)
        ref = plain.percache_stack_reuse(layers, F, EPS, bf16(seqs[:, :pos + 1]))
        torch.cuda.synchronize()
        for b in range(batch):
            assert pc.percache_kv_len(0, seq_slots[b]) == t_prompt + step + 1 == pc.percache_kv_len(L - 1, seq_slots[b])
        check_hidden(host(out[:, 0]), host(ref[:, -1]), f"decode step {step} (batch {batch} D {D} heads {Hq}/{Hkv} H {H} layers {L} "
                     f"chunks {n_c}x{C} prompt {t_prompt}) vs full prefill", rel_max=2.0 ** -5)
    for b in range(batch):
        h = seqs[b]
        for W in Ws:
            h, _, _ = oracle_block(h, W, Hq, Hkv, D, 10000.0)
        check_hidden(host(out[b, 0]), h[-1], f"last decode step vs oracle stack, query {b}")
    if not full_slot:
        return
    # a sequence slot that is full refuses the step and nothing changes
    filler = bf16(g.standard_normal((Hkv, C - t_prompt - n_steps, D)))
    for l in range(L):
        pc.percache_kv_append(l, seq_slots[0], filler, filler)
    with pytest.raises(PercacheError) as e:
        pc.percache_stack_decode(layers, F, EPS, x, chains, seq_slots)
    assert e.value.status == -4 and pc.percache_kv_len(0, seq_slots[-1]) == t_prompt + n_steps + (C - t_prompt - n_steps if batch == 1 else 0)


@pytest.mark.parametrize("D,G,T,slots,n_chunks,n_splits", [
    (128, 2, 1, "bf16", 6, 0), (128, 1, 16, "bf16", 3, 2), (128, 3, 6, "8bit", 5, 0), (128, 4, 8, "mixed", 7, 3), (64, 7, 1, "mixed", 70, 0),
    (64, 7, 4, "bf16", 5, 4), (64, 1, 32, "8bit", 2, 0), (128, 2, 9, "mixed", 66, 0), (128, 16, 1, "8bit", 4, 2), (64, 4, 1, "bf16", 0, 0),
])
def test_attention_of_very_few_rows(D, G, T, slots, n_chunks, n_splits):
    """The kernel for at most 32 rows per kv head: one and two blocks of 16 rows, several fresh tokens (causal among them, over
    both blocks of 16 fresh keys), chunks of 1 to 128 tokens and unused ones, lists past 64 chunks, each slot format, with the
    key axis cut as the library chooses and as forced; through the fused call (which starts from the projection's sums) and
    through the attention call alone."""
    g = np.random.default_rng(7000 + D + 16 * G + T)
    Hkv, H, C, B = 2, 128, 128, 2
    Hq, n_slots = G * Hkv, max(2, 2 * n_chunks)
    kind = dict(kv_fp8=True) if slots == "8bit" else dict(n_slots_8bit=n_slots // 2) if slots == "mixed" else {}
    pc = Percache(n_layers=1, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=n_slots, slot_capacity=C,
                  max_pos=n_chunks * C + T, device=DEV, **kind)
    ids = g.permutation(n_slots)[:B * n_chunks].reshape(B, n_chunks).astype(np.int32)
    used = np.where(g.random((B, n_chunks)) < 0.2, 0, g.integers(1, C + 1, (B, n_chunks))).astype(np.int32)
    for s in ids.reshape(-1):
        pc.percache_kv_put(0, int(s), bf16(g.standard_normal((Hkv, C, D))), bf16(g.standard_normal((Hkv, C, D))))
    W = wl.round_bf16(g.standard_normal(((Hq + 2 * Hkv) * D, H)).astype(np.float32) * np.float32(0.1))
    X = wl.round_bf16(g.standard_normal((B, T, H)).astype(np.float32))
    kf, vf = (torch.empty((B, Hkv, T, D), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    fused = pc.percache_prefill_reuse(0, bf16(X), bf16(W), ids, used, k_fresh_out=kf, v_fresh_out=vf)
    q, k1, v1 = pc.percache_qkv_rope(0, bf16(X), bf16(W), ids, used)
    alone = pc.percache_attention_reuse(0, q, k1, v1, ids, used, n_splits=n_splits)
    torch.cuda.synchronize()
    for b in range(B):
        kv = [pc.percache_kv_get(0, int(s)) for s in ids[b]]
        sk = np.stack([host(k) for k, _ in kv]) if kv else np.zeros((0, Hkv, C, D), np.float32)
        sv = np.stack([host(v) for _, v in kv]) if kv else sk.copy()
        ref, _, _, _ = oracle.prefill_reuse(X[b], W, Hq, Hkv, D, 10000.0, sk, sv, np.arange(n_chunks, dtype=np.int32), used[b])
        check_close(host(fused[b]), ref, f"fused D={D} G={G} T={T} {slots} query {b}")
        check_close(host(alone[b]), ref, f"attention alone, n_splits {n_splits}, query {b}")
        # (the two paths round the same fp32 sums, taken in another order over the slices)
        assert np.abs(host(kf[b]) - host(k1[b])).max() <= 2.0 ** -7 * np.abs(host(k1[b])).max()
        assert np.abs(host(vf[b]) - host(v1[b])).max() <= 2.0 ** -7 * np.abs(host(v1[b])).max()
    pc.close()


@pytest.mark.parametrize("slots,T", [("bf16", 1), ("bf16", 5), ("mixed", 3), ("8bit", 1)])
def test_decode_step_appends_over_a_block_border(slots, T):
    """Decoding steps that fill, cross and open 64-key blocks of the sequence slots, with queries that append nothing and
    queries of both slot formats in one batch: every slot must read back what separate appends of the same K/V give."""
    D, Hq, Hkv, H, F, C, B = 128, 4, 2, 128, 64, 192, 3
    layer = dev_layers([wl.stack_weights(33, 0, H, Hq, Hkv, D, F)])[0]
    kind = dict(kv_fp8=True) if slots == "8bit" else dict(n_slots_8bit=2) if slots == "mixed" else {}
    pc, twin = (Percache(n_layers=1, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=6, slot_capacity=C, max_pos=C,
                         device=DEV, **kind) for _ in range(2))
    g = np.random.default_rng(8000 + T)
    own, start = [0, 4, 5], [63, 0, 64 - T]             # (mixed: slots 4 and 5 are 8-bit)
    for b in (0, 2):
        k, v = bf16(g.standard_normal((Hkv, start[b], D))), bf16(g.standard_normal((Hkv, start[b], D)))
        for p in (pc, twin):
            p.percache_kv_put(0, own[b], k, v)
    for step in range(3):
        have = [pc.percache_kv_len(0, s) for s in own]
        n_chunks, ids = [int(n > 0) for n in have], [[s if n else 0] for s, n in zip(own, have)]
        append = [own[0], -1 if step == 1 else own[1], own[2]]
        x = bf16(g.standard_normal((B, T, H)))
        pc.percache_stack_decode([layer], F, EPS, x, ids, append, n_chunks=n_chunks)
        n = (x.float() * torch.rsqrt((x.float() ** 2).mean(-1, keepdim=True) + EPS) * layer["gain1"].float()).bfloat16()
        _, k1, v1 = twin.percache_qkv_rope(0, n, layer["wqkv"], ids, None, n_chunks)
        for b in range(B):
            if append[b] < 0:
                assert pc.percache_kv_len(0, own[b]) == have[b]
                continue
            twin.percache_kv_append(0, own[b], k1[b], v1[b])
            assert pc.percache_kv_len(0, own[b]) == have[b] + T
            got, ref = pc.percache_kv_get(0, own[b]), twin.percache_kv_get(0, own[b])
            torch.cuda.synchronize()
            is8 = slots == "8bit" or (slots == "mixed" and own[b] >= 4)
            for x_got, x_ref in zip(got, ref):
                # the two differ by a rounding of the normed row and one of the result (2^-8 each way of the largest value,
                # at most two steps), an 8-bit code then by at most one step of 1/8
                assert (x_got.float() - x_ref.float()).abs().max() <= (2.0 ** -3 if is8 else 2.0 ** -6) * x_ref.float().abs().max(), (step, b)
                if not is8:
                    assert torch.equal(x_got[:, :have[b]], x_ref[:, :have[b]])
            twin.percache_kv_put(0, own[b], *got)       # the twin goes on from the step's own values
    pc.close()
    twin.close()


@pytest.mark.parametrize("D,G,T,tiles", [(128, 2, 2, 7), (64, 7, 1, 4), (128, 3, 4, 12), (128, 4, 1, 36)])   # (36: past two tiles a workgroup, cut to one round)
def test_partitions_cost_no_precision(D, G, T, tiles):
    """Cutting the key axis of a few-row call is the library's choice, not the caller's: the merged result must be as close to
    attention in 64 bits as one partition's.  Both round the probabilities and the result to bf16 once; partials kept in bf16
    add a rounding of about the result's own size (a quarter more root-mean-square error).  Over the 8000 to 25000 outputs
    here two equally good results differ by 2 to 3 % in it."""
    g = np.random.default_rng(7700 + D + tiles)
    Hkv, C, B = 4, 64, 8 if G == 7 else 4
    Hq = G * Hkv
    pc = Percache(n_layers=1, hidden=128, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=B * tiles, slot_capacity=C,
                  max_pos=tiles * C + T, device=DEV)
    kv = torch.from_numpy(g.standard_normal((2, B, tiles, Hkv, C, D)).astype(np.float32)).to(DEV, torch.bfloat16)
    for b in range(B):
        for t in range(tiles):
            pc.percache_kv_put(0, b * tiles + t, kv[0, b, t], kv[1, b, t])
    ids = np.arange(B * tiles, dtype=np.int32).reshape(B, tiles)
    q, kf, vf = (bf16(g.standard_normal((B, n, T, D))) for n in (Hq, Hkv, Hkv))
    auto, one = (pc.percache_attention_reuse(0, q, kf, vf, ids, n_splits=n) for n in (0, 1))
    torch.cuda.synchronize()
    k, v = (torch.cat([x.double().permute(0, 2, 1, 3, 4).reshape(B, Hkv, tiles * C, D), f.double()], 2).repeat_interleave(G, 1).cpu()
            for x, f in zip(kv, (kf, vf)))
    s = (q.double().cpu() @ k.transpose(2, 3)) / D ** 0.5
    s += torch.triu(torch.full((T, tiles * C + T), float("-inf"), dtype=torch.float64), diagonal=tiles * C + 1)
    ref = (s.softmax(-1) @ v).transpose(1, 2).reshape(B, T, Hq * D)
    e_auto, e_one = (((x.double().cpu() - ref).norm() / ref.norm()).item() for x in (auto, one))
    assert not torch.equal(auto, one)                 # (the library does cut these)
    assert e_auto <= 1.06 * e_one, (e_auto, e_one)
    pc.close()


@pytest.mark.parametrize("slots,T", [("8bit", 1), ("8bit", 24), ("mixed", 1), ("mixed", 24), ("mixed", 32)])
def test_long_calls_with_two_workgroups_per_cu(slots, T):
    """More workgroups than CUs over 8-bit and mixed slots: rings of two stages, row blocks finished one after the other behind
    the first tiles, ragged chunks (64 kv heads, partitions of 4 and 5 tiles)."""
    g = np.random.default_rng(7800 + T)
    Hkv, D, H, C, n_chunks = 64, 128, 128, 128, 12
    kind = dict(kv_fp8=True) if slots == "8bit" else dict(n_slots_8bit=n_chunks // 2)
    pc = Percache(n_layers=1, hidden=H, n_q_heads=Hkv, n_kv_heads=Hkv, head_dim=D, n_slots=n_chunks, slot_capacity=C,
                  max_pos=n_chunks * C + T, device=DEV, **kind)
    ids = g.permutation(n_chunks).astype(np.int32)[None]
    used = np.where(np.arange(n_chunks) % 5 == 4, 1, g.integers(65, C + 1, n_chunks)).astype(np.int32)[None]
    for s in range(n_chunks):
        pc.percache_kv_put(0, s, bf16(g.standard_normal((Hkv, C, D))), bf16(g.standard_normal((Hkv, C, D))))
    W = wl.round_bf16(g.standard_normal((3 * Hkv * D, H)).astype(np.float32) * np.float32(0.1))
    X = wl.round_bf16(g.standard_normal((1, T, H)).astype(np.float32))
    kf, vf = (torch.empty((1, Hkv, T, D), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    fused = pc.percache_prefill_reuse(0, bf16(X), bf16(W), ids, used, k_fresh_out=kf, v_fresh_out=vf)
    q, k1, v1 = pc.percache_qkv_rope(0, bf16(X), bf16(W), ids, used)
    alone = pc.percache_attention_reuse(0, q, k1, v1, ids, used)
    torch.cuda.synchronize()
    sk, sv = (np.stack(x) for x in zip(*[[host(t) for t in pc.percache_kv_get(0, int(s))] for s in ids[0]]))
    ref, _, _, _ = oracle.prefill_reuse(X[0], W, Hkv, Hkv, D, 10000.0, sk, sv, np.arange(n_chunks, dtype=np.int32), used[0])
    check_close(host(fused[0]), ref, f"fused {slots} T={T}")
    check_close(host(alone[0]), ref, f"attention alone {slots} T={T}")
    for got, want in ((kf, k1), (vf, v1)):   # (the same fp32 sums, taken in another order over the slices)
        assert np.abs(host(got) - host(want)).max() <= 2.0 ** -7 * np.abs(host(want)).max()
    pc.close()


@pytest.mark.parametrize("D,G,slots", [(128, 2, "bf16"), (64, 7, "bf16"), (128, 20, "bf16"), (128, 3, "mixed"), (64, 1, "8bit")])
def test_what_stands_behind_the_used_length_takes_no_part(D, G, slots):
    """Tokens of a chunk beyond the used length hold infinities and NaN (8-bit slots: NaN codes): the few-row attention over the
    tokens in front of them is finite and right."""
    g = np.random.default_rng(7900 + D + G)
    Hkv, C, H, n_chunks = 2, 128, 128, 4
    Hq = G * Hkv
    kind = dict(kv_fp8=True) if slots == "8bit" else dict(n_slots_8bit=2) if slots == "mixed" else {}
    pc = Percache(n_layers=1, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=n_chunks, slot_capacity=C, max_pos=n_chunks * C + 1,
                  device=DEV, **kind)
    used = np.array([[33, 64, 97, 1]], np.int32)
    k, v = (wl.round_bf16(g.standard_normal((n_chunks, Hkv, C, D)).astype(np.float32)) for _ in range(2))
    for s in range(n_chunks):
        stale = np.arange(C) >= used[0, s]
        kk, vv = k[s].copy(), v[s].copy()
        # (a block of an 8-bit slot shares one scale: there only NaN, which leaves the scale alone)
        kk[:, stale], vv[:, stale] = np.nan, np.nan if slots != "bf16" else np.inf
        pc.percache_kv_put(0, s, bf16(kk), bf16(vv))
    q, kf, vf = (bf16(g.standard_normal((1, n, 1, D))) for n in (Hq, Hkv, Hkv))
    out = pc.percache_attention_reuse(0, q, kf, vf, np.arange(n_chunks, dtype=np.int32)[None], used)
    torch.cuda.synchronize()
    got = [pc.percache_kv_get(0, s) for s in range(n_chunks)]
    ck, cv = (torch.cat([host_t.double().cpu()[:, :used[0, s]] for s, host_t in enumerate(x)] + [f[0].double().cpu()], 1)
              for x, f in zip(zip(*got), (kf, vf)))
    p = ((q[0].double().cpu() @ ck.repeat_interleave(G, 0).transpose(1, 2)) / D ** 0.5).softmax(-1)
    check_close(host(out[0]).reshape(-1), (p @ cv.repeat_interleave(G, 0)).reshape(-1).numpy(), f"D={D} G={G} {slots}")
    pc.close()


def test_a_query_that_appends_what_is_not_a_number_spoils_no_other():
    """Two queries share a prefix slot in one decoding step; the first appends to it, and its hidden row is infinite: its own
    output is not a number, the other's is what it is without the first."""
    D, Hq, Hkv, H, F, C = 128, 4, 2, 128, 64, 128
    layer = dev_layers([wl.stack_weights(34, 0, H, Hq, Hkv, D, F)])[0]
    g = np.random.default_rng(8100)
    k, v = (bf16(g.standard_normal((Hkv, 77, D))) for _ in range(2))
    x = bf16(g.standard_normal((2, 1, H)))
    outs = []
    for bad in (False, True):
        pc = Percache(n_layers=1, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=2, slot_capacity=C, max_pos=C, device=DEV)
        pc.percache_kv_put(0, 0, k, v)
        h = x.clone()
        if bad:
            h[0] = float("inf")
        outs.append(pc.percache_stack_decode([layer], F, EPS, h, [[0], [0]], [0, -1]).clone())
        torch.cuda.synchronize()
        assert pc.percache_kv_len(0, 0) == 78
        pc.close()
    assert not torch.isfinite(outs[1][0]).all()
    assert torch.equal(outs[0][1], outs[1][1])


@pytest.mark.parametrize("D,heads,B,T,which,slots", [
    (128, (16, 8), 2, 1, "qk", "bf16"), (128, (16, 8), 1, 3, "qk bias", "bf16"), (128, (24, 8), 1, 9, "qk bias", "bf16"), (64, (14, 2), 3, 1, "qk bias", "bf16"),
    (64, (14, 2), 2, 4, "qk", "bf16"), (128, (16, 8), 2, 1, "q", "bf16"), (64, (8, 4), 2, 5, "k bias", "bf16"), (128, (16, 8), 2, 2, "qk bias", "8bit"),
    (64, (14, 2), 2, 3, "qk", "8bit"), (128, (64, 64), 1, 24, "qk bias", "8bit"), (128, (64, 64), 1, 24, "qk", "mixed"), (128, (64, 64), 1, 2, "qk", "mixed"),
])
def test_decoding_step_with_head_norms(D, heads, B, T, which, slots):
    """q and the fresh k with bias and head norms finished inside the decode attention: one and two row blocks, gains of q or k
    alone, the forms of long calls (64 kv heads); hidden states and the K/V that were appended, against the oracle's block."""
    (Hq, Hkv), H, F, C = heads, 128, 64, 64
    long = heads == (64, 64)
    n_chunks = 20 if long else 2
    g = np.random.default_rng(8200 + D + 7 * T + Hq)
    W = wl.stack_weights(35, 0, H, Hq, Hkv, D, F)
    W.Wo = W.Wo * np.float32(4)    # (the attention's share of the output: a gain read at the wrong place is off by 4 % or more)
    layer, extras = dev_layers([W])[0], dict(bias=None, q_gain=None, k_gain=None, eps=EPS)
    for name, arg in (("q", "q_gain"), ("k", "k_gain")):
        if name in which.split()[0]:
            extras[arg] = wl.round_bf16(1 + 0.3 * g.standard_normal(D).astype(np.float32))
            layer[name + "_norm"] = bf16(extras[arg])
    if "bias" in which:
        extras["bias"] = wl.round_bf16(0.5 * g.standard_normal((Hq + 2 * Hkv) * D).astype(np.float32))
        layer["qkv_bias"] = bf16(extras["bias"])
    n_slots = B * (n_chunks + 1)
    kind = dict(kv_fp8=True) if slots == "8bit" else dict(n_slots_8bit=n_slots // 2) if slots == "mixed" else {}
    pc = Percache(n_layers=1, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=n_slots, slot_capacity=C,
                  max_pos=(n_chunks + 1) * C, device=DEV, **kind)
    chain = np.arange(n_slots, dtype=np.int32).reshape(B, n_chunks + 1)
    own, have = [int(s) for s in chain[:, -1]], 37
    for s in chain.reshape(-1):
        n = have if int(s) in own else C
        pc.percache_kv_put(0, int(s), bf16(g.standard_normal((Hkv, n, D))), bf16(g.standard_normal((Hkv, n, D)) + 2 * g.standard_normal((Hkv, 1, D))))
    kept = [[tuple(host(t) for t in pc.percache_kv_get(0, int(s))) for s in row] for row in chain]
    x = wl.round_bf16(g.standard_normal((B, T, H)).astype(np.float32))
    out = pc.percache_stack_decode([layer], F, EPS, bf16(x), chain, own)
    torch.cuda.synchronize()
    for b in range(B):
        sk, sv = (np.zeros((n_chunks + 1, Hkv, C, D), np.float32) for _ in range(2))
        used = np.array([C] * n_chunks + [have], np.int32)
        for c in range(n_chunks + 1):
            sk[c, :, :used[c]], sv[c, :, :used[c]] = kept[b][c]
        ref, k, v = oracle_block(x[b], W, Hq, Hkv, D, 10000.0, sk, sv, np.arange(n_chunks + 1, dtype=np.int32), used, extras=extras)
        check_hidden(host(out[b]), ref, f"D={D} heads {heads} T={T} {which} {slots} query {b}")
        assert pc.percache_kv_len(0, own[b]) == have + T
        is8 = slots == "8bit" or (slots == "mixed" and own[b] >= n_slots - n_slots // 2)
        for got, want in zip(pc.percache_kv_get(0, own[b]), (k, v)):
            want = np.asarray(want)[:, -T:]
            # one rounding of the normed row and one of the result (two steps of 2^-8 of the largest value each way), an 8-bit
            # code then by at most one step of 1/8
            assert np.abs(host(got)[:, have:] - want).max() <= (2.0 ** -3 if is8 else 2.0 ** -6) * np.abs(want).max(), (b, is8)
    pc.close()


@pytest.mark.parametrize("B,T,tiles,Hq", [(1, 1, 45, 4), (1, 1, 57, 4), (1, 1, 59, 4), (1, 1, 120, 4), (2, 1, 45, 4), (1, 2, 57, 4), (2, 1, 83, 4), (1, 1, 40, 16),
                                          (1, 1, 57, 16), (1, 1, 59, 16), (2, 1, 17, 16), (1, 2, 19, 16)])
def test_o_proj_merges_long_partition_lists(B, T, tiles, Hq):
    """Decoding steps of one and two rows over 17 to 120 cached tiles of two kv heads: the o_proj merges up to 30 partitions, 20 at a
    time, and up to 10 of two rows of 16 heads, with the largest scores in the first, the last and the middle chunks.  59 tiles and more,
    and 19 of two rows of 16 heads, lie past what it merges: 31 and 11 partitions."""
    D, Hkv, H, F, C = 128, 2, 256, 64, 320
    W = wl.stack_weights(36, 0, H, Hq, Hkv, D, F)
    # (the attention's share of the output; with the chunks' mean values below, a chunk left out or counted twice is off by 10 % or more)
    W.Wo = W.Wo * np.float32(8 if Hq == 4 else 4)
    n_chunks = -(-tiles * 64 // C)
    g = np.random.default_rng(8300 + tiles + B)
    pc = Percache(n_layers=1, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=B * n_chunks, slot_capacity=C,
                  max_pos=n_chunks * C + T, device=DEV)
    used = np.full((B, n_chunks), C, np.int32)
    used[:, -1] = tiles * 64 - (n_chunks - 1) * C - 11
    x = wl.round_bf16(g.standard_normal((B, T, H)).astype(np.float32))
    for loud in ((0,), (n_chunks - 1,), (n_chunks // 2, 1)):
        sk, sv = (wl.round_bf16(g.standard_normal((B, n_chunks, Hkv, C, D)).astype(np.float32)) for _ in range(2))
        sv = wl.round_bf16(sv + 2 * g.standard_normal((B, n_chunks, Hkv, 1, D)).astype(np.float32))
        for c in range(n_chunks):
            sk[:, c] = wl.round_bf16(sk[:, c] * np.float32(2.0 if c in loud else 0.3))
        for b in range(B):
            for c in range(n_chunks):
                pc.percache_kv_put(0, b * n_chunks + c, bf16(sk[b, c]), bf16(sv[b, c]))
        out = pc.percache_stack_decode(dev_layers([W]), F, EPS, bf16(x), np.arange(B * n_chunks, dtype=np.int32).reshape(B, -1), [-1] * B, used_len=used)
        torch.cuda.synchronize()
        for b in range(B):
            ref, _, _ = oracle_block(x[b], W, Hq, Hkv, D, 10000.0, sk[b], sv[b], np.arange(n_chunks, dtype=np.int32), used[b])
            check_hidden(host(out[b]), ref, f"{tiles} tiles, loud chunks {loud}, B={B} T={T} query {b}")
    pc.close()


def _step_inputs(H, Hq, Hkv, D, F, L, variant, g):
    Ws = []
    for _ in range(L):
        n = (Hq + 2 * Hkv) * D
        w = dict(gain1=1 + 0.1 * g.standard_normal(H), wqkv=0.02 * g.standard_normal((n, H)), wo=0.02 * g.standard_normal((H, Hq * D)),
                 gain2=1 + 0.1 * g.standard_normal(H), w_gate=0.02 * g.standard_normal((F, H)), w_up=0.02 * g.standard_normal((F, H)),
                 w_down=0.02 * g.standard_normal((H, F)))
        if variant == "bias":
            w["qkv_bias"] = 0.5 * g.standard_normal(n)
        if variant == "norm":
            w.update(q_norm=1 + 0.1 * g.standard_normal(D), k_norm=1 + 0.1 * g.standard_normal(D))
        Ws.append({k: bf16(v.astype(np.float32)) for k, v in w.items()})
    return Ws


def _one_launch_room(pc, Ws, F, B, T, max_chunks):
    """Where in a step's workspace the part of the one launch for all layers begins, which nothing else writes: the least size that a call is not
    refused for.  (Asked with a misaligned pointer: refused for that next, so nothing runs.)"""
    arr = pc._weights(Ws)
    keep, ids_p, _, n_p, _ = pc._chunk_args(B, np.zeros((B, max_chunks), np.int32), None, [0] * B)
    own, own_p = _host_i32([-1] * B)
    buf = torch.zeros(16, dtype=torch.uint8, device=DEV)

    def status(n_bytes):
        return pc.lib.percache_stack_decode(pc.ctx, arr, len(Ws), F, EPS, buf.data_ptr(), B, T, ids_p, None, n_p, max_chunks, own_p, buf.data_ptr(),
                                            (buf.data_ptr() + 255) // 256 * 256 + 16, n_bytes, None)
    lo, hi = 0, pc.percache_stack_workspace_bytes(B, T, max_chunks, F)
    assert status(hi) == -1
    while hi - lo > 1:
        mid = (lo + hi) // 2
        st = status(mid)
        assert st in (-1, -5)
        lo, hi = (mid, hi) if st == -5 else (lo, mid)
    return hi


def _in_one_launch(pc, Ws, F, B, T, max_chunks, step):
    """Whether step(), a call of that shape, took all layers in one launch: then the first word of that launch's workspace, its counter of items, is not as
    it was."""
    pc._stack_workspace(B, T, pc.percache_stack_workspace_bytes(B, T, max_chunks, F))
    pc._step_ws.fill_(173)
    step()
    torch.cuda.synchronize()
    at = (-pc._step_ws.data_ptr()) % 256 + _one_launch_room(pc, Ws, F, B, T, max_chunks)
    return bool((pc._step_ws[at:at + 4] != 173).any())


@pytest.mark.parametrize("H,Hq,Hkv,D,F,L,B,T,chunks,C,slots,variant", [
    (128, 2, 1, 64, 64, 2, 1, 1, 0, 64, "bf16", "plain"),        # wavefronts without a slice, nothing cached, one piece
    (256, 4, 2, 128, 512, 4, 4, 1, 3, 128, "8bit", "norm"),
    (1024, 16, 8, 128, 3072, 4, 1, 1, 6, 512, "mixed", "norm"),
    (896, 14, 2, 64, 4864, 8, 1, 2, 5, 192, "mixed", "bias"),
    (896, 14, 2, 64, 4864, 34, 1, 1, 70, 64, "bf16", "bias"),    # two launches of layers, chunks past the 64th, one row past kRowCols
    (3072, 24, 8, 128, 8192, 2, 1, 1, 4, 320, "bf16", "plain"),
    (128, 2, 1, 64, 16384, 2, 1, 1, 1, 64, "bf16", "plain"),     # the widest contraction
    (1024, 16, 8, 128, 3072, 8, 4, 1, 2, 128, "bf16", "plain"),  # the widest of four rows
    (384, 14, 1, 64, 192, 2, 1, 1, 16, 960, "bf16", "plain"),    # 240 tiles: four to a piece, the longest merge
    (384, 15, 1, 128, 192, 2, 1, 1, 6, 192, "mixed", "norm"),    # the most query rows of a kv head at either head size
    (256, 16, 1, 64, 192, 2, 1, 1, 6, 192, "8bit", "plain"),
    (256, 4, 4, 128, 320, 4, 1, 4, 2, 128, "8bit", "plain"),
])
def test_step_in_one_launch_against_one_by_one(H, Hq, Hkv, D, F, L, B, T, chunks, C, slots, variant):
    """Steps of a few rows take all layers in one launch unless the QKV or attention kernels' times were asked for.  Both round the same
    values to bf16, in other orders of summation: per layer about six roundings that two runs may take differently, 2^-9 / sqrt(3) each, carried
    on with a factor of about 1.5: 4.2e-3 sqrt(layers); the bound is 6e-3 sqrt(layers).  The first layer's K/V must agree to one rounding."""
    g = np.random.default_rng(17)
    Ws = _step_inputs(H, Hq, Hkv, D, F, L, variant, g)
    n_slots = B * chunks + 2 * B
    kind = dict(kv_fp8=True) if slots == "8bit" else dict(n_slots_8bit=n_slots // 2) if slots == "mixed" else {}
    pc = Percache(n_layers=L, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=n_slots, slot_capacity=C, max_pos=chunks * C + C + 3 * T,
                  device=DEV, **kind)
    ids = [int(x) for x in g.permutation(n_slots)]
    if slots == "mixed":   # the two runs' own slots of the same format
        ids = sorted(ids)
    lists = [ids[2 * B + b * chunks: 2 * B + (b + 1) * chunks] for b in range(B)]
    own = [ids[:B], ids[B:2 * B]]
    for s in [s for row in lists for s in row]:
        n = int(g.integers(C - 63 if C > 512 else 1, C + 1))
        for layer in range(L):
            pc.percache_kv_put(layer, s, bf16(g.standard_normal((Hkv, n, D))), bf16(g.standard_normal((Hkv, n, D))))
    xs = [bf16(g.standard_normal((B, T, H))) for _ in range(3)]
    outs = [[], []]
    for way in (0, 1):
        pc.percache_profile_enable(way == 1, [2])
        for i, x in enumerate(xs):
            took = _in_one_launch(pc, Ws, F, B, T, chunks + (i > 0), lambda: outs[way].append(host(
                pc.percache_stack_decode(Ws, F, EPS, x, [lists[b] + ([own[way][b]] if i else []) for b in range(B)], own[way]))))
            assert took == (way == 0), (way, i)
    pc.percache_profile_enable(False)
    for i, (a, b) in enumerate(zip(*outs)):
        check_hidden(a, b, f"step {i} in one launch against one by one", rel_max=2.0 ** -4 * max(1, L) ** 0.5, rel_fro=6e-3 * L ** 0.5)
    for b in range(B):
        assert pc.percache_kv_len(0, own[0][b]) == pc.percache_kv_len(L - 1, own[0][b]) == 3 * T
        for x, y in zip(pc.percache_kv_get(0, own[0][b]), pc.percache_kv_get(0, own[1][b])):
            check_hidden(host(x), host(y), "first layer's K/V", rel_max=2.0 ** -4 if slots != "bf16" else 2.0 ** -7)


@pytest.mark.parametrize("H,Hq,Hkv,D,F,L,B,T,tiles,one", [
    (1024, 16, 8, 128, 3072, 1, 1, 1, 2, False), (1024, 16, 8, 128, 3072, 2, 1, 1, 38, True), (1024, 16, 8, 128, 3072, 2, 1, 1, 39, False),
    (1024, 16, 8, 128, 3072, 4, 1, 1, 110, True), (1024, 16, 8, 128, 3072, 4, 1, 1, 111, False),
    (2048, 16, 8, 128, 2048, 4, 1, 1, 62, True), (2048, 16, 8, 128, 2048, 4, 1, 1, 63, False),
    (3072, 2, 1, 64, 128, 2, 1, 1, 2, True), (3200, 2, 1, 64, 128, 2, 1, 1, 2, False), (4096, 2, 1, 64, 128, 4, 1, 1, 2, True), (4224, 2, 1, 64, 128, 4, 1, 1, 2, False),
    (256, 2, 1, 64, 16384, 2, 1, 1, 2, True), (256, 2, 1, 64, 16448, 2, 1, 1, 2, False),
    (256, 4, 2, 64, 256, 3, 2, 1, 2, False), (256, 4, 2, 64, 256, 4, 2, 1, 2, True), (256, 4, 2, 64, 256, 4, 2, 1, 0, False),
    (256, 4, 2, 64, 4608, 4, 2, 1, 2, True), (256, 4, 2, 64, 4672, 4, 2, 1, 2, False), (256, 4, 2, 64, 6144, 8, 2, 1, 2, True), (256, 4, 2, 64, 6208, 8, 2, 1, 2, False),
    (256, 16, 8, 64, 256, 4, 2, 1, 18, True), (256, 16, 8, 64, 256, 4, 2, 1, 19, False),
])
def test_which_steps_take_one_launch(H, Hq, Hkv, D, F, L, B, T, tiles, one):
    """Both sides of every line of the rule (256 CUs), and the same result up to rounding on either.  (Weights of few distinct layers.)"""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the lines lie elsewhere")
    g = np.random.default_rng(31)
    Ws = _step_inputs(H, Hq, Hkv, D, F, 1, "plain", g) * L
    C = max(64, tiles * 64)
    pc = Percache(n_layers=L, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=B, slot_capacity=C, max_pos=C + T, device=DEV)
    for layer in range(L if tiles else 0):
        for s in range(B):
            pc.percache_kv_put(layer, s, bf16(g.standard_normal((Hkv, C, D))), bf16(g.standard_normal((Hkv, C, D))))
    x = bf16(g.standard_normal((B, T, H)))
    lists = np.arange(B, dtype=np.int32).reshape(B, 1) if tiles else np.zeros((B, 0), np.int32)
    outs = []
    assert _in_one_launch(pc, Ws, F, B, T, lists.shape[1], lambda: outs.append(pc.percache_stack_decode(Ws, F, EPS, x, lists, [-1] * B))) == one
    pc.percache_profile_enable(True, [2])
    ref = pc.percache_stack_decode(Ws, F, EPS, x, lists, [-1] * B)
    pc.percache_profile_enable(False)
    check_hidden(host(outs[0]), host(ref), f"{tiles} tiles", rel_max=2.0 ** -4 * L ** 0.5, rel_fro=6e-3 * L ** 0.5)
    assert one or torch.equal(outs[0], ref)
    pc.close()


def test_steps_on_two_streams_at_once():
    """Two programs' steps queued on two streams, neither waiting for the other: each result is the one it has alone, bit for bit."""
    g = np.random.default_rng(5)
    H, Hq, Hkv, D, F, L = 256, 4, 2, 64, 512, 6
    Ws = _step_inputs(H, Hq, Hkv, D, F, L, "plain", g)
    pcs = [Percache(n_layers=L, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=4, slot_capacity=128, max_pos=512, device=DEV) for _ in range(2)]
    for pc in pcs:
        for layer in range(L):
            for s in range(3):
                pc.percache_kv_put(layer, s, bf16(g.standard_normal((Hkv, 100, D))), bf16(g.standard_normal((Hkv, 100, D))))
    xs = [bf16(g.standard_normal((1, 1, H))) for _ in range(2)]
    alone = []
    for pc, x in zip(pcs, xs):
        assert _in_one_launch(pc, Ws, F, 1, 1, 3, lambda: alone.append(pc.percache_stack_decode(Ws, F, EPS, x, [[0, 1, 2]], [-1])))
    streams = [torch.cuda.Stream() for _ in range(2)]
    outs = [[], []]
    for _ in range(20):
        for i in (0, 1):
            with torch.cuda.stream(streams[i]):
                outs[i].append(pcs[i].percache_stack_decode(Ws, F, EPS, xs[i], [[0, 1, 2]], [-1]))
    torch.cuda.synchronize()
    for i in (0, 1):
        assert all(torch.equal(o, alone[i]) for o in outs[i])


@pytest.mark.parametrize("B,L", [(1, 34), (2, 4)])
def test_step_in_one_launch_captured(B, L):
    """A step from a device table captured once and replayed between eager calls: the captured list bit for bit every time (its counters and hand-over buffers
    are set anew by the replay itself), then lists of other lengths written into the table, longer ones and an empty one among them."""
    g = np.random.default_rng(37)
    H, Hq, Hkv, D, F, C, n_c = 256, 4, 2, 64, 320, 320, 6
    Ws = _step_inputs(H, Hq, Hkv, D, F, 2, "norm", g) * (L // 2)
    pc = Percache(n_layers=L, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=B * n_c, slot_capacity=C, max_pos=n_c * C + 1, device=DEV)
    for layer in range(L):
        for s in range(B * n_c):
            pc.percache_kv_put(layer, s, bf16(g.standard_normal((Hkv, C, D))), bf16(g.standard_normal((Hkv, C, D))))
    x, out = bf16(g.standard_normal((B, 1, H))), bf16(np.zeros((B, 1, H)))
    ids = np.arange(B * n_c, dtype=np.int32).reshape(B, n_c)
    lists = [g.integers(1, 130, (B, n_c)), np.full((B, n_c), C), np.zeros((B, n_c), np.int64), g.integers(0, C + 1, (B, n_c))]
    table = pc.percache_chunk_table_put(ids, lists[0])
    arr = pc.percache_stack_reuse_table(Ws, F, EPS, x, table, out)
    assert _in_one_launch(pc, Ws, F, B, 1, n_c, lambda: pc.percache_stack_reuse_table(Ws, F, EPS, x, table, out, weights=arr))
    eager = out.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pc.percache_stack_reuse_table(Ws, F, EPS, x, table, out, weights=arr)
    for used in lists:
        pc.percache_chunk_table_put(ids, used, table=table)
        ref = pc.percache_stack_reuse(Ws, F, EPS, x, ids, used)
        for _ in range(3):
            pc._step_ws.fill_(int(g.integers(0, 256)))
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            if used is lists[0]:
                assert torch.equal(out, eager)
            check_hidden(host(out), host(ref), "replayed", rel_max=2.0 ** -4 * L ** 0.5, rel_fro=6e-3 * L ** 0.5)   # (as above)
    pc.close()


def test_step_in_a_workspace_sized_for_a_longer_call():
    """28 layers hand on more between their parts than 6 fresh tokens need as workspace: a step in a buffer of the longer call's size is taken,
    launch by launch, one byte less than that takes is refused, and a step leaves the workspace that the binding holds for prompts where it is."""
    g = np.random.default_rng(23)
    H, Hq, Hkv, D, F, L, C = 256, 8, 4, 64, 512, 28, 512
    Ws = _step_inputs(H, Hq, Hkv, D, F, L, "plain", g)
    pc = Percache(n_layers=L, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=7, slot_capacity=C, max_pos=8 * C, device=DEV)
    for layer in range(L):
        for s in range(6):
            pc.percache_kv_put(layer, s, bf16(g.standard_normal((Hkv, C, D))), bf16(g.standard_normal((Hkv, C, D))))
    x = bf16(g.standard_normal((1, 1, H)))
    whole = pc.percache_stack_decode(Ws, F, EPS, x, [range(6)], [-1])
    full, longer = (pc.percache_stack_workspace_bytes(1, t, 6, F) for t in (1, 6))
    assert longer < full
    least = _one_launch_room(pc, Ws, F, 1, 1, 6)
    arr = pc._weights(Ws)
    keep, ids_p, _, n_p, _ = pc._chunk_args(1, [range(6)], None, None)
    none, none_p = _host_i32([-1])
    out = torch.empty_like(x)

    def step(n_bytes, one):
        buf = torch.full((n_bytes + 512,), 173, dtype=torch.uint8, device=DEV)
        at = (-buf.data_ptr()) % 256
        out.zero_()
        assert pc.lib.percache_stack_decode(pc.ctx, arr, L, F, EPS, x.data_ptr(), 1, 1, ids_p, None, n_p, 6, none_p, out.data_ptr(),
                                            buf.data_ptr() + at, n_bytes, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        assert (buf[:at] == 173).all() and (buf[at + n_bytes:] == 173).all()
        assert bool((buf[at + least:at + least + 4] != 173).any()) == one
        return out.clone()
    one_by_one = step(longer, False)
    check_hidden(host(one_by_one), host(whole), "step in the smaller workspace", rel_max=2.0 ** -4 * L ** 0.5, rel_fro=6e-3 * L ** 0.5)   # (as above)
    assert torch.equal(step(least, False), one_by_one) and torch.equal(step(full, True), whole)
    h = bf16(g.standard_normal((1, 6, H)))
    pc.percache_stack_reuse(Ws, F, EPS, h, [range(6)])
    held = pc._ws.data_ptr()
    pc.percache_stack_decode(Ws, F, EPS, x, [range(6)], [-1])
    assert pc._ws.data_ptr() == held
    pc.close()


def test_step_through_more_than_64_launches_of_layers():
    """2080 layers are 65 launches in a row, each with a counter of its own in front of the first layer's input.  All but six layers add nothing
    (their output weights are zeros), so the result is that of the launches one by one up to the rounding of six layers."""
    g = np.random.default_rng(29)
    H, Hq, Hkv, D, F, L = 128, 2, 1, 64, 64, 2080
    live = dict(zip((0, 31, 32, 2047, 2048, L - 1), _step_inputs(H, Hq, Hkv, D, F, 6, "plain", g)))
    still = {k: torch.zeros_like(v) if k in ("wo", "w_down") else v for k, v in live[0].items()}
    Ws = [live.get(l, still) for l in range(L)]
    pc = Percache(n_layers=L, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=1, slot_capacity=64, max_pos=64, device=DEV)
    x = bf16(g.standard_normal((1, 1, H)))
    one = pc.percache_stack_decode(Ws, F, EPS, x, np.zeros((1, 0), np.int32), [-1])
    torch.cuda.synchronize()
    pc.percache_profile_enable(True, [2])
    each = pc.percache_stack_decode(Ws, F, EPS, x, np.zeros((1, 0), np.int32), [-1])
    pc.percache_profile_enable(False)
    assert not torch.equal(one, x)
    assert _in_one_launch(pc, Ws, F, 1, 1, 0, lambda: pc.percache_stack_decode(Ws, F, EPS, x, np.zeros((1, 0), np.int32), [-1]))
    check_hidden(host(one), host(each), "2080 layers", rel_max=2.0 ** -4 * 6 ** 0.5, rel_fro=6e-3 * 6 ** 0.5)   # (as above)
    pc.close()
