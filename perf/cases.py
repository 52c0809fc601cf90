"""Timing cases: what a program built on this library asks of it, from one query against a small bank to the prefill of
whole prompts, through the public binding.

A case is a dict of plain values; ``prepare`` makes what such a program holds before the call (context, store, bank,
weights, inputs) on the GPU from a seed, ``run`` is one pass through the entry points, ``work`` the bytes and flops that
no implementation can do without, ``tolerance`` how far another correct implementation's results may lie off.

Kinds of pass
  front    query-level match of a batch of queries against the QA bank and, with k > 0, the k best chunks per query
           from a second bank (dense retrieval)
  refresh  new knowledge chunks against every stored query (cache refresh)
  layer    one layer's cache-reusing prefill of a batch of queries; with save = True the fresh K/V go to slots
  stack    a whole stack over cached chunks (mode "reuse"), or the ordinary prefill of a prompt with nothing cached that
           fills the cache, with the chunk tensors read back for storing (mode "populate")
  answer   a prompt's fresh part over cached chunks (if fresh > 0), then one decoding step per generated token
  store    chunk tensors written to slots and read back
"""
import numpy as np
import torch

from paper_2601_11553_amd.binding import Percache

DEV = "cuda:0"
EPS = 1e-6
TAU = 0.85
# width, query heads, kv heads, head size, ffn width
SHAPES = {"0.6B": (1024, 16, 8, 128, 3072), "3B": (3072, 24, 8, 128, 8192), "d64": (896, 14, 2, 64, 4864)}


def listed():
    return [
        # one user's query on a small personal cache: match against 2000 stored questions, then 3 of 1000 chunks
        dict(name="front_small", kind="front", probes=1, qa_rows=2000, chunk_rows=1000, dim=768, k=3),
        # a batch of 8 queries in front of a large shared cache: match, then the 8 best chunks each
        dict(name="front_step", kind="front", probes=8, qa_rows=200_000, chunk_rows=50_000, dim=1024, k=8),
        # offline matching of 1024 queries against the large bank
        dict(name="match_batch", kind="front", probes=1024, qa_rows=200_000, chunk_rows=0, dim=1024, k=0),
        # 64 chunks were added: which stored answers are out of date?
        dict(name="refresh_scan", kind="refresh", new=64, qa_rows=200_000, dim=1024),
        # one short query over 4 cached chunks, a layer of a 0.6B-shaped model: latency
        dict(name="layer_small", kind="layer", shape="0.6B", batch=1, fresh=64, chunks=4, chunk=512, slots_total=16,
             ragged=False, slots="bf16", table=False, save=False),
        # 8 queries over long cached contexts, a layer of a 3B-shaped model, fresh K/V kept: throughput
        dict(name="layer_step", kind="layer", shape="3B", batch=8, fresh=256, chunks=16, chunk=1024, slots_total=1032,
             ragged=False, slots="bf16", table=False, save=True),
        # the same service with 8-bit slots and natural chunk lengths (chunks are cut at sentence ends, not at 64)
        dict(name="layer_8bit", kind="layer", shape="3B", batch=6, fresh=203, chunks=13, chunk=1024, slots_total=512,
             ragged=True, slots="8bit", table=False, save=True),
        # the paper's online prefill: 28 layers over 8 retrieved chunks with 128 fresh tokens
        dict(name="stack_reuse", kind="stack", mode="reuse", shape="0.6B", layers=28, batch=1, fresh=128, chunks=8, chunk=512,
             ragged=False, slots="bf16", variant="plain", table=False),
        # cache population: the full prompt prefilled once, its chunks stored and read back for the chunk files
        dict(name="stack_populate", kind="stack", mode="populate", shape="0.6B", layers=28, batch=1, fresh=128, chunks=8, chunk=512,
             ragged=False, slots="bf16", variant="plain", table=False),
        # one user's answer: 100 fresh tokens over ragged cached chunks, then 16 tokens, a model with head norms
        dict(name="answer_one", kind="answer", shape="0.6B", layers=28, batch=1, fresh=100, chunks=6, chunk=512, new=16,
             ragged=True, slots="bf16", variant="norm"),
        # 8 users decoding over long cached contexts, 4 layers of a 3B-shaped model
        dict(name="decode_batch", kind="answer", shape="3B", layers=4, batch=8, fresh=0, chunks=16, chunk=1024, new=4,
             ragged=True, slots="bf16", variant="plain"),
        # chunk tensors into the store and back out (loading and saving chunk files), half of the slots 8-bit
        dict(name="store_io", kind="store", shape="3B", chunks=16, tokens=1000, slots="mixed"),
    ]


def _logint(rng, lo, hi):
    return max(lo, min(hi, int(round(float(lo) * (float(hi) / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["front", "refresh", "layer", "layer", "stack", "populate", "answer", "store"])
    if kind == "front":
        k = rng.choice([0, 0, 2, 3, 5, 8])
        return dict(kind="front", probes=_logint(rng, 1, 1024), qa_rows=_logint(rng, 500, 200_000),
                    chunk_rows=_logint(rng, 200, 60_000) if k else 0, dim=rng.choice([384, 512, 768, 1024]), k=k)
    if kind == "refresh":
        return dict(kind="refresh", new=_logint(rng, 1, 256), qa_rows=_logint(rng, 1000, 200_000), dim=rng.choice([384, 512, 768, 1024]))
    shape = rng.choice(list(SHAPES))
    slots = rng.choice(["bf16", "bf16", "8bit", "mixed"])
    ragged = rng.random() < 0.6
    if kind == "layer":
        batch, chunks, chunk = _logint(rng, 1, 8), rng.randint(1, 16), rng.choice([128, 192, 256, 512, 1024])
        return dict(kind="layer", shape=shape, batch=batch, fresh=_logint(rng, 8, 256), chunks=chunks, chunk=chunk,
                    slots_total=batch * chunks + 8, ragged=ragged, slots=slots, table=rng.random() < 0.3, save=rng.random() < 0.5)
    variant = rng.choice(["plain", "bias", "norm"])
    # (the 3B-shaped model at a few layers: a draw stays within the listed cases' cost)
    layers = _logint(rng, 1, 8 if shape == "3B" else 28)
    if kind == "stack":
        batch = rng.choice([1, 1, 2, 4])
        return dict(kind="stack", mode="reuse", shape=shape, layers=layers, batch=batch, fresh=_logint(rng, 8, 256), chunks=rng.randint(1, 8),
                    chunk=rng.choice([128, 256, 512]), ragged=ragged, slots=slots, variant=variant, table=rng.random() < 0.3)
    if kind == "populate":
        return dict(kind="stack", mode="populate", shape=shape, layers=layers, batch=1, fresh=_logint(rng, 8, 128),
                    chunks=rng.randint(1, 4 if shape == "3B" else 8), chunk=rng.choice([128, 256, 512]), ragged=False, slots=slots, variant=variant, table=False)
    if kind == "answer":
        return dict(kind="answer", shape=shape, layers=layers, batch=_logint(rng, 1, 8), fresh=rng.choice([0, _logint(rng, 8, 192)]),
                    chunks=rng.randint(1, 8), chunk=rng.choice([256, 512, 1024]), new=rng.randint(1, 8), ragged=ragged, slots=slots, variant=variant)
    return dict(kind="store", shape=shape, chunks=_logint(rng, 1, 48), tokens=_logint(rng, 16, 1024), slots=slots)


# ------------------------------------------------------------------------------------------------ inputs
class _Gen:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))
        self.host = np.random.default_rng(int(seed))

    def normal(self, *shape, scale=1.0, dtype=torch.bfloat16):
        if dtype != torch.float32 and int(np.prod(shape)) > (1 << 28):   # (bounds the fp32 temporary)
            return torch.stack([self.normal(*shape[1:], scale=scale, dtype=dtype) for _ in range(shape[0])])
        return (torch.randn(shape, generator=self.g, device=DEV) * scale).to(dtype)

    def unit_rows(self, x):
        return x / x.norm(dim=-1, keepdim=True)


def _embeddings(g, rows, dim, probes):
    """Clustered unit-norm rows (about 100 a cluster) and queries near them: half noisy copies of rows, half new draws."""
    n_c = max(1, rows // 100)
    centres = g.unit_rows(torch.randn((n_c, dim), generator=g.g, device=DEV))
    of = torch.randint(0, n_c, (rows,), generator=g.g, device=DEV)
    bank = g.unit_rows(centres[of] + 0.05 * torch.randn((rows, dim), generator=g.g, device=DEV)).half()
    n_copy = (probes + 1) // 2
    src = torch.randint(0, rows, (n_copy,), generator=g.g, device=DEV)
    copies = bank[src].float() + 0.01 * torch.randn((n_copy, dim), generator=g.g, device=DEV)
    c = torch.randint(0, n_c, (probes - n_copy,), generator=g.g, device=DEV)
    new = centres[c] + 0.05 * torch.randn((probes - n_copy, dim), generator=g.g, device=DEV)
    return bank, g.unit_rows(torch.cat([copies, new])).half().contiguous()


def _bank(rows, dim, emb):
    pc = Percache(n_layers=1, hidden=64, n_q_heads=2, n_kv_heads=1, head_dim=64, n_slots=1, slot_capacity=64, max_pos=64,
                  bank_capacity=rows, emb_dim=dim, device=DEV)
    pc.percache_bank_put(0, emb)
    return pc


def _lengths(case, g, n):
    """Stored lengths of n chunks: whole slots, or lengths between half a slot and a whole one."""
    C = case["chunk"]
    return [int(x) for x in g.host.integers(C // 2, C + 1, n)] if case["ragged"] else [C] * n


def _context(case, n_slots, capacity, max_pos, n_layers):
    H, Hq, Hkv, D, _ = SHAPES[case["shape"]]
    kind = dict(kv_fp8=True) if case["slots"] == "8bit" else dict(n_slots_8bit=n_slots // 2) if case["slots"] == "mixed" else {}
    return Percache(n_layers=n_layers, hidden=H, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=n_slots, slot_capacity=capacity,
                    max_pos=max_pos, device=DEV, **kind)


def _fill(pc, case, g, slots, lengths, n_layers):
    _, _, Hkv, D, _ = SHAPES[case["shape"]]
    for layer in range(n_layers):
        for s0 in range(0, len(slots), 64):
            part = range(s0, min(s0 + 64, len(slots)))
            top = max(lengths[i] for i in part)
            k, v = g.normal(len(part), Hkv, top, D), g.normal(len(part), Hkv, top, D)
            if all(lengths[i] == top for i in part):
                pc.percache_kv_put_batch(layer, [slots[i] for i in part], k, v)
            else:
                for j, i in enumerate(part):
                    n = lengths[i]
                    pc.percache_kv_put(layer, slots[i], k[j, :, :n].contiguous(), v[j, :, :n].contiguous())


def _weights(case, g):
    H, Hq, Hkv, D, F = SHAPES[case["shape"]]
    n_out = (Hq + 2 * Hkv) * D
    layers = []
    for _ in range(case["layers"]):
        w = dict(gain1=(1 + g.normal(H, scale=0.1, dtype=torch.float32)).bfloat16(), wqkv=g.normal(n_out, H, scale=0.02), wo=g.normal(H, Hq * D, scale=0.02),
                 gain2=(1 + g.normal(H, scale=0.1, dtype=torch.float32)).bfloat16(), w_gate=g.normal(F, H, scale=0.02), w_up=g.normal(F, H, scale=0.02),
                 w_down=g.normal(H, F, scale=0.02))
        if case["variant"] == "bias":
            w.update(qkv_bias=g.normal(n_out, scale=0.5))
        if case["variant"] == "norm":
            w.update(q_norm=(1 + g.normal(D, scale=0.1, dtype=torch.float32)).bfloat16(), k_norm=(1 + g.normal(D, scale=0.1, dtype=torch.float32)).bfloat16())
        layers.append(w)
    return layers


def prepare(case, seed):
    g = _Gen(seed)
    s = dict(case=case)
    kind = case["kind"]
    if kind == "front":
        emb, s["probes"] = _embeddings(g, case["qa_rows"], case["dim"], case["probes"])
        s["qa"] = _bank(case["qa_rows"], case["dim"], emb)
        P = case["probes"]
        s["out"] = (torch.empty(P, dtype=torch.int32, device=DEV), torch.empty(P, dtype=torch.float32, device=DEV), torch.empty(P, dtype=torch.uint8, device=DEV))
        if case["k"]:
            emb, _ = _embeddings(g, case["chunk_rows"], case["dim"], 1)
            s["chunks"] = _bank(case["chunk_rows"], case["dim"], emb)
        return s
    if kind == "refresh":
        emb, s["new"] = _embeddings(g, case["qa_rows"], case["dim"], case["new"])
        s["qa"] = _bank(case["qa_rows"], case["dim"], emb)
        s["kth"] = 0.2 + 0.3 * torch.rand(case["qa_rows"], generator=g.g, device=DEV)
        return s
    H, Hq, Hkv, D, F = SHAPES[case["shape"]]
    if kind == "store":
        n, T = case["chunks"], case["tokens"]
        s["pc"] = _context(case, 2 * n, (T + 63) // 64 * 64, 64, 1)
        s["slots"] = [int(x) for x in g.host.permutation(2 * n)[:n]]
        s["k"], s["v"] = g.normal(n, Hkv, T, D), g.normal(n, Hkv, T, D)
        s["ko"], s["vo"] = torch.empty_like(s["k"]), torch.empty_like(s["v"])
        return s
    B, C, n_c = case["batch"], case["chunk"], case["chunks"]
    T = case["fresh"]
    if kind == "layer":
        n_slots = max(case["slots_total"], B * n_c + B)
        cap = max(C, (T + 63) // 64 * 64)
        s["pc"] = pc = _context(case, n_slots, cap, n_c * C + T, 1)
        ids = g.host.permutation(n_slots)
        s["ids"], s["spare"] = ids[:B * n_c].reshape(B, n_c).astype(np.int32), [int(x) for x in ids[B * n_c:B * n_c + B]]
        _fill(pc, case, g, [int(x) for x in ids[:B * n_c]], _lengths(case, g, B * n_c), 1)
        s["x"], s["w"] = g.normal(B, T, H), g.normal((Hq + 2 * Hkv) * D, H, scale=0.02)
        s["attn"] = torch.empty((B, T, Hq * D), dtype=torch.bfloat16, device=DEV)
        s["kf"], s["vf"] = (torch.empty((B, Hkv, T, D), dtype=torch.bfloat16, device=DEV) for _ in range(2))
        s["table"] = pc.percache_chunk_table_put(s["ids"]) if case["table"] else None
        return s
    L = case["layers"]
    s["layers"] = _weights(case, g)
    if kind == "stack":
        total = n_c * C + T
        s["pc"] = pc = _context(case, 2 * B * n_c, C, total, L)
        ids = g.host.permutation(2 * B * n_c)[:B * n_c]
        s["ids"] = ids.reshape(B, n_c).astype(np.int32)
        if case["mode"] == "reuse":
            _fill(pc, case, g, [int(x) for x in ids], _lengths(case, g, B * n_c), L)
            s["h"] = g.normal(B, T, H)
            s["table"] = pc.percache_chunk_table_put(s["ids"]) if case["table"] else None
        else:
            s["h"] = g.normal(B, total, H)
            s["bounds"] = [c * C for c in range(n_c + 1)]
            s["k"], s["v"] = (torch.empty((L, n_c, Hkv, C, D), dtype=torch.bfloat16, device=DEV) for _ in range(2))
        s["h_out"] = torch.empty_like(s["h"])
        return s
    # answer: slots of the chunks, then one slot per query for its prompt and the generated tokens
    own_cap = (T + case["new"] + 63) // 64 * 64
    s["pc"] = pc = _context(case, B * n_c + B, max(C, own_cap), n_c * C + T + case["new"], L)
    ids = g.host.permutation(B * n_c + B)
    s["ids"], s["own"] = ids[:B * n_c].reshape(B, n_c).astype(np.int32), [int(x) for x in ids[B * n_c:]]
    s["chain"] = np.concatenate([s["ids"], np.asarray(s["own"], np.int32)[:, None]], axis=1)
    _fill(pc, case, g, [int(x) for x in s["ids"].reshape(-1)], _lengths(case, g, B * n_c), L)
    s["h"] = g.normal(B, T, H) if T else None
    s["h_out"] = torch.empty_like(s["h"]) if T else None
    s["tok"] = [g.normal(B, 1, H) for _ in range(case["new"])]
    s["tok_out"] = [torch.empty_like(t) for t in s["tok"]]
    return s


# ------------------------------------------------------------------------------------------------ one pass
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "front":
        s["qa"].percache_lookup(s["probes"], TAU, *s["out"])
        return s["out"] + (s["chunks"].percache_lookup_topk(s["probes"], case["k"]) if case["k"] else ())
    if kind == "refresh":
        return s["qa"].percache_bank_refresh_scan(s["new"], s["kth"])
    pc = s["pc"]
    if kind == "store":
        pc.percache_kv_put_batch(0, s["slots"], s["k"], s["v"])
        return pc.percache_kv_get_batch(0, s["slots"], case["tokens"], s["ko"], s["vo"])
    if kind == "layer":
        if s["table"] is not None:
            pc.percache_prefill_reuse_table(0, s["x"], s["w"], s["table"], s["attn"], s["kf"], s["vf"])
        else:
            pc.percache_prefill_reuse(0, s["x"], s["w"], s["ids"], attn_out=s["attn"], k_fresh_out=s["kf"], v_fresh_out=s["vf"])
        if case["save"]:
            pc.percache_kv_put_batch(0, s["spare"], s["kf"], s["vf"])
        return s["attn"], s["kf"], s["vf"]
    F = SHAPES[case["shape"]][4]
    if kind == "stack":
        if case["mode"] == "populate":
            pc.percache_stack_reuse(s["layers"], F, EPS, s["h"], save_bounds=s["bounds"], save_slots=s["ids"], h_out=s["h_out"])
            for layer in range(case["layers"]):
                pc.percache_kv_get_batch(layer, s["ids"][0], case["chunk"], s["k"][layer], s["v"][layer])
            return s["h_out"], s["k"], s["v"]
        if s["table"] is not None:
            pc.percache_stack_reuse_table(s["layers"], F, EPS, s["h"], s["table"], s["h_out"])
        else:
            pc.percache_stack_reuse(s["layers"], F, EPS, s["h"], s["ids"], h_out=s["h_out"])
        return s["h_out"]
    started = case["fresh"] > 0
    if started:   # the prompt's own K/V go to the query's slot
        pc.percache_stack_reuse(s["layers"], F, EPS, s["h"], s["ids"], save_bounds=[0, case["fresh"]],
                                save_slots=[[o] for o in s["own"]], h_out=s["h_out"])
    else:         # a new answer behind a prompt that is cached as a whole
        for layer in range(case["layers"]):
            for o in s["own"]:
                pc.percache_kv_evict(layer, o)
    for x, y in zip(s["tok"], s["tok_out"]):
        pc.percache_stack_decode(s["layers"], F, EPS, x, s["chain"] if started else s["ids"], s["own"], h_out=y)
        started = True
    return ([s["h_out"]] if case["fresh"] else []) + s["tok_out"]


# ------------------------------------------------------------------------------------------------ what a pass cannot do without
def _kv_bytes(case, tokens):
    _, _, Hkv, D, _ = SHAPES[case["shape"]]
    per = 2.0 * Hkv * D * 2
    return tokens * per * {"bf16": 1.0, "8bit": 0.5, "mixed": 0.75}[case["slots"]]


def _block_flops(case, rows):
    H, Hq, Hkv, D, F = SHAPES[case["shape"]]
    return 2.0 * rows * ((Hq + 2 * Hkv) * D * H + Hq * D * H + 3 * F * H)


def _block_bytes(case):
    H, Hq, Hkv, D, F = SHAPES[case["shape"]]
    return 2.0 * ((Hq + 2 * Hkv) * D * H + Hq * D * H + 3 * F * H)


def work(case):
    kind = case["kind"]
    if kind == "front":
        P, d, k = case["probes"], case["dim"], case["k"]
        rows = case["qa_rows"] + (case["chunk_rows"] if k else 0)
        return {"bytes": rows * (d * 2.0 + 4) + P * d * 2.0 + P * (9 + 8.0 * k), "flops": 2.0 * rows * d * P}
    if kind == "refresh":
        n, d, rows = case["new"], case["dim"], case["qa_rows"]
        return {"bytes": rows * (d * 2.0 + 4 + 4 + 9) + n * d * 2.0, "flops": 2.0 * rows * d * n}
    H, Hq, Hkv, D, F = SHAPES[case["shape"]]
    if kind == "store":   # dense tensors in, slots written, slots read, dense tensors out
        dense = case["chunks"] * case["tokens"] * 2.0 * Hkv * D * 2
        return {"bytes": 2 * dense + 2 * _kv_bytes(case, case["chunks"] * case["tokens"]), "flops": 0}
    B, T = case["batch"], case["fresh"]
    pre = case["chunks"] * case["chunk"] * (0.75 if case["ragged"] else 1.0)   # mean cached length of a query
    attn = lambda rows, keys: 4.0 * B * Hq * D * rows * keys  # noqa: E731
    if kind == "layer":
        n_out = (Hq + 2 * Hkv) * D
        fresh_kv = B * T * 2.0 * Hkv * D * 2
        return {"bytes": 2.0 * (B * T * H + n_out * H + B * T * Hq * D) + fresh_kv + _kv_bytes(case, B * pre) + (_kv_bytes(case, B * T) if case["save"] else 0),
                "flops": 2.0 * B * T * H * n_out + attn(T, pre + (T + 1) / 2)}
    L = case["layers"]
    if kind == "stack" and case["mode"] == "populate":
        total = case["chunks"] * case["chunk"] + T
        dense = case["chunks"] * case["chunk"] * 2.0 * Hkv * D * 2
        return {"bytes": L * (_block_bytes(case) + 2 * _kv_bytes(case, case["chunks"] * case["chunk"]) + dense) + 4.0 * total * H,
                "flops": L * (_block_flops(case, total) + attn(total, (total + 1) / 2))}
    if kind == "stack":
        return {"bytes": L * (_block_bytes(case) + _kv_bytes(case, B * pre)) + 4.0 * B * T * H,
                "flops": L * (_block_flops(case, B * T) + attn(T, pre + (T + 1) / 2))}
    n = case["new"]
    b = L * (_block_bytes(case) + _kv_bytes(case, B * (pre + T))) + 4.0 * B * T * H if T else 0.0
    f = L * (_block_flops(case, B * T) + attn(T, pre + (T + 1) / 2)) if T else 0.0
    for i in range(n):
        b += L * (_block_bytes(case) + _kv_bytes(case, B * (pre + T + i + 1))) + 4.0 * B * H
        f += L * (_block_flops(case, B) + attn(1, pre + T + i + 1))
    return {"bytes": b, "flops": f}


def tolerance(case):
    kind = case["kind"]
    if kind == "store":
        return "exact"   # copies, and codes whose rounding is fixed
    if kind in ("front", "refresh"):
        # fp32 sums of at most 1024 exact fp16 products: 2e-7 (one value: 1e-6) from the sums in 64 bits; an index may
        # differ where two similarities are closer than that (none did)
        return {"rel": 2e-6, "max": 1e-5, "differ": 0.002}
    if kind == "layer":
        # attention 3.5e-3 (largest 2.3e-2), fresh K and V 1.7e-3 from the same pass unrounded: one rounding to bf16 of
        # q, k, v, the probabilities and the result
        return {"rel": 1.4e-2, "max": 0.1}
    # hidden states kept in bf16 between the steps of a block: from the same stack unrounded 8e-3 after 4 layers, 1.2e-2
    # after 8 and 1.4e-2 to 1.75e-2 (largest 9e-2) after 20 to 28
    return {"rel": min(3e-2, 1.6e-2 * case["layers"] ** 0.5), "max": 0.36}
