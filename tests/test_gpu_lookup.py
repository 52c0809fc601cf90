"""GPU parity of the query-level match (Sec. 4.2.1) against the CPU oracle, through the C ABI.

Bar: index and hit flag bit-exact, except that where the oracle's two best similarities differ by less
than 1e-4 any index whose oracle similarity is within 1e-4 of the best is accepted; similarity within 2e-5.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_11553_amd import workloads as wl
from paper_2601_11553_amd.binding import KERNEL_LOOKUP, Percache, PercacheError

from gpu_util import DEV, f16, host

pytestmark = pytest.mark.gpu


def _ctx(capacity, dim):
    return Percache(n_layers=1, hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, n_slots=1, slot_capacity=64,
                    max_pos=64, bank_capacity=capacity, emb_dim=dim, device=DEV)


def _compare(bank, probes, tau, idx, sim, hit):
    o_idx, o_sim, o_hit, o_sim2 = oracle.lookup(bank, probes, tau)
    idx, sim, hit = idx.cpu().numpy(), sim.cpu().numpy(), hit.cpu().numpy()
    assert np.abs(sim - o_sim).max() < 2e-5, np.abs(sim - o_sim).max()
    clear = (o_sim - o_sim2) >= 1e-4
    assert np.array_equal(idx[clear], o_idx[clear]), np.nonzero(idx[clear] != o_idx[clear])
    for p in np.nonzero(~clear)[0]:
        s = oracle.similarities(bank, probes[p])
        assert o_sim[p] - s[idx[p]] < 1e-4
    assert np.array_equal(hit, o_hit)
    return int((~clear).sum())


def test_config0_lookup():
    w = wl.lookup_config0("f16")
    pc = _ctx(64, 128)
    pc.percache_bank_put(0, f16(w.bank))
    assert pc.percache_bank_size() == 64
    idx, sim, hit = pc.percache_lookup(f16(w.probes), w.tau)
    torch.cuda.synchronize()
    _compare(w.bank, w.probes, w.tau, idx, sim, hit)
    assert idx[0].item() == w.source[0] and hit[0].item() == 1 and abs(sim[0].item() - 1.0) < 1e-3
    assert hit[1:].sum().item() == 0


@pytest.mark.parametrize("n_clusters,per_cluster,n_probes", [(37, 27, 70), (50, 100, 16), (13, 5, 1), (64, 64, 130)])
def test_clustered_ragged_sizes(n_clusters, per_cluster, n_probes):
    """Bank sizes that are not multiples of the 16-row block, probe counts across the 32-probe pass."""
    w = wl.lookup_clustered("t", 11, n_clusters, per_cluster, 1024, n_probes, 0.05, 0.02, 0.92, n_exact=3, n_near=3)
    N = w.bank.shape[0]
    pc = _ctx(N + 5, 1024)
    # two puts: appends must continue where the first stopped
    cut = N // 3
    pc.percache_bank_put(0, f16(w.bank[:cut]))
    pc.percache_bank_put(cut, f16(w.bank[cut:]))
    idx, sim, hit = pc.percache_lookup(f16(w.probes), w.tau)
    torch.cuda.synchronize()
    _compare(w.bank, w.probes, w.tau, idx, sim, hit)
    assert hit[-6:].all()


@pytest.mark.parametrize("dim,n_probes", [(64, 5), (64, 20), (192, 7), (256, 31), (384, 9), (384, 25), (768, 3), (768, 33), (2048, 20),
                                          (512, 100), (512, 129), (768, 260), (1024, 128)])   # 512/100 and 1024/128: the 128-probe pass
def test_every_embedding_width(dim, n_probes):
    """Each row-chunk width of the streaming kernel (one chunk per row up to 256 elements, several beyond),
    with one and two probe blocks, on a bank long enough that every wavefront streams many row blocks."""
    w = wl.lookup_clustered("w", 100 + dim, 1031, 97, dim, n_probes, 0.05, 0.02, 0.92, n_exact=1, n_near=1)
    N = w.bank.shape[0]
    pc = _ctx(N, dim)
    pc.percache_bank_put(0, f16(w.bank))
    idx, sim, hit = pc.percache_lookup(f16(w.probes), w.tau)
    torch.cuda.synchronize()
    _compare(w.bank, w.probes, w.tau, idx, sim, hit)


@pytest.mark.parametrize("seed", list(range(16)))
def test_seeded_random_bank_shapes(seed):
    """Embedding width, bank size (ragged against every block size) and probe count drawn from a seed: every kernel
    of the lookup (one or two probe blocks per pass, the 128-probe pass, the matrix-product kernel) meets odd sizes."""
    g = np.random.default_rng(3000 + seed)
    dim = int(g.choice([64, 128, 192, 256, 384, 512, 768, 1024]))
    n_clusters = int(g.integers(1, 60))
    per_cluster = int(g.integers(1, 70))
    n_probes = int(g.choice([1, 5, 16, 17, 32, 33, 100, 128, 129, 200]))
    w = wl.lookup_clustered("r", 3100 + seed, n_clusters, per_cluster, dim, n_probes, 0.05, 0.02, 0.92, n_exact=1, n_near=1)
    pc = _ctx(w.bank.shape[0], dim)
    pc.percache_bank_put(0, f16(w.bank))
    idx, sim, hit = pc.percache_lookup(f16(w.probes), w.tau)
    torch.cuda.synchronize()
    _compare(w.bank, w.probes, w.tau, idx, sim, hit)


def test_ties_zero_vectors_and_empty_bank():
    d = 128
    g = np.random.default_rng(5)
    bank = wl.round_f16(g.standard_normal((40, d)).astype(np.float32))
    bank[7] = 0.0                    # zero-norm row: similarity 0
    bank[30] = bank[12] * 2.0        # same direction as row 12: exact tie, lowest index wins
    probes = np.stack([bank[12], np.zeros(d, np.float32), bank[30] * 0.5, -bank[3]]).astype(np.float32)
    pc = _ctx(64, d)
    idx, sim, hit = pc.percache_lookup(f16(probes), 0.5)
    torch.cuda.synchronize()
    assert idx.cpu().tolist() == [-1] * 4 and not hit.any().item() and torch.isneginf(sim).all().item()
    pc.percache_bank_put(0, f16(bank))
    idx, sim, hit = pc.percache_lookup(f16(probes), 0.5)
    torch.cuda.synchronize()
    o_idx, o_sim, o_hit, _ = oracle.lookup(bank, probes, 0.5)
    assert idx.cpu().tolist() == o_idx.tolist()
    assert idx[0].item() == 12 and idx[2].item() == 12 and idx[1].item() == 0
    assert np.array_equal(hit.cpu().numpy(), o_hit)
    assert np.abs(sim.cpu().numpy() - o_sim).max() < 2e-5


@pytest.mark.parametrize("n_probes,k", [(40, 1), (128, 1), (40, 8)])
def test_ties_and_zero_vectors_in_the_128_probe_pass(n_probes, k):
    """Exact ties (lowest row wins), a zero row, a zero probe and a ragged last 32-row block, at a width and probe
    counts the 128-probe pass takes."""
    d = 512
    g = np.random.default_rng(15)
    bank = wl.round_f16(g.standard_normal((75, d)).astype(np.float32))
    bank[7] = 0.0
    bank[40] = bank[12] * 2.0
    bank[70] = bank[12] * 0.5
    probes = wl.round_f16(g.standard_normal((n_probes, d)).astype(np.float32))
    probes[0] = bank[12]
    probes[1] = 0.0
    probes[n_probes - 1] = bank[70]
    pc = _ctx(128, d)
    pc.percache_bank_put(0, f16(bank))
    if k == 1:
        idx, sim, hit = pc.percache_lookup(f16(probes), 0.5)
        torch.cuda.synchronize()
        o_idx, o_sim, o_hit, _ = oracle.lookup(bank, probes, 0.5)
        assert idx.cpu().tolist() == o_idx.tolist()
        assert idx[0].item() == 12 and idx[n_probes - 1].item() == 12 and idx[1].item() == 0
        assert np.array_equal(hit.cpu().numpy(), o_hit)
        assert np.abs(sim.cpu().numpy() - o_sim).max() < 2e-5
    else:
        idx, sim = pc.percache_lookup_topk(f16(probes), k)
        torch.cuda.synchronize()
        assert idx[0, :3].cpu().tolist() == [12, 40, 70] and idx[1, :k].cpu().tolist() == list(range(k))
        _compare_topk(bank, probes, k, idx, sim)


@pytest.mark.parametrize("n_rows,d,n_probes", [(75, 512, 200), (300, 64, 256), (1031, 192, 600), (5000, 1024, 1000),
                                                (257, 128, 1152), (256, 256, 768), (3, 64, 250),
                                                (1031, 192, 150), (300, 64, 100), (5000, 1024, 170), (75, 128, 33), (600, 256, 300),
                                                (700, 128, 3000), (1, 64, 300), (2100, 2048, 384)])
def test_ties_zero_vectors_and_ragged_ends_in_the_256_row_tiles(n_rows, d, n_probes):
    """The matrix-product kernel on 256-row tiles (best match only; 256-probe tiles where the probes fill them to three
    quarters, 128-probe tiles with the deeper ring otherwise; more probe tiles than CUs / 8; a one-row bank): exact ties
    (lowest row wins) inside one lane's rows, across lanes, across wavefronts and across tiles; a zero row and a zero probe; banks that end inside a tile, inside a 32-row block, or hold fewer
    rows than one block; a single k-step (64 elements) and many."""
    g = np.random.default_rng(n_rows + d)
    bank = wl.round_f16(g.standard_normal((n_rows, d)).astype(np.float32))
    probes = wl.round_f16(g.standard_normal((n_probes, d)).astype(np.float32))
    probes[1] = 0.0
    if n_rows >= 75:
        bank[7] = 0.0
        bank[40] = bank[12] * 2.0     # same cosine as row 12: another 32-row block, another wavefront
        bank[13] = bank[12] * 0.5     # the next row: same lane or its neighbour
        bank[70] = bank[12] * 0.25
        probes[0] = bank[12]
        probes[n_probes - 1] = bank[70]
    if n_rows >= 300:
        bank[n_rows - 1] = bank[12] * 4.0   # the bank's last row, in a later tile: the earlier tile's row keeps the match
        bank[290] = bank[280]               # a tie that the later tile opens and wins by row order
        probes[5] = bank[290]
    pc = _ctx(n_rows + 3, d)
    pc.percache_bank_put(0, f16(bank))
    idx, sim, hit = pc.percache_lookup(f16(probes), 0.5)
    torch.cuda.synchronize()
    o_idx, o_sim, o_hit, o_sim2 = oracle.lookup(bank, probes, 0.5)
    if n_rows >= 75:
        assert idx[0].item() == 12 and idx[n_probes - 1].item() == 12
    if n_rows >= 300:
        assert idx[5].item() == 280
    assert idx[1].item() == 0
    _compare(bank, probes, 0.5, idx, sim, hit)
    # scaled copies have equal cosines only up to rounding of the norms: the planted rows are checked above, the rest by _compare


def test_overwrite_rows_and_error_paths():
    d = 128
    g = np.random.default_rng(6)
    bank = wl.round_f16(g.standard_normal((32, d)).astype(np.float32))
    pc = _ctx(64, d)
    pc.percache_bank_put(0, f16(bank))
    new = wl.round_f16(g.standard_normal((4, d)).astype(np.float32))
    pc.percache_bank_put(10, f16(new))
    bank[10:14] = new
    probes = np.concatenate([new[:2], bank[:2]])
    idx, sim, hit = pc.percache_lookup(f16(probes), 0.9)
    torch.cuda.synchronize()
    assert idx.cpu().tolist() == [10, 11, 0, 1] and hit.all().item()
    with pytest.raises(PercacheError) as e:
        pc.percache_bank_put(32, f16(np.concatenate([bank, bank[:8]])))   # 32 + 40 rows > capacity 64
    assert e.value.status == -5
    with pytest.raises(PercacheError) as e:
        pc.percache_bank_put(40, f16(bank[:1]))                           # would leave a hole
    assert e.value.status == -1
    assert pc.percache_bank_size() == 32
    nobank = Percache(n_layers=1, hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, n_slots=1, slot_capacity=64,
                      max_pos=64, device=DEV)
    with pytest.raises(PercacheError) as e:
        nobank.percache_lookup(f16(probes), 0.9)
    assert e.value.status == -2


def test_config3_full_size_every_probe():
    """200k x 1024 fp16 bank, the 1024 probes of the recipe plus the hit-branch block; every one of the 1152 probes
    goes through the oracle's exhaustive scan."""
    w = wl.lookup_config3(n_exact=64, n_near=64)
    N, d = w.bank.shape
    P = w.probes.shape[0]
    pc = _ctx(N, d)
    pc.percache_bank_put(0, f16(w.bank))
    probes_dev = f16(w.probes)
    idx, sim, hit = pc.percache_lookup(probes_dev, w.tau)
    torch.cuda.synchronize()
    # one probe at a time (the paper's case) must give the same answers as the batched call
    for p in (0, 513, P - 1):
        i1, s1, h1 = pc.percache_lookup(probes_dev[p:p + 1], w.tau)
        torch.cuda.synchronize()
        assert i1.item() == idx[p].item() and h1.item() == hit[p].item() and abs(s1.item() - sim[p].item()) < 2e-6
    # 128 probes go through the 128-probe pass, the full call through the matrix-product kernel: same answers
    for lo in (0, 1000):
        i3, s3, h3 = pc.percache_lookup(probes_dev[lo:lo + 128], w.tau)
        torch.cuda.synchronize()
        assert torch.equal(i3, idx[lo:lo + 128]) and torch.equal(h3, hit[lo:lo + 128]) and (s3 - sim[lo:lo + 128]).abs().max().item() < 2e-6
    print("cfg3: oracle scan of all probes ...", flush=True)
    n_near_ties = _compare(w.bank, w.probes, w.tau, idx, sim, hit)
    print(f"cfg3: {P} probes through the oracle, {n_near_ties} with top-2 gap < 1e-4; hits in main block "
          f"{int(hit[:1024].sum())}/1024, in hit block {int(hit[1024:].sum())}/128", flush=True)
    idx_h, hit_h = idx.cpu().numpy(), hit.cpu().numpy()
    copies = w.source[:1024] >= 0
    assert np.array_equal(idx_h[:1024][copies], w.source[:1024][copies])   # perturbed copies find their source
    assert hit_h[1024:].all() and np.array_equal(idx_h[1024:], w.source[1024:])


def _compare_topk(bank, probes, k, idx, sim):
    o_idx, o_sim, o_next = oracle.lookup_topk(bank, probes, k)
    idx, sim = idx.cpu().numpy(), sim.cpu().numpy()
    fin = np.isfinite(o_sim)
    assert np.array_equal(np.isfinite(sim), fin) and np.array_equal(idx[~fin], o_idx[~fin])
    assert np.abs(sim[fin] - o_sim[fin]).max() < 2e-5
    n_loose = 0
    for p in range(probes.shape[0]):
        assert len(set(idx[p][fin[p]])) == int(fin[p].sum())                      # no row twice
        ranked = np.concatenate([o_sim[p], [o_next[p]]])
        s_all = None
        for j in range(k):
            if not fin[p, j]:
                continue
            clear = (j == 0 or ranked[j - 1] - ranked[j] >= 1e-4) and ranked[j] - ranked[j + 1] >= 1e-4
            if clear:
                assert idx[p, j] == o_idx[p, j], (p, j)
            else:                                                                   # near-tie: any row that close is right
                if s_all is None:
                    s_all = oracle.similarities(bank, probes[p])
                assert abs(s_all[idx[p, j]] - o_sim[p, j]) < 1e-4, (p, j)
                n_loose += 1
    return n_loose


@pytest.mark.parametrize("dim,n_probes,k", [(1024, 40, 8), (1024, 3, 3), (128, 17, 5), (384, 33, 2), (64, 5, 8), (1024, 150, 8), (192, 300, 4)])
def test_topk_vs_oracle(dim, n_probes, k):
    w = wl.lookup_clustered("k", 300 + dim, 523, 41, dim, n_probes, 0.05, 0.02, 0.92, n_exact=1, n_near=1)
    pc = _ctx(w.bank.shape[0], dim)
    pc.percache_bank_put(0, f16(w.bank))
    idx, sim = pc.percache_lookup_topk(f16(w.probes), k)
    i1, s1, _ = pc.percache_lookup(f16(w.probes), w.tau)
    torch.cuda.synchronize()
    loose = _compare_topk(w.bank, w.probes, k, idx, sim)
    assert torch.equal(idx[:, 0], i1) and torch.equal(sim[:, 0], s1)              # rank 1 is the query-level match
    print(f"top-{k}: {loose} near-tie entries judged by similarity", flush=True)


# rows around the kernels' groups: every row one (up to 8192, past 128 probes 4096), one block, a group's worth more and less, groups of several blocks (stream and wide from 65 536 rows on, tiles from
# 16 384), the last workgroup's part empty or ragged; 32 | 33, 128 | 129 and 192 probes are other kernels
@pytest.mark.parametrize("rows,dim,n_probes,k", [
    (3, 128, 2, 8), (16, 64, 9, 8), (17, 384, 33, 5), (1025, 512, 64, 8), (8192, 512, 33, 3), (8193, 768, 128, 8), (5003, 1024, 70, 8), (4097, 64, 200, 8), (16384, 64, 130, 8), (16385, 64, 130, 8),
    (8191, 64, 32, 5), (8192, 640, 7, 8), (8193, 64, 20, 8), (4093, 128, 260, 8), (4096, 64, 129, 3), (65536, 128, 16, 3), (65553, 64, 32, 8), (140001, 64, 5, 2), (70001, 512, 40, 8), (70001, 768, 128, 3), (40001, 1024, 8, 8), (33000, 64, 300, 5)])
def test_topk_groups(rows, dim, n_probes, k):
    """Planted beside random rows: copies of a row in its group and far away, zero rows, rows that are not numbers; probes near the copies (two of the
    best in one group) and a zero probe (every similarity the same).  In a workspace that holds the groups and in the smallest one taken.
    Bound on similarities: fp32 sums of at most 1024 exact products of unit vectors, 2e-6."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + dim)
    bank = torch.randn((rows, dim), generator=g, device=DEV).half()
    probes = torch.randn((n_probes, dim), generator=g, device=DEV).half()
    copies = sorted({r for r in (1, 5, 11, rows // 2, rows - 1) if 0 < r < rows})
    if rows > 16:
        for r in copies[1:]:
            bank[r] = bank[1]
        bank[7], bank[2], bank[0] = 0, float("nan"), float("inf")
    probes[0] = bank[1] if rows > 1 else probes[0]
    probes[1] = 0
    pc = _ctx(rows + 3, dim)
    pc.percache_bank_put(0, bank)
    idx, sim = pc.percache_lookup_topk(probes, k)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    least = max(n_cu * (256 if n_probes > 32 else 32), ((rows + 3) // 2048 + 1) * 32, ((rows + 3) // 6144 + 1) * 128) * 64
    ws = torch.full((least + 256,), 255, dtype=torch.uint8, device=DEV)
    i2, s2 = torch.empty_like(idx), torch.empty_like(sim)
    pc._check(pc.lib.percache_lookup_topk(pc.ctx, probes.data_ptr(), n_probes, k, i2.data_ptr(), s2.data_ptr(), (ws.data_ptr() + 255) // 256 * 256, least,
                                          torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    b, p = bank.double(), probes.double()
    counts = torch.isfinite(b).all(dim=1)
    unit = lambda x: x / x.norm(dim=1, keepdim=True).clamp(min=1e-30)  # noqa: E731
    ref = unit(p) @ unit(torch.where(counts[:, None], b, 0.0)).t()
    ref = torch.where(counts[None], ref, float("-inf"))
    want, order = torch.sort(ref, dim=1, descending=True, stable=True)
    kk = min(k, int(counts.sum()))
    for i, s in ((idx, sim), (i2, s2)):
        assert (i[:, kk:] == -1).all() and torch.isneginf(s[:, kk:]).all()
        got = torch.gather(ref, 1, i[:, :kk].long())
        assert (got - want[:, :kk]).abs().max().item() < 2e-6 and (s[:, :kk].double() - got).abs().max().item() < 2e-6
        assert all(len(set(r)) == kk for r in i[:, :kk].tolist())
        assert i[1, :kk].tolist() == order[1, :kk].tolist()                                   # equal similarities: lower rows first
        if rows > 16:
            assert i[0, :min(kk, len(copies))].tolist() == copies[:kk]
    pc.close()


@pytest.mark.parametrize("rows,dim,n_probes", [(70001, 128, 16), (70001, 512, 40), (70001, 512, 128), (20011, 64, 300), (3001, 64, 200)])
@pytest.mark.parametrize("copies", [9, 65, 300, 1000])
def test_topk_many_equal_groups(rows, dim, n_probes, copies):
    """Copies of a row in as many groups or nearly so: more candidates than a wavefront ranks, up to nearly as many as there is room for.  The lowest rows,
    for a probe that is the row, for one near it and, of all rows, for a zero probe."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + copies)
    bank = torch.randn((rows, dim), generator=g, device=DEV).half()
    probes = torch.randn((n_probes, dim), generator=g, device=DEV).half()
    at = torch.unique((torch.arange(copies, device=DEV) * (rows - 40) // copies) + 3)
    bank[at] = bank[3].clone()
    near = [i for i in range(0, n_probes, 3)]
    probes[near] = bank[3].clone()
    probes[near[1:]] += (0.02 * torch.randn((len(near) - 1, dim), generator=g, device=DEV)).half()
    probes[1] = 0
    pc = _ctx(rows, dim)
    pc.percache_bank_put(0, bank)
    idx, sim = pc.percache_lookup_topk(probes, 8)
    torch.cuda.synchronize()
    assert (idx[near] == at[:8][None]).all() and (sim[near] == sim[near][:, :1]).all()
    assert idx[1].tolist() == list(range(8)) and (sim[1] == 0).all()
    pc.close()


@pytest.mark.parametrize("rows,dim,n_probes", [(200, 64, 1024), (6000, 768, 1), (70001, 512, 40), (140001, 64, 20), (20011, 64, 300), (33001, 64, 1024), (33001, 64, 1200), (3001, 64, 2500), (9001, 640, 100)])
def test_topk_in_the_lookups_workspace(rows, dim, n_probes):
    """The workspace of a call for the best row is as large as lists in every workgroup take, on any bank, and a call for 8 rows takes it as well: one
    pass of the bank for up to 1024 probes, a few more for more of them, and the rows it finds in the larger one."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + dim)
    bank = torch.randn((rows, dim), generator=g, device=DEV).half()
    bank[5:: 997] = bank[5].clone()
    probes = torch.randn((n_probes, dim), generator=g, device=DEV).half()
    probes[0] = bank[5]
    pc = _ctx(rows, dim)
    pc.percache_bank_put(0, bank)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    least = n_cu * (256 if n_probes > 32 else 32) * 64
    small, large = pc.lib.percache_lookup_workspace_bytes(pc.ctx, n_probes), pc.lib.percache_lookup_topk_workspace_bytes(pc.ctx, n_probes)
    assert small == least <= large <= n_probes * 4096 * 17 + least
    pc.percache_lookup(probes, 0.5)
    held = pc._lookup_ws.data_ptr()
    assert pc._lookup_ws.numel() == small + 256
    idx, sim = pc.percache_lookup_topk(probes, 8)
    pc.percache_lookup(probes, 0.5)
    assert pc._lookup_ws.data_ptr() == held
    ws = torch.full((small + 512,), 255, dtype=torch.uint8, device=DEV)
    at = (ws.data_ptr() + 255) // 256 * 256
    i2, s2 = torch.empty_like(idx), torch.empty_like(sim)
    pc.percache_profile_enable(True, kernels=[KERNEL_LOOKUP])
    pc._check(pc.lib.percache_lookup_topk(pc.ctx, probes.data_ptr(), n_probes, 8, i2.data_ptr(), s2.data_ptr(), at, small, torch.cuda.current_stream().cuda_stream))
    _, passes = pc.percache_profile_read(KERNEL_LOOKUP)
    pc.percache_profile_enable(False)
    assert passes == 1 if n_probes <= 4 * n_cu else passes <= -(-n_probes // 512)
    assert torch.equal(idx, i2) and torch.equal(sim, s2)
    assert (ws[at - ws.data_ptr() + small:] == 255).all()
    ref = torch.nn.functional.normalize(probes.double(), dim=1) @ torch.nn.functional.normalize(bank.double(), dim=1).t()
    want = torch.sort(ref, dim=1, descending=True, stable=True).values[:, :8]
    assert (torch.gather(ref, 1, idx.long()) - want).abs().max().item() < 2e-6    # (fp32 sums of at most 1024 exact products of unit vectors)
    assert pc.lib.percache_lookup_topk(pc.ctx, probes.data_ptr(), n_probes, 8, i2.data_ptr(), s2.data_ptr(), at, small - 1, 0) < 0
    pc.close()


# groups of 128 rows and more of each kind: the k groups in doubt hold more rows than there is room for, so the best are kept in between
@pytest.mark.parametrize("rows,dim,n_probes", [(530001, 64, 20), (225001, 512, 64), (225001, 512, 100), (200001, 64, 512), (16384, 64, 129)])
def test_topk_more_equal_rows_than_room(rows, dim, n_probes):
    """All rows alike but the first and one in the middle: the lowest ones, for the row itself, its opposite (the two other rows first) and a zero probe."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows)
    bank = torch.randn((1, dim), generator=g, device=DEV).half().repeat(rows, 1)
    bank[0], bank[rows // 2] = -bank[1], -bank[1]
    probes = bank[1:2].repeat(n_probes, 1)
    probes[2::3] = -bank[1]
    probes[1] = 0
    pc = _ctx(rows, dim)
    pc.percache_bank_put(0, bank)
    idx, _ = pc.percache_lookup_topk(probes, 8)
    torch.cuda.synchronize()
    want = torch.arange(1, 9, dtype=torch.int32, device=DEV).repeat(n_probes, 1)
    want[2::3] = torch.tensor([0, rows // 2, 1, 2, 3, 4, 5, 6], dtype=torch.int32, device=DEV)
    want[1] = torch.arange(8, dtype=torch.int32, device=DEV)
    assert torch.equal(idx, want)
    pc.close()


# from 32 768 rows on (256 CUs) 33 to 64 probes take blocks of two sets of 32 rows; the last block without a second set, with one row of it, whole
@pytest.mark.parametrize("rows,dim,n_probes", [(32768, 512, 33), (32769, 1024, 64), (32801, 768, 64), (49152, 512, 40), (33000, 384, 50)])
def test_two_sets_of_rows_a_block(rows, dim, n_probes):
    """Best rows and the refresh scan against 64 bits; equal rows in both sets and in other workgroups: the lowest one, of equal new chunks the lower one.
    Bound: fp32 sums of at most 1024 exact products of unit vectors, 2e-6."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows)
    bank = torch.randn((rows, dim), generator=g, device=DEV).half()
    probes = torch.randn((n_probes, dim), generator=g, device=DEV).half()
    for r in (70, 99, rows // 2, rows - 1):
        bank[r] = bank[40]
    bank[64], bank[rows - 2] = 0, float("nan")
    probes[n_probes - 1], probes[n_probes - 2] = bank[40], bank[40]
    probes[0] = 0
    pc = _ctx(rows, dim)
    pc.percache_bank_put(0, bank)
    kth = torch.full((rows,), 0.1, device=DEV)
    idx, sim, hit = pc.percache_lookup(probes, 0.1)
    best, new, stale = pc.percache_bank_refresh_scan(probes, kth)
    torch.cuda.synchronize()
    b, p = bank.double(), probes.double()
    unit = lambda x: x / x.norm(dim=1, keepdim=True).clamp(min=1e-30)  # noqa: E731
    ref = unit(p) @ unit(torch.nan_to_num(b)).t()
    ref[:, rows - 2] = float("-inf")
    got = torch.gather(ref, 1, idx.long()[:, None])[:, 0]
    assert (ref.max(dim=1).values - got).max().item() < 2e-6 and (sim.double() - got).abs().max().item() < 2e-6
    assert idx[n_probes - 1].item() == 40 and idx[0].item() == 0 and torch.equal(hit.bool(), sim > 0.1)
    ok = torch.arange(rows, device=DEV) != rows - 2
    got = torch.gather(ref, 0, new.long().clamp(min=0)[None])[0]
    assert (ref.max(dim=0).values - got)[ok].max().item() < 2e-6 and (best.double() - got)[ok].abs().max().item() < 2e-6
    assert new[rows - 2].item() == -1 and torch.isneginf(best[rows - 2]) and stale[rows - 2].item() == 0
    assert all(new[r].item() == n_probes - 2 for r in (40, 70, 99, rows // 2, rows - 1)) and new[64].item() == 0
    assert torch.equal(stale.bool()[ok], (best > kth)[ok])
    pc.close()


@pytest.mark.parametrize("dim,n_first,n_last", [(64, 32, 16), (128, 32, 16), (256, 64, 5), (640, 32, 16), (640, 96, 16), (2048, 16, 16), (384, 128, 16), (1024, 128, 40)])
def test_refresh_scan_equal_chunks_in_different_passes(dim, n_first, n_last):
    """The last pass of a call takes fewer new chunks than the others; copies of earlier ones in it have the same similarities, so that the lower index
    stands."""
    g = torch.Generator(device=DEV)
    g.manual_seed(dim + n_first)
    rows = 40
    pc = _ctx(rows, dim)
    for _ in range(20):
        new = torch.randn((n_first + n_last, dim), generator=g, device=DEV)
        new = (new / new.norm(dim=1, keepdim=True)).half()
        new[n_first:] = new[:n_last].clone()
        pc.percache_bank_put(0, new[torch.arange(rows, device=DEV) % n_last].clone())   # (the best new chunk of a row is its copy)
        best, which, _ = pc.percache_bank_refresh_scan(new, torch.zeros(rows, device=DEV))
        assert which.tolist() == [r % n_last for r in range(rows)]
    pc.close()


def test_topk_ties_small_bank_and_errors():
    d = 128
    g = np.random.default_rng(12)
    bank = wl.round_f16(g.standard_normal((5, d)).astype(np.float32))
    bank[3] = bank[1] * 2.0
    probes = np.stack([bank[1], bank[4]])
    pc = _ctx(16, d)
    idx, sim = pc.percache_lookup_topk(f16(probes), 4)
    torch.cuda.synchronize()
    assert (idx == -1).all().item() and torch.isneginf(sim).all().item()           # empty bank
    pc.percache_bank_put(0, f16(bank))
    idx, sim = pc.percache_lookup_topk(f16(probes), 8)
    torch.cuda.synchronize()
    assert idx[0, :2].tolist() == [1, 3] and (idx[:, 5:] == -1).all().item() and torch.isneginf(sim[:, 5:]).all().item()
    o_idx, o_sim, _ = oracle.lookup_topk(bank, probes, 8)
    assert np.array_equal(idx.cpu().numpy(), o_idx)
    with pytest.raises(PercacheError) as e:
        pc.percache_lookup_topk(f16(probes), 9)
    assert e.value.status == -2


@pytest.mark.parametrize("dim,n_new", [(1024, 5), (1024, 70), (128, 33)])
def test_refresh_scan_vs_oracle(dim, n_new):
    """Cache refresh (Sec. 4.1.3): stored queries in the bank, thresholds from the oracle's top-k over the chunk embeddings,
    new chunks scanned; against the oracle's row-by-row definition, and against a direct re-ranking."""
    k = 3
    wq = wl.lookup_clustered("q", 500 + dim, 97, 53, dim, 4, 0.05, 0.02, 0.92)       # bank rows = stored queries
    wc = wl.lookup_clustered("c", 600 + dim, 97, 31, dim, 4, 0.05, 0.02, 0.92)       # bank rows = knowledge chunks
    g = np.random.default_rng(dim + n_new)
    pick = g.integers(0, wq.bank.shape[0], size=n_new)
    new = wl.round_f16(wq.bank[pick] + 0.03 * g.standard_normal((n_new, dim)).astype(np.float32))
    _, o_sk, _ = oracle.lookup_topk(wc.bank, wq.bank, k)                              # each stored query's best chunks
    kth = torch.from_numpy(np.ascontiguousarray(o_sk[:, k - 1], np.float32)).to(DEV)
    qctx = _ctx(wq.bank.shape[0], dim)
    qctx.percache_bank_put(0, f16(wq.bank))
    best_sim, best_new, stale = qctx.percache_bank_refresh_scan(f16(new), kth)
    torch.cuda.synchronize()
    o_sim, o_new, o_stale = oracle.refresh_scan(wq.bank, new, kth.cpu().numpy())
    bs, bn, st = best_sim.cpu().numpy(), best_new.cpu().numpy(), stale.cpu().numpy()
    assert np.abs(bs - o_sim).max() < 2e-5
    loose = 0
    for j in np.nonzero(bn != o_new)[0]:                                              # only near-ties may differ
        s = oracle.similarities(new, wq.bank[j])
        assert o_sim[j] - s[bn[j]] < 1e-4
        loose += 1
    margin = np.abs(o_sim - kth.cpu().numpy()) > 2e-5           # the similarity tolerance: closer than that, either decision
    assert np.array_equal(st[margin], o_stale[margin])
    assert st[pick].all()                                                             # a near copy of a query enters its top-k
    print(f"refresh scan: {int(st.sum())}/{st.size} stored queries outdated, {loose} near-tie indices", flush=True)


@pytest.mark.parametrize("dim,n_new,rows", [(384, 33, 22309), (512, 64, 8192), (768, 128, 16385), (1024, 129, 31), (1024, 100, 30000)])
def test_refresh_scan_wide_passes(dim, n_new, rows):
    """More than 32 new chunks: 128 a pass of the bank, several row blocks per workgroup, a ragged last one, exact ties."""
    g = np.random.default_rng(rows + n_new)
    bank = wl.round_f16(g.standard_normal((rows, dim)).astype(np.float32))
    new = wl.round_f16(g.standard_normal((n_new, dim)).astype(np.float32))
    new[n_new - 1] = new[3]                                       # the same similarity twice: the lower index wins
    bank[rows // 2] = new[3]
    bank[rows - 1] = 0.0                                          # a zero row: every similarity is 0
    kth = torch.full((rows,), 0.1, device=DEV)
    qctx = _ctx(rows, dim)
    qctx.percache_bank_put(0, f16(bank))
    best_sim, best_new, stale = qctx.percache_bank_refresh_scan(f16(new), kth)
    torch.cuda.synchronize()
    bs, bn, st = best_sim.cpu().numpy(), best_new.cpu().numpy(), stale.cpu().numpy()
    o_sim, o_new, o_stale = oracle.refresh_scan(bank, new, kth.cpu().numpy())
    assert np.abs(bs - o_sim).max() < 2e-5
    assert bn[rows // 2] == 3 and bn[rows - 1] == 0 and bs[rows - 1] == 0.0
    for j in np.nonzero(bn != o_new)[0]:                          # only near-ties may differ
        s = oracle.similarities(new, bank[j])
        assert o_sim[j] - s[bn[j]] < 2e-5
    margin = np.abs(o_sim - 0.1) > 2e-5
    assert np.array_equal(st[margin], o_stale[margin])


@pytest.mark.parametrize("dim,n_new", [(384, 5), (384, 32), (384, 33), (512, 100), (1024, 64), (768, 130), (640, 40), (640, 16)])
def test_refresh_scan_rows_and_chunks_that_are_not_numbers(dim, n_new):
    """Bank rows with a NaN or an infinity have no similarity: index -1, similarity -inf, not outdated; a new chunk with a NaN
    takes no part.  One and several passes, streaming and 128-probe ones, with and without padding probes."""
    rows = 300
    g = np.random.default_rng(dim + n_new)
    bank = wl.round_f16(g.standard_normal((rows, dim)).astype(np.float32))
    new = wl.round_f16(g.standard_normal((n_new, dim)).astype(np.float32))
    bad = [0, 17, 130, rows - 1]
    bank[bad, 3] = [np.nan, np.inf, -np.inf, np.nan]
    new[2, dim - 1] = np.nan
    qctx = _ctx(rows, dim)
    qctx.percache_bank_put(0, f16(bank))
    best_sim, best_new, stale = qctx.percache_bank_refresh_scan(f16(new), torch.full((rows,), 0.05, device=DEV))
    torch.cuda.synchronize()
    bs, bn, st = best_sim.cpu().numpy(), best_new.cpu().numpy(), stale.cpu().numpy()
    assert (bn[bad] == -1).all() and (bs[bad] == -np.inf).all() and (st[bad] == 0).all()
    good = np.setdiff1d(np.arange(rows), bad)
    e, c = bank[good].astype(np.float64), new.astype(np.float64)
    sims = (e @ c.T) / (np.linalg.norm(e, axis=1)[:, None] * np.linalg.norm(c, axis=1)[None])
    sims[:, 2] = -np.inf
    assert np.abs(bs[good] - sims.max(1)).max() < 2e-5
    assert np.abs(sims[np.arange(len(good)), bn[good]] - sims.max(1)).max() < 2e-5
    clear = np.abs(sims.max(1) - 0.05) > 2e-5
    assert np.array_equal(st[good][clear] == 1, sims.max(1)[clear] > 0.05)


@pytest.mark.parametrize("rows,dim,k", [(1, 64, 1), (15, 384, 8), (2000, 768, 3), (4096, 768, 1), (4097, 768, 4), (4033, 128, 5), (4096, 2048, 2)])
def test_merge_inside_the_launch_equals_the_merge_apart(rows, dim, k):
    """Calls of up to 4 probes over at most 64 workgroups' rows merge their lists of up to 4 inside the launch, others and captured ones in a launch of
    their own: the same bits, whatever the workspace held, and again from a captured call replayed between eager ones."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + dim)
    pc = Percache(n_layers=1, hidden=64, n_q_heads=2, n_kv_heads=1, head_dim=64, n_slots=1, slot_capacity=64, max_pos=64, bank_capacity=rows, emb_dim=dim,
                  device=DEV)
    bank = torch.randn((rows, dim), generator=g, device=DEV).half()
    bank[rows // 2] = bank[0]                                  # a tie
    pc.percache_bank_put(0, bank)
    probes = torch.randn((16, dim), generator=g, device=DEV).half()
    probes[0] = bank[0]
    probes[5] = 0

    def call(p):
        return pc.percache_lookup(p, 0.3) if k == 1 else pc.percache_lookup_topk(p, k)
    apart = [t.clone() for t in call(probes)]                  # 16 probes
    for n in (1, 3, 4, 5, 9):
        for fill in (0, 255):
            pc._lookup_ws.fill_(fill)
            assert all(torch.equal(a[:n], b) for a, b in zip(apart, call(probes[:n].contiguous()))), (n, fill)
    few = probes[2:6].contiguous()
    call(few)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = call(few)
    for _ in range(4):
        for t in out:
            t.zero_()
        graph.replay()
        call(probes[:1].contiguous())
        torch.cuda.synchronize()
        assert all(torch.equal(a[2:6], b) for a, b in zip(apart, out))


@pytest.mark.parametrize("rows,dim,k", [(4096, 768, 1), (4096, 768, 3), (2000, 1024, 4), (2000, 2048, 8)])
def test_merge_inside_the_launch_beside_kernels_that_hold_the_cus(rows, dim, k):
    """Lookups whose workgroups get a CU only as another stream's long workgroups leave theirs, in whatever order that is: the bits of the call
    alone, eager and captured."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + dim)
    pc = Percache(n_layers=1, hidden=64, n_q_heads=2, n_kv_heads=1, head_dim=64, n_slots=1, slot_capacity=64, max_pos=64, bank_capacity=rows, emb_dim=dim,
                  device=DEV)
    pc.percache_bank_put(0, torch.randn((rows, dim), generator=g, device=DEV).half())
    probes = torch.randn((4, dim), generator=g, device=DEV).half()

    def call():
        return pc.percache_lookup(probes, 0.05) if k == 1 else pc.percache_lookup_topk(probes, k)
    alone = [t.clone() for t in call()]
    pc._lookup_ws.fill_(255)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = call()
    other = Percache(n_layers=1, hidden=64, n_q_heads=2, n_kv_heads=1, head_dim=64, n_slots=1, slot_capacity=64, max_pos=64, device=DEV)
    kv = torch.randn((8 << 20) // 2, generator=g, device=DEV).bfloat16()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        other.percache_peak_attention_tile_loop(kv, 16)
    torch.cuda.synchronize()
    outs = []
    for i in range(8):
        with torch.cuda.stream(side):
            for tiles in (700, 64):      # (of a millisecond, of a tenth)
                other.percache_peak_attention_tile_loop(kv, tiles)
        for _ in range(6):
            outs.append(call())
            graph.replay()
            outs.append([t.clone() for t in captured])
    torch.cuda.synchronize()
    for out in outs:
        assert all(torch.equal(a, b) for a, b in zip(alone, out))
    pc.close()
    other.close()
