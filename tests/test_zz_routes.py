"""Which kernel a call launches, where the result alone cannot tell.  The names come from torch's profiler, whose hooks lengthen every later launch of the
process: these tests come last, behind the ones that look at times."""
import numpy as np
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

from paper_2601_11553_amd import workloads as wl
from paper_2601_11553_amd.binding import Percache

from gpu_util import DEV, bf16, check_close, fill_slots, host, make_ctx
from test_gpu_prefill import SHARED_BLOCKS, TWO_HEAD_TILES

pytestmark = pytest.mark.gpu


def _kernels_of(call):
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    return [e.name for e in p.events() if e.device_type == torch.autograd.DeviceType.CUDA]


def _need_256_cus():
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the lines lie elsewhere")


@pytest.mark.parametrize("hidden,n_q_heads,n_kv_heads,batch,t_fresh,blocks", TWO_HEAD_TILES)
def test_which_projections_take_two_head_tiles(hidden, n_q_heads, n_kv_heads, batch, t_fresh, blocks):
    _need_256_cus()
    pc = Percache(n_layers=1, hidden=hidden, n_q_heads=n_q_heads, n_kv_heads=n_kv_heads, head_dim=128, n_slots=1, slot_capacity=64, max_pos=t_fresh, device=DEV)
    x, w = torch.zeros((batch, t_fresh, hidden), device=DEV).bfloat16(), torch.zeros(((n_q_heads + 2 * n_kv_heads) * 128, hidden), device=DEV).bfloat16()
    names = _kernels_of(lambda: pc.percache_qkv_rope(0, x, w))
    assert any("qkv_rope_kernelILi128E" in n for n in names), names
    two_heads = [n for n in names if "qkv_rope_kernelILi128E" in n and "ELb1E" in n]
    assert bool(two_heads) == bool(blocks) and all(f"qkv_rope_kernelILi128ELi{blocks}E" in n for n in two_heads), names
    pc.close()


def _pair_kernel(names, D):
    assert any("attention" in n for n in names), names
    return any(f"reuse_attention_wide_kernelILi{D}ELb1E" in n for n in names)


@pytest.mark.parametrize("t_fresh,Hq,Hkv,D,batch", SHARED_BLOCKS)
def test_prompts_of_the_numbers_test_take_shared_128_row_blocks(t_fresh, Hq, Hkv, D, batch):
    _need_256_cus()
    w = wl.make_prefill("pair", 77, "bf16", 128, Hq, Hkv, D, batch, t_fresh, 3, 128, 8)
    pc = make_ctx(w)
    fill_slots(pc, w, w.slot_ids.reshape(-1))
    q, kf, vf = pc.percache_qkv_rope(0, bf16(w.X), bf16(w.Wqkv), w.slot_ids)
    assert _pair_kernel(_kernels_of(lambda: pc.percache_attention_reuse(0, q, kf, vf, w.slot_ids, n_chunks=[0] * batch)), D)
    pc.close()


@pytest.mark.parametrize("t_fresh,Hq,Hkv,D,batch,chunks,pair", [
    (256, 16, 8, 128, 8, 0, True), (400, 16, 8, 128, 6, 0, False), (192, 24, 8, 128, 6, 0, False),   # one round, more, more with the blocks that stand for nothing
    (1300, 16, 8, 128, 2, 0, True), (1300, 16, 8, 128, 2, 2, False),                                  # partitions otherwise; over more than two thirds cached
    (900, 28, 4, 128, 2, 0, False), (1920, 16, 8, 128, 2, 0, False), (1984, 24, 8, 128, 1, 0, True), (2050, 16, 8, 128, 2, 0, False),  # two rounds: of short prompts, whole ones, less, more
    (4000, 16, 8, 128, 1, 2, True), (4000, 16, 8, 128, 1, 4, False), (4224, 16, 8, 128, 1, 0, True),
    (2500, 14, 2, 128, 1, 0, False), (4224, 14, 2, 128, 1, 0, False), (4224, 14, 2, 64, 1, 0, True),  # two kv heads on eight XCDs
])
def test_which_prompts_take_shared_128_row_blocks(t_fresh, Hq, Hkv, D, batch, chunks, pair):
    """Both sides of the lines of the rule (256 CUs), and the same result up to rounding as with two partitions of the key axis, which never take them."""
    _need_256_cus()
    C = 512
    pc = Percache(n_layers=1, hidden=64, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, n_slots=max(1, batch * chunks), slot_capacity=C, max_pos=t_fresh + C * chunks, device=DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(t_fresh)
    rnd = lambda *s: torch.randn(s, generator=g, device=DEV).bfloat16()  # noqa: E731
    for s in range(batch * chunks):
        pc.percache_kv_put(0, s, rnd(Hkv, C, D), rnd(Hkv, C, D))
    q, kf, vf = rnd(batch, Hq, t_fresh, D), rnd(batch, Hkv, t_fresh, D), rnd(batch, Hkv, t_fresh, D)
    ids = np.arange(batch * chunks, dtype=np.int32).reshape(batch, chunks)
    outs = []
    assert _pair_kernel(_kernels_of(lambda: outs.append(pc.percache_attention_reuse(0, q, kf, vf, ids))), D) == pair
    ref = pc.percache_attention_reuse(0, q, kf, vf, ids, n_splits=2)
    check_close(host(outs[0]), host(ref), f"T={t_fresh} batch {batch} chunks {chunks}")
    pc.close()


@pytest.mark.parametrize("tiles,merged", [(45, True), (57, True), (59, False)])
def test_which_steps_merge_their_partials_in_the_o_proj(tiles, merged):
    """One layer, one row of 4 heads: launch by launch, up to 30 partials merged by the o_proj itself."""
    D, Hkv, H, F = 128, 2, 256, 64
    pc = Percache(n_layers=1, hidden=H, n_q_heads=4, n_kv_heads=Hkv, head_dim=D, n_slots=1, slot_capacity=tiles * 64, max_pos=tiles * 64 + 1, device=DEV)
    z = lambda *s: torch.zeros(s, device=DEV).bfloat16()  # noqa: E731
    pc.percache_kv_put(0, 0, z(Hkv, tiles * 64, D), z(Hkv, tiles * 64, D))
    w = dict(gain1=z(H), wqkv=z(8 * D, H), wo=z(H, 4 * D), gain2=z(H), w_gate=z(F, H), w_up=z(F, H), w_down=z(H, F))
    names = _kernels_of(lambda: pc.percache_stack_decode([w], F, 1e-6, z(1, 1, H), [[0]], [-1]))
    assert any("decode_attention_kernel" in n for n in names) and any("oproj_merge_few_kernel" in n for n in names) == merged, names
    pc.close()
