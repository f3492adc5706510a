"""Self-planned batches of single rows: all contexts laid end to end and cut into equal ranges of cache blocks.
Sizes where that can go wrong - more sequences than lanes, the largest batch that plans itself and the first
that does not (beyond it the planner's items), ranges that hold many short sequences, empty sequences between them - and the new rows that the
same kernel stores into the cache on its way (needs an MI355X)."""
import pytest
import torch

from paper_2603_06588_amd import binding, workloads as W
from helpers import bits, compare_with_oracle, plan_header

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("nseq,hi,Hq,Hkv,d", [(64, 300, 8, 2, 128), (65, 300, 8, 2, 128), (512, 90, 8, 2, 64), (513, 90, 8, 2, 64),
                                              (256, 90, 8, 2, 64), (257, 90, 8, 2, 64), (384, 90, 8, 2, 128), (385, 90, 8, 2, 128),
                                              (512, 90, 4, 1, 128), (513, 90, 4, 1, 128), (192, 90, 32, 8, 128), (193, 90, 32, 8, 128),
                                              (200, 40, 32, 8, 128), (3, 5000, 16, 2, 128),
                                              (14, 500, 32, 8, 128), (4, 131, 64, 8, 128), (95, 200, 32, 8, 128)])
def test_ranges_over_many_sequences(nseq, hi, Hq, Hkv, d):
    lens = [1 + (i * 7919) % hi for i in range(nseq)]
    qlens = [0 if i % 11 == 5 else 1 for i in range(nseq)]
    print(f"[case] stream decode nseq={nseq} hi={hi} Hq={Hq} Hkv={Hkv} d={d}", flush=True)
    b = W.random_batch(2100 + nseq, lens, qlens, Hq, Hkv, d, torch.bfloat16, num_probe_heads=3, max_sel_q=2, max_spans=2)
    b.query_sel[:, 0], b.query_sel[:, 1] = 0, 1
    b.query_sel[1, 0] = -1
    bd = b.to(DEV)
    out = torch.full_like(bd.q, float("nan"))
    mass = torch.full((nseq, 3, 2, 2), float("nan"), dtype=torch.float32, device=DEV)
    call = binding.call_from_batch(bd, batch_kind=binding.BATCH_DECODE_ONLY, out=out, mass=mass)
    call.workspace.fill_(0xFF)
    call.launch()
    torch.cuda.synchronize()
    assert call.device_status() == 0
    items, keys = plan_header(call)[1:3]
    assert (items > 0) == (keys > 0) == (nseq > {(4, 1, 128): 512, (8, 2, 128): 384, (8, 2, 64): 256}.get((Hq, Hkv, d), 192))
    print(compare_with_oracle(b, out, mass, label="stream"), flush=True)


@pytest.mark.parametrize("kv8,d,Hq,Hkv", [(False, 128, 32, 8), (True, 128, 32, 8), (False, 64, 8, 2), (True, 64, 16, 2)])
def test_new_rows_are_stored_by_the_streaming_kernel(kv8, d, Hq, Hkv):
    """Cache bytes and results equal those of a separate write followed by a call without new rows; a sequence whose
    length is clamped, one without rows and one whose block id is outside the cache store nothing."""
    lens, qlens = [500, 33, 257, 1, 16, 17, 700, 48, 90, 64], [1, 1, 1, 1, 1, 1, 1, 0, 1, 1]
    b = W.random_batch(2200 + d, lens, qlens, Hq, Hkv, d, torch.bfloat16, num_probe_heads=4, max_sel_q=1, max_spans=2,
                       poison=False)
    if kv8:
        b = W.fp8_cache_variant(b, 2201)
    b.seq_lens[6] = 16 * b.max_blocks_per_seq + 3                 # beyond the table: clamped, its new row has no slot
    b.block_table[6] = torch.where(b.block_table[6] > b.num_blocks, torch.zeros_like(b.block_table[6]), b.block_table[6])
    b.block_table[8, (90 - 1) // 16] = b.num_blocks + 7           # no such block: nothing may be stored for it
    gen = torch.Generator().manual_seed(5)
    k_new = torch.randn((b.total_q, Hkv, d), generator=gen).to(torch.bfloat16).to(DEV)
    v_new = torch.randn((b.total_q, Hkv, d), generator=gen).to(torch.bfloat16).to(DEV)
    first, second = b.to(DEV), b.to(DEV)
    first.k_cache, first.v_cache = b.k_cache.clone().to(DEV), b.v_cache.clone().to(DEV)
    second.k_cache, second.v_cache = b.k_cache.clone().to(DEV), b.v_cache.clone().to(DEV)
    binding.hook_kv_write(k_new, v_new, first.block_table, first.seq_lens, first.cu_q_lens, first.k_cache, first.v_cache,
                          k_scale=first.k_scale, v_scale=first.v_scale)
    ref = binding.call_from_batch(first, batch_kind=binding.BATCH_DECODE_ONLY)
    ref.launch()
    call = binding.call_from_batch(second, batch_kind=binding.BATCH_DECODE_ONLY, k_new=k_new, v_new=v_new)
    call.launch()
    torch.cuda.synchronize()
    view = (lambda t: t) if kv8 else bits
    assert torch.equal(view(first.k_cache), view(second.k_cache)) and torch.equal(view(first.v_cache), view(second.v_cache))
    rows = [i for i, n in enumerate(qlens) if n and i != 8]       # what sequence 8 attends to at its last position is undefined
    cu = b.cu_q_lens.tolist()
    for i in rows:
        assert torch.equal(bits(call.out[cu[i]]), bits(ref.out[cu[i]])), i
        assert torch.equal(bits(call.mass[i]), bits(ref.mass[i])), i
    assert call.device_status() == ref.device_status() == 2


def test_new_row_in_a_range_of_256_blocks():
    """Each range is one whole context and each wave streams exactly the 64 blocks whose ids fill its register."""
    n, heads, d = 6, 128, 64                 # 128 workgroups per range: six ranges
    b = W.random_batch(2300, [4096] + [16] * (n - 1), [1] * n, heads, heads, d, torch.bfloat16, num_probe_heads=1, max_sel_q=1,
                       max_spans=1, poison=False)
    for i in range(1, n):                    # the other contexts: the first one's blocks and a last block of their own
        b.block_table[i, 255] = b.block_table[i, 0]
        b.block_table[i, :255] = b.block_table[0, :255]
    b.seq_lens[:] = 4096
    gen = torch.Generator().manual_seed(6)
    k_new, v_new = (torch.randn((n, heads, d), generator=gen).to(torch.bfloat16).to(DEV) for _ in range(2))
    first, second = b.to(DEV), b.to(DEV)
    second.k_cache, second.v_cache = first.k_cache.clone(), first.v_cache.clone()
    binding.hook_kv_write(k_new, v_new, first.block_table, first.seq_lens, first.cu_q_lens, first.k_cache, first.v_cache)
    ref = binding.call_from_batch(first, batch_kind=binding.BATCH_DECODE_ONLY)
    ref.launch()
    call = binding.call_from_batch(second, batch_kind=binding.BATCH_DECODE_ONLY, k_new=k_new, v_new=v_new)
    call.launch()
    torch.cuda.synchronize()
    assert torch.equal(bits(first.k_cache), bits(second.k_cache)) and torch.equal(bits(first.v_cache), bits(second.v_cache))
    assert torch.equal(bits(call.out), bits(ref.out)) and torch.equal(bits(call.mass), bits(ref.mass))


@pytest.mark.parametrize("nseq,kv8,d,Hq,Hkv", [(3, False, 128, 32, 8), (40, False, 128, 32, 2), (64, True, 128, 32, 8), (17, False, 64, 8, 2),
                                               (20, True, 64, 16, 4), (65, False, 128, 32, 8), (32, False, 128, 32, 8), (33, False, 128, 32, 8),
                                               (64, False, 128, 32, 8), (64, False, 128, 4, 2)])
@pytest.mark.parametrize("chunk", [False, True])
def test_new_rows_are_read_by_the_other_sequences_of_the_call(nseq, kv8, d, Hq, Hkv, chunk):
    """Rows of one context at consecutive positions: each reads the rows that those in front of it bring, as if all had
    been written before the call.  (One context also meets the block again further in front; with `chunk` one sequence
    contradicts the hint, whose rows are written and read all the same.)  Up to 32 sequences, over an 8-bit cache, at head size
    64 and for groups of 8 heads key rows are fetched by whole lines, otherwise by half lines."""
    print(f"[case] shared context nseq={nseq} kv8={kv8} d={d} Hq={Hq} Hkv={Hkv} chunk={chunk}", flush=True)
    lens, qlens = [300 + i for i in range(nseq)], [1] * nseq
    if chunk:
        lens[1], qlens[1], qlens[2] = 302, 2, 0              # brings the rows at positions 300 and 301
    b = W.random_batch(2400 + nseq, lens, qlens, Hq, Hkv, d, torch.bfloat16, num_probe_heads=4, max_sel_q=1, max_spans=2, poison=False)
    if kv8:
        b = W.fp8_cache_variant(b, 2401)
    last = nseq - 1
    b.block_table[:] = b.block_table[last]
    b.block_table[0, 2] = b.block_table[last, (300 - 1) // 16]
    b.query_sel[:, 0], b.query_sel[:, 1] = 0, 1
    gen = torch.Generator().manual_seed(7)
    k_new, v_new = (3 * torch.randn((b.total_q, Hkv, d), generator=gen).to(torch.bfloat16).to(DEV) for _ in range(2))
    first, second = b.to(DEV), b.to(DEV)
    first.k_cache, first.v_cache = b.k_cache.clone().to(DEV), b.v_cache.clone().to(DEV)
    second.k_cache, second.v_cache = b.k_cache.clone().to(DEV), b.v_cache.clone().to(DEV)
    binding.hook_kv_write(k_new, v_new, first.block_table, first.seq_lens, first.cu_q_lens, first.k_cache, first.v_cache,
                          k_scale=first.k_scale, v_scale=first.v_scale)
    ref = binding.call_from_batch(first, batch_kind=binding.BATCH_DECODE_ONLY)
    call = binding.call_from_batch(second, batch_kind=binding.BATCH_DECODE_ONLY, k_new=k_new, v_new=v_new)
    for c in (ref, call):
        c.out.fill_(7.0)                                      # (rows that are not computed stay untouched)
        c.launch()
    torch.cuda.synchronize()
    view = (lambda t: t) if kv8 else bits
    assert torch.equal(view(first.k_cache), view(second.k_cache)) and torch.equal(view(first.v_cache), view(second.v_cache))
    assert torch.equal(bits(call.out), bits(ref.out)) and torch.equal(bits(call.mass), bits(ref.mass))
    assert call.device_status() == ref.device_status() == (8 if chunk else 0)
