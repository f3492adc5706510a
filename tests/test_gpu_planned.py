"""Batches whose work lists come from the planning kernel, which smaller batches do without: every form of the kernels that
read those lists against the oracle (needs an MI355X)."""
import pytest
import torch

from oracle.capture import kv_write
from paper_2603_06588_amd import binding, workloads as W
from helpers import beyond_self_planning, bits, compare_with_oracle, plan_header, planned_reference

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("kind", [0, 1, 2])
@pytest.mark.parametrize("Hq,Hkv,d,kv8", [(32, 8, 128, False), (32, 8, 128, True), (8, 2, 64, False), (8, 2, 64, True), (6, 2, 128, True),
                                          (4, 2, 64, True), (4, 4, 128, False), (16, 2, 64, False), (16, 2, 128, True)])
def test_planned_batches_with_new_rows(Hq, Hkv, d, kv8, kind):
    """Chunks on prior context, rows of one and of several items (256 keys each here), the new tokens' rows written by
    the planning launch; then the same lists once more for other queries."""
    lens, qlens = [333, 90, 700, 65, 40, 1500, 257, 16], [333, 1, 100, 2, 0, 1, 1, 16]
    keep = {0: range(8), 1: (0, 2, 3, 4, 7), 2: (1, 4, 5, 6)}[kind]
    lens, qlens = [lens[i] for i in keep], [qlens[i] for i in keep]
    print(f"[case] planned kind={kind} Hq={Hq} Hkv={Hkv} d={d} kv8={kv8}", flush=True)
    b = W.random_batch(2700 + Hq + d, lens, qlens, Hq, Hkv, d, torch.bfloat16, num_probe_heads=3, max_sel_q=9, max_spans=3, poison=False)
    if kv8:
        b = W.fp8_cache_variant(b, 2701)
    gen = torch.Generator().manual_seed(2702)
    k_new, v_new = (torch.randn((b.total_q, Hkv, d), generator=gen).to(torch.bfloat16) for _ in range(2))
    after = b.to("cpu")
    after.k_cache, after.v_cache = kv_write(k_new, v_new, b.block_table, b.seq_lens, b.cu_q_lens, b.k_cache, b.v_cache,
                                            *((b.k_scale, b.v_scale) if kv8 else ()))
    bd = beyond_self_planning(b)
    call = binding.call_from_batch(bd, batch_kind=kind, k_new=k_new.to(DEV), v_new=v_new.to(DEV))
    call.workspace.fill_(0xFF)
    call.out.fill_(float("nan"))
    call.mass.fill_(float("nan"))
    call.launch()
    torch.cuda.synchronize()
    lists = plan_header(call)
    assert lists[2] == 256 and lists[3] == 0 and lists[1] == sum(-(-L // 256) for L, n in zip(lens, qlens) if n == 1)
    view = (lambda t: t.cpu()) if kv8 else bits
    assert torch.equal(view(bd.k_cache), view(after.k_cache)) and torch.equal(view(bd.v_cache), view(after.v_cache))
    assert (call.mass[b.num_seqs:] == 0).all()
    call.mass = call.mass[:b.num_seqs]
    print("      ", compare_with_oracle(after, call.out, call.mass, label="planned"), flush=True)

    other = after.to("cpu")
    other.q = torch.roll(b.q, 1, dims=0).contiguous()
    again = binding.call_from_batch(beyond_self_planning(other), batch_kind=kind, plan_mode=binding.PLAN_REUSE, workspace=call.workspace)
    again.out.fill_(float("nan"))
    again.mass.fill_(0.0)
    again.launch()
    torch.cuda.synchronize()
    fresh = planned_reference(other, batch_kind=kind)
    assert plan_header(again) == lists
    assert torch.equal(bits(again.out), bits(fresh.out)) and torch.equal(bits(again.mass[:b.num_seqs]), bits(fresh.mass))


@pytest.mark.parametrize("kv8", [False, True])
def test_more_single_rows_than_plan_themselves_with_long_contexts_among_them(kv8):
    """Enough rows for the longest items, some of them of two items."""
    lens = [1 + (i * 37) % 60 for i in range(520)]
    lens[3], lens[300], lens[519] = 8193, 9000, 8192
    b = W.random_batch(2710, lens, [1] * 520, 16, 8, 64, torch.bfloat16, num_probe_heads=2, max_sel_q=1, max_spans=2)
    if kv8:
        b = W.fp8_cache_variant(b, 2711)
    call = binding.call_from_batch(b.to(DEV), batch_kind=binding.BATCH_DECODE_ONLY)
    call.out.fill_(float("nan"))
    call.mass.fill_(float("nan"))
    call.launch()
    torch.cuda.synchronize()
    assert plan_header(call) == [0, 522, 8192, 0]
    print("      ", compare_with_oracle(b, call.out, call.mass, label="long items"), flush=True)


@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("planned", [False, True])
def test_batches_on_both_sides_of_the_planner(planned, kv8):
    """The largest batch that streams in equal ranges and the smallest that is planned, with new rows, over every head
    size and group size of the two kernels' key layouts and every number of workgroups per range that the line depends on."""
    for Hq, Hkv, d, most, most_kv8 in ((8, 2, 128, 384, 256), (16, 2, 128, 320, 213), (8, 2, 64, 256, 256), (2, 2, 128, 384, 256),
                                       (4, 1, 128, 512, 341), (8, 1, 64, 284, 284), (6, 2, 128, 192, 192), (8, 4, 128, 288, 192),
                                       (10, 5, 128, 192, 192), (32, 4, 128, 192, 192)):
        n = (most_kv8 if kv8 else most) + planned
        lens = [1 + (i * 29) % 180 for i in range(n)]
        print(f"[case] n={n} Hq={Hq} d={d} kv8={kv8}", flush=True)
        b = W.random_batch(2720 + n, lens, [1] * n, Hq, Hkv, d, torch.bfloat16, num_probe_heads=2, max_sel_q=1, max_spans=2)
        if kv8:
            b = W.fp8_cache_variant(b, 2721)
        gen = torch.Generator().manual_seed(2722)
        k_new, v_new = (torch.randn((n, Hkv, d), generator=gen).to(torch.bfloat16) for _ in range(2))
        after = b.to("cpu")
        after.k_cache, after.v_cache = kv_write(k_new, v_new, b.block_table, b.seq_lens, b.cu_q_lens, b.k_cache, b.v_cache,
                                                *((b.k_scale, b.v_scale) if kv8 else ()))
        call = binding.call_from_batch(b.to(DEV), batch_kind=binding.BATCH_DECODE_ONLY, k_new=k_new.to(DEV), v_new=v_new.to(DEV))
        call.workspace.fill_(0xFF)
        call.out.fill_(float("nan"))
        call.mass.fill_(float("nan"))
        call.launch()
        torch.cuda.synchronize()
        assert plan_header(call) == [0, n if planned else 0, 256 if planned else 0, 0]
        print("      ", compare_with_oracle(after, call.out, call.mass, label="n=%d" % n), flush=True)


@pytest.mark.parametrize("kv8", [False, True])
def test_one_long_context_among_many_short_ones(kv8):
    """Items are cut to a workgroup's share where the largest that fill the chip would be much longer."""
    lens = [1 + (i * 37) % 90 for i in range(300)]
    lens[7] = 16000
    b = W.random_batch(2730, lens, [1] * 300, 16, 8, 64, torch.bfloat16, num_probe_heads=2, max_sel_q=1, max_spans=2)
    if kv8:
        b = W.fp8_cache_variant(b, 2731)
    call = binding.call_from_batch(b.to(DEV), batch_kind=binding.BATCH_DECODE_ONLY)
    call.workspace.fill_(0xFF)
    call.out.fill_(float("nan"))
    call.mass.fill_(float("nan"))
    call.launch()
    torch.cuda.synchronize()
    assert plan_header(call) == [0, 299 + 16000 // 1024 + 1, 1024, 0]      # 331 pieces of 512 keys * 8 / 768 = 1765 keys
    print("      ", compare_with_oracle(b, call.out, call.mass, label="one long"), flush=True)


@pytest.mark.parametrize("Hq,Hkv,d,kv8", [(8, 2, 128, False), (16, 2, 64, True), (3, 1, 128, False)])
def test_planned_sequences_of_few_and_many_records(Hq, Hkv, d, kv8):
    """The merge gives a head one wave, which takes four records at a time, or sixteen where a sequence has more than four:
    record counts on both sides of those steps, the last record of one key, of one block and whole."""
    counts = [1, 2, 3, 4, 5, 8, 15, 16, 17, 20, 31, 32, 33, 48, 49]
    lens = [256 * (c - 1) + (1, 16, 256)[k % 3] for k, c in enumerate(counts)] + [1 + i % 9 for i in range(505)]
    b = W.random_batch(2740 + Hq, lens, [1] * len(lens), Hq, Hkv, d, torch.bfloat16, num_probe_heads=2, max_sel_q=1, max_spans=2)
    if kv8:
        b = W.fp8_cache_variant(b, 2741)
    call = binding.call_from_batch(b.to(DEV), batch_kind=binding.BATCH_DECODE_ONLY)
    call.workspace.fill_(0xFF)
    call.out.fill_(float("nan"))
    call.mass.fill_(float("nan"))
    call.launch()
    torch.cuda.synchronize()
    assert plan_header(call) == [0, sum(counts) + 505, 256, 0]
    print("      ", compare_with_oracle(b, call.out, call.mass, label="records"), flush=True)
