"""A row attends to keys 0..pos and nothing behind its position reaches it, whatever the later key and value rows hold
(needs an MI355X)."""
import pytest
import torch

import oracle
from paper_2603_06588_amd import binding, workloads as W
from helpers import F32_OUT_ATOL, bits, plan_header

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _run(b_cpu, **kw):
    b = b_cpu.to(DEV)
    call = binding.call_from_batch(b, **kw)
    call.out.fill_(float("nan"))
    call.mass.fill_(float("nan"))
    call.launch()
    torch.cuda.synchronize()
    return call


def _row(b, seq, key):
    return int(b.block_table[seq, key // 16]), key % 16


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("at,what", [(20, float("inf")), (69, float("nan")), (47, float("-inf")), (0, float("inf"))])
def test_fp32_rows_before_a_value_that_is_not_finite(d, at, what):
    """Rows in front of it keep their bits, also those that share its block of 16 rows and those whose last block it
    closes (the last token's value row stands in for the rows behind it); rows that see it are what the oracle says."""
    b = W.random_batch(3100 + d, [70, 300], [70, 30], 4, 2, d, torch.float32, num_probe_heads=2, max_sel_q=2, max_spans=2)
    clean = _run(b)
    bad = b.to("cpu")
    bad.k_cache, bad.v_cache = b.k_cache.clone(), b.v_cache.clone()
    blk, r = _row(b, 0, at)
    bad.v_cache[blk, 1, r, 5] = what                      # kv head 1: query heads 2 and 3
    bad.v_cache[blk, 1, r, d - 1] = what
    got = _run(bad)
    ref, _ = oracle.attn_probe_batch(bad)
    ref, out = ref[:70], got.out[:70].cpu().double()
    assert torch.equal(bits(got.out[:at]), bits(clean.out[:at])) and torch.equal(bits(got.out[70:]), bits(clean.out[70:]))
    assert torch.equal(torch.isfinite(out), torch.isfinite(ref)) and torch.equal(torch.isnan(out), torch.isnan(ref))
    fin = torch.isfinite(ref)
    assert (out[fin] - ref[fin]).abs().max() <= F32_OUT_ATOL and torch.equal(out[~fin & ~torch.isnan(ref)], ref[~fin & ~torch.isnan(ref)])
    assert torch.equal(bits(got.mass), bits(clean.mass))
    # a key row that is not finite is masked for the rows in front of it all the same
    bad.v_cache = b.v_cache
    bad.k_cache[blk, 1, r, 3] = float("nan")
    assert torch.equal(bits(_run(bad).out[:at]), bits(clean.out[:at]))


@pytest.mark.parametrize("G,d,kv8", [(1, 64, False), (2, 64, False), (3, 64, True), (1, 128, False), (2, 128, True), (1, 128, True), (4, 128, False),
                                      (4, 64, False), (4, 128, True), (4, 64, True), (8, 128, False)])
@pytest.mark.parametrize("at", [70, 200])
def test_row_blocks_before_a_tile_whose_value_is_not_finite(G, d, kv8, at):
    """Row blocks that share a workgroup (groups of fewer than four heads) walk its tiles together, but a block of 32
    rows never multiplies a tile of 64 keys behind its last row; nor does one that has a workgroup of its own (4 and 8 heads)."""
    b = W.random_batch(3200 + d, [300, 140], [300, 140], 2 * G, 2, d, torch.bfloat16, num_probe_heads=2, max_sel_q=300, max_spans=2)
    b.query_sel[:, 0], b.query_sel[:, 1] = 0, 300
    if kv8:
        b = W.fp8_cache_variant(b, 3201)
    clean = _run(b, batch_kind=binding.BATCH_PREFILL_ONLY)
    bad = b.to("cpu")
    bad.v_cache = b.v_cache.clone()
    blk, r = _row(b, 0, at)
    bad.v_cache[blk, 1, r, 5] = 0x7F if kv8 else float("inf")
    got = _run(bad, batch_kind=binding.BATCH_PREFILL_ONLY)
    first = at // 64 * 64
    assert torch.equal(bits(got.out[:first]), bits(clean.out[:first])) and torch.equal(bits(got.out[300:]), bits(clean.out[300:]))
    assert torch.equal(bits(got.out[:, :G]), bits(clean.out[:, :G])) and torch.equal(bits(got.mass), bits(clean.mass))
    hit = ~torch.isfinite(got.out[at:300, G:, 5].float())
    assert bool(hit.all()) and torch.isfinite(got.out[:300, :, :5].float()).all()


@pytest.mark.parametrize("Hq,Hkv,kv8", [(64, 16, False), (64, 16, True), (64, 8, False)])
def test_row_blocks_of_eight_waves_before_a_value_that_is_not_finite(Hq, Hkv, kv8):
    """The same where eight waves share a tile's fetch: two row blocks of a group of four heads, one of a group of eight."""
    L, at, G = 2100, 1100, Hq // Hkv
    b = W.random_batch(3300 + Hkv, [L], [L], Hq, Hkv, 128, torch.bfloat16, num_probe_heads=2, max_sel_q=2, max_spans=2)
    b.query_sel[:, 0], b.query_sel[:, 1] = 1000, 1002
    if kv8:
        b = W.fp8_cache_variant(b, 3301)
    clean = _run(b, batch_kind=binding.BATCH_PREFILL_ONLY)
    assert plan_header(clean)[0] == (L + 32 * 8 // G - 1) // (32 * 8 // G)       # (the number of row blocks says how many waves)
    bad = b.to("cpu")
    bad.v_cache = b.v_cache.clone()
    blk, r = _row(b, 0, at)
    bad.v_cache[blk, 1, r, 5] = 0x7F if kv8 else float("inf")
    got = _run(bad, batch_kind=binding.BATCH_PREFILL_ONLY)
    first = at // 64 * 64
    assert torch.equal(bits(got.out[:first]), bits(clean.out[:first])) and torch.equal(bits(got.mass), bits(clean.mass))
    others = [h for h in range(Hq) if h // G != 1]
    assert torch.equal(bits(got.out[:, others]), bits(clean.out[:, others]))
    mine = got.out[:, G:2 * G].float()
    assert bool((~torch.isfinite(mine[at:, :, 5])).all()) and torch.isfinite(mine[:, :, :5]).all()
