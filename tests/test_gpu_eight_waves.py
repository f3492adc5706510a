"""Deep row blocks in numbers go to workgroups of eight waves, two of which share the fetch of a cache block: the same bits
as with four (the batch with so many empty sequences that it has few rows to each), and the oracle's results (needs an
MI355X)."""
import pytest
import torch

from paper_2603_06588_amd import binding, workloads as W
from helpers import bits, compare_with_oracle, plan_header, planned_reference

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # seed, contexts, new rows, q heads, kv heads, 8-bit cache, row blocks of a workgroup of eight waves
    (5001, [2100], [2100], 64, 16, False, 33),                   # groups of 4: 64 rows, the last block 52 of them; plans itself
    (5002, [1111, 1029], [1111, 1029], 64, 8, False, 68),        # groups of 8: 32 rows, planned
    (5003, [1700, 1291], [1600, 1201], 48, 4, False, 44),        # groups of 12, behind other tokens
    (5004, [2200, 1025], [1290, 1025], 64, 16, True, 38),        # 8-bit cache, groups of 4
    (5005, [2070], [2065], 64, 8, True, 65),                     # 8-bit cache, groups of 8, alone
]


@pytest.mark.parametrize("seed,lens,n,Hq,Hkv,kv8,blocks", CASES)
def test_eight_waves(seed, lens, n, Hq, Hkv, kv8, blocks):
    print(f"[case] eight waves: {lens} new {n} heads {Hq}/{Hkv} kv8 {kv8}", flush=True)
    b = W.random_batch(seed, lens, n, Hq, Hkv, 128, torch.bfloat16, num_probe_heads=5, max_sel_q=40, max_spans=3)
    b.query_sel[:, 0] = torch.tensor([x - 40 for x in n], dtype=torch.int32)
    b.query_sel[:, 1] = torch.tensor(n, dtype=torch.int32)
    if kv8:
        b = W.fp8_cache_variant(b, seed + 1)
    call = binding.call_from_batch(b.to(DEV), batch_kind=binding.BATCH_PREFILL_ONLY)
    call.workspace.fill_(0xFF)
    call.out.fill_(float("nan"))
    call.mass.fill_(float("nan"))
    call.launch()
    torch.cuda.synchronize()
    assert plan_header(call)[0] == blocks
    four = planned_reference(b, batch_kind=binding.BATCH_PREFILL_ONLY)
    assert plan_header(four)[0] == sum((x + 31) // 32 for x in n)
    assert torch.equal(bits(call.out), bits(four.out)) and torch.equal(bits(call.mass), bits(four.mass))
    first = 0
    rows = []
    for x in n:                       # the ends of row blocks and tiles, the selected rows
        rows += [first + r for r in (0, 1, 31, 32, 63, 64, 500, 511, 512) + tuple(range(x - 40, x)) if r < x]
        first += x
    print("      ", compare_with_oracle(b, call.out, call.mass, rows=rows), flush=True)
