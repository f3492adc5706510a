"""A row attends to keys 0..pos and nothing behind its position reaches it, whatever the later key and value rows hold
(needs an MI355X)."""
import pytest
import torch

import oracle
from paper_2603_06588_amd import binding, workloads as W
from helpers import F32_OUT_ATOL, bits

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
