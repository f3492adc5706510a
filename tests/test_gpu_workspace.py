"""Workspaces smaller than the size reported: accepted as long as they hold the planner's lists and records, with the
planned kernels doing the work, and refused below (needs an MI355X)."""
import pytest
import torch

from paper_2603_06588_amd import binding, workloads as W
from helpers import compare_with_oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _header(call):
    return call.workspace[:16].view(torch.int32).tolist()      # prefill items, decode items, chunk keys, status


@pytest.mark.parametrize("lens,qlens,kind", [([1240], [1], 2), ([1240], [1], 0), ([90, 700, 33, 5000], [1, 1, 1, 1], 2),
                                             ([90, 700, 33, 400], [1, 70, 0, 1], 0), ([200, 90], [200, 40], 1)])
def test_smallest_workspace_that_is_accepted(lens, qlens, kind):
    b = W.random_batch(2500 + len(lens), lens, qlens, 32, 8, 128, torch.bfloat16, num_probe_heads=3, max_sel_q=2, max_spans=2)
    call = binding.call_from_batch(b.to(DEV), batch_kind=kind)
    reported, run = call.workspace.numel(), binding.load_library().hook_attn_probe
    low, high = 0, reported // 256                             # refused, accepted (in units of the alignment)
    while high - low > 1:
        mid = (low + high) // 2
        call.args.workspace_bytes = 256 * mid
        status = run(call.args)
        assert status in (0, 4)
        low, high = (low, mid) if status == 0 else (mid, high)
    call.args.workspace_bytes = 256 * high
    call.workspace.fill_(0xFF)
    call.out.fill_(float("nan"))
    call.mass.fill_(float("nan"))
    assert run(call.args) == 0
    torch.cuda.synchronize()
    header = _header(call)
    assert header[3] == 0 and 256 * high < reported
    if kind != 1:                                              # (prompts of one call this size need no planner and no records)
        assert header[2] >= 256 and header[1] >= sum(n == 1 for n in qlens)
    assert bool((call.workspace[256 * high:] == 0xFF).all())
    print(compare_with_oracle(b, call.out, call.mass, label="smallest workspace"), flush=True)
