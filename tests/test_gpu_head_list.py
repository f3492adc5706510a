"""A head list that is not what it should be - repeated, out-of-range or unordered heads - leaves no entry of `mass`
unwritten, and every path gives it the same values (needs an MI355X)."""
import pytest
import torch

from paper_2603_06588_amd import binding, workloads as W
from helpers import bits, planned_reference

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("heads", [[3, 3, 9], [2, 9, 32], [-1, 0, 31], [7, 3, 12], [31, 30, 1, 1, 0, 40, -5, 2], list(range(31, -1, -1)),
                                   [0, 31]], ids=str)
@pytest.mark.parametrize("lens,qlens,kind", [([70, 300, 33], [1, 1, 1], 2), ([90], [90], 1), ([200, 90], [100, 40], 1),
                                             ([90, 200, 33, 70], [1, 70, 0, 1], 0)])
def test_every_entry_is_written(heads, lens, qlens, kind):
    b = W.random_batch(2600, lens, qlens, 32, 8, 128, torch.bfloat16, num_probe_heads=len(heads), max_sel_q=3, max_spans=2)
    b.probe_heads = torch.tensor(heads, dtype=torch.int32)
    b.query_sel[:, 0], b.query_sel[:, 1] = 0, 2
    ref = planned_reference(b)
    call = binding.call_from_batch(b.to(DEV), batch_kind=kind)
    call.mass.fill_(float("nan"))
    call.launch()
    torch.cuda.synchronize()
    assert torch.isfinite(call.mass).all()
    assert torch.equal(call.mass == 0, ref.mass == 0)
    if kind == 1:
        assert torch.equal(bits(call.mass), bits(ref.mass))
    # single rows are cut differently by the planner: fp32 sums of up to 300 terms in another order
    assert (call.mass - ref.mass).abs().max().item() <= 2e-5
