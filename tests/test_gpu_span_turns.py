"""The second kernel of the span pass takes eight, four, two or one spans at a time, by how many workgroups that makes, and
its waves share out the spans that have to be walked: all four, last turns that are not full, spans in order, some of
them long, and spans that overlap (needs an MI355X)."""
import pytest
import torch

import oracle
from paper_2603_06588_amd import binding, workloads as W
from test_gpu_span_mass import _selected_rows

pytestmark = pytest.mark.gpu
# fp32 sums of at most 2700 exponentials, in another order than the oracle's, and logits of up to 2^4 in fp32: 2700 ulps of 2^-24 and
# 2^4 of them in the exponent stay below 2e-4 of a mass that is at most 1
TOL = 2e-4


@pytest.mark.parametrize("layout", ["in order", "long", "overlapping"])
@pytest.mark.parametrize("seqs,heads,spans,rows,d", [
    (4, 8, 33, 17, 64),      # eight at a time, one in the last turn
    (4, 8, 18, 1, 128),      # four, two in the last
    (2, 8, 30, 1, 128),      # two
    (2, 4, 17, 33, 64),      # two, one in the last; two blocks of 32 rows
    (1, 1, 9, 32, 128),      # one
    (1, 2, 1, 40, 64),
    (4, 8, 5, 100, 64),      # four where eight would do, since the table is wide enough for long ones; four blocks of 32 rows
])
def test_spans_taken_in_turns(seqs, heads, spans, rows, d, layout):
    print(f"[case] span turns: {seqs} sequences, {heads} heads, {spans} spans, {rows} rows, d {d}, {layout}", flush=True)
    ctx = [2700 - 411 * i for i in range(seqs)]
    b = W.random_batch(8000 + spans, ctx, [rows + 3] * seqs, 8, 2, d, torch.bfloat16, std=1.0, num_probe_heads=heads,
                       max_sel_q=rows, max_spans=spans)
    b.query_sel[:, 0], b.query_sel[:, 1] = 2, 2 + rows
    gen = torch.Generator().manual_seed(8001)
    for i, L in enumerate(ctx):
        cut = torch.sort(torch.randint(0, L, (2 * spans,), generator=gen)).values.view(spans, 2)
        if layout == "long":          # one of more than 1024 keys, the others around it
            cut = torch.sort(torch.cat([torch.tensor([37, 37 + 1101]), torch.randint(37 + 1101, L, (2 * spans - 2,), generator=gen)])).values.view(spans, 2)
        if layout == "overlapping":
            cut[:, 0] = (cut[:, 0] - 70).clamp(min=0)
        b.key_spans[i] = cut.to(b.key_spans.dtype)
    _, want = oracle.attn_probe_batch(b, rows=_selected_rows(b))
    got = binding.hook_span_mass_batch(b.to("cuda:0"))
    torch.cuda.synchronize()
    err = (got.cpu().double() - want).abs().max().item()
    print(f"       mass error {err:.2e}", flush=True)
    assert err <= TOL
