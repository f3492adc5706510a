"""Cache writes look the rows' sequences up in a copy of the row offsets as long as that fits its place: both sides of that,
in the launch of its own (255 sequences) and in the planning launch (1023), rows at the borders of sequences among them
(needs an MI355X)."""
import pytest
import torch

from oracle.capture import kv_write
from paper_2603_06588_amd import binding, workloads as W
from helpers import bits

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("seqs,in_call", [(1, False), (255, False), (256, False), (1, True), (1023, True), (1024, True)])
def test_new_rows_of_many_sequences(seqs, in_call):
    print(f"[case] new rows of {seqs} sequences, in the attention call: {in_call}", flush=True)
    n = [(1, 2, 0, 9)[i % 4] for i in range(seqs)]
    lens = [x + 5 * (i % 7) for i, x in enumerate(n)]
    b = W.random_batch(7000 + seqs, lens, n, 4, 2, 64, torch.bfloat16, num_probe_heads=1, max_sel_q=1, poison=False)
    gen = torch.Generator().manual_seed(7001)
    k_new, v_new = (torch.randn((b.total_q, 2, 64), generator=gen).to(torch.bfloat16) for _ in range(2))
    want_k, want_v = kv_write(k_new, v_new, b.block_table, b.seq_lens, b.cu_q_lens, b.k_cache, b.v_cache)
    d = b.to(DEV)
    if in_call:
        binding.call_from_batch(d, k_new=k_new.to(DEV), v_new=v_new.to(DEV)).launch()
    else:
        binding.hook_kv_write(k_new.to(DEV), v_new.to(DEV), d.block_table, d.seq_lens, d.cu_q_lens, d.k_cache, d.v_cache)
    torch.cuda.synchronize()
    assert torch.equal(bits(d.k_cache.cpu()), bits(want_k)) and torch.equal(bits(d.v_cache.cpu()), bits(want_v))
