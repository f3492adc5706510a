"""One sequence of query rows on its own (the single-prompt case) plans itself inside the chunk kernel: no
planning launch.  Results must equal the planned path bit for bit (same work items, same code) and the
oracle within tolerance, and `mass` must be written entry by entry without a planner's zero-fill
(needs an MI355X)."""
import pytest
import torch

from paper_2603_06588_amd import binding, workloads as W
from helpers import bits, compare_with_oracle, plan_header, planned_reference

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _run(b_cpu, kind, sentinel=float("nan"), **kw):
    b = b_cpu.to(DEV)
    out = torch.full_like(b.q, sentinel)
    mass = torch.full((b.num_seqs, b.num_probe_heads, b.max_sel_q, b.max_spans), float("nan"), dtype=torch.float32,
                      device=DEV)
    call = binding.call_from_batch(b, batch_kind=kind, out=out, mass=mass, **kw)
    call.workspace.fill_(0xFF)
    call.launch()
    torch.cuda.synchronize()
    return call


CASES = [
    # seed, L, n, Hq, Hkv, query_sel, label
    (1401, 2048, 2048, 32, 8, (2047, 2048), "a 2048-token prompt, last row"),
    (1402, 777, 777, 8, 2, (770, 777), "ragged length, last 7 rows"),
    (1403, 1500, 300, 8, 2, (-3, 2), "a chunk on prior context; the range begins before the chunk"),
    (1404, 333, 333, 6, 2, (330, 340), "G = 3 (one head per wave); the range reaches past the chunk"),
    (1405, 200, 200, 4, 2, (0, 0), "G = 2; nothing selected"),
    (1406, 190, 190, 4, 4, (100, 104), "G = 1; rows in the middle"),
    (1407, 65, 2, 16, 2, (0, 2), "two rows on prior context, G = 8"),
    (1408, 4100, 4100, 8, 2, (0, 4100), "all rows selected, more than 4096 slots"),
]


@pytest.mark.parametrize("seed,L,n,Hq,Hkv,sel,label", CASES)
def test_single_prompt_equals_planned_path_and_oracle(seed, L, n, Hq, Hkv, sel, label):
    print(f"[case] single prompt: {label}", flush=True)
    nq = max(4, min(sel[1] - sel[0], 4100)) if sel[1] > sel[0] else 4
    b = W.random_batch(seed, [L], [n], Hq, Hkv, 128, torch.bfloat16, num_probe_heads=min(5, Hq), max_sel_q=nq,
                       max_spans=3)
    b.query_sel[0, 0], b.query_sel[0, 1] = sel
    own = _run(b, binding.BATCH_PREFILL_ONLY)
    # the words a planner would have left: [row blocks, 0, 0, status]
    hdr = own.workspace[:16].view(torch.int32).tolist()
    assert hdr[1:4] == [0, 0, 0] and hdr[0] > 0, hdr
    planned = planned_reference(b, batch_kind=binding.BATCH_PREFILL_ONLY)
    assert plan_header(planned)[0] == hdr[0]
    assert torch.equal(bits(own.out), bits(planned.out))
    assert torch.equal(bits(own.mass), bits(planned.mass))          # also: no entry left at the NaN it started with
    print("      ", compare_with_oracle(b, own.out, own.mass, label=label), flush=True)


def test_single_prompt_invalid_contents_are_flagged():
    b = W.random_batch(1410, [300], [300], 8, 2, 128, torch.bfloat16, num_probe_heads=3, max_sel_q=2, max_spans=2)

    def variant(L=None, n=None):
        v = b.to("cpu")
        v.seq_lens = v.seq_lens.clone()
        v.cu_q_lens = v.cu_q_lens.clone()
        if L is not None:
            v.seq_lens[0] = L
        if n is not None:
            v.cu_q_lens[1] = n
        return v

    for v, want in ((variant(L=100), 1), (variant(n=1), 8), (variant(L=-5), 4), (variant(n=0), 0)):
        call = _run(v, binding.BATCH_PREFILL_ONLY, sentinel=7.0)
        assert call.device_status() == want
        assert (call.out == 7.0).all() and (call.mass == 0).all()
    # a length beyond the block table is clamped and computed
    v = variant(L=16 * b.max_blocks_per_seq + 77)
    call = _run(v, binding.BATCH_PREFILL_ONLY, sentinel=7.0)
    assert call.device_status() == 2 and torch.isfinite(call.mass).all()


def test_single_prompt_reusing_call_and_static_scratch():
    b = W.random_batch(1420, [900], [900], 32, 8, 128, torch.bfloat16, num_probe_heads=4, max_sel_q=3, max_spans=2)
    b.query_sel[0, 0], b.query_sel[0, 1] = 899, 900
    fresh = _run(b, binding.BATCH_PREFILL_ONLY)
    bd = b.to(DEV)
    mass = torch.full_like(fresh.mass, 5.0)
    call = binding.call_from_batch(bd, batch_kind=binding.BATCH_PREFILL_ONLY, plan_mode=binding.PLAN_REUSE, mass=mass,
                                   workspace=fresh.workspace)
    call.launch()
    torch.cuda.synchronize()
    assert torch.equal(bits(call.out), bits(fresh.out))
    assert torch.equal(bits(call.mass[:, :, 0]), bits(fresh.mass[:, :, 0]))
    assert (call.mass[:, :, 1:] == 5.0).all()          # slots without a row: never written by a reusing call
    st = binding.call_from_batch(bd, batch_kind=binding.BATCH_PREFILL_ONLY)
    st.out.fill_(float("nan"))
    st.mass.fill_(float("nan"))
    st.launch_static()
    torch.cuda.synchronize()
    assert torch.equal(bits(st.out), bits(fresh.out)) and torch.equal(bits(st.mass), bits(fresh.mass))


def test_single_prompt_with_new_rows_written_in_the_call():
    b_cpu = W.random_batch(1430, [640], [200], 32, 8, 128, torch.bfloat16, num_probe_heads=4, max_sel_q=2, max_spans=2)
    ref = _run(b_cpu, binding.BATCH_PREFILL_ONLY)
    b = b_cpu.to(DEV)
    k_new = torch.empty(200, 8, 128, dtype=torch.bfloat16, device=DEV)
    v_new = torch.empty_like(k_new)
    for t in range(200):
        pos = 640 - 200 + t
        blk, off = int(b.block_table[0, pos // 16]), pos % 16
        k_new[t], v_new[t] = b.k_cache[blk, :, off], b.v_cache[blk, :, off]
        b.k_cache[blk, :, off] = float("nan")
        b.v_cache[blk, :, off] = float("nan")
    call = binding.call_from_batch(b, batch_kind=binding.BATCH_PREFILL_ONLY, k_new=k_new, v_new=v_new)
    call.launch()
    torch.cuda.synchronize()
    assert torch.equal(bits(call.out), bits(ref.out)) and torch.equal(bits(call.mass), bits(ref.mass))


@pytest.mark.parametrize("d,kv8", [(64, False), (64, True), (128, True)])
def test_single_prompt_other_head_size_and_cache_type(d, kv8):
    b = W.random_batch(1440 + d, [777], [300], 8, 2, d, torch.bfloat16, num_probe_heads=3, max_sel_q=4, max_spans=3)
    if kv8:
        b = W.fp8_cache_variant(b, 1441)
    own, planned = _run(b, binding.BATCH_PREFILL_ONLY), planned_reference(b)
    assert torch.equal(bits(own.out), bits(planned.out)) and torch.equal(bits(own.mass), bits(planned.mass))
    print("      ", compare_with_oracle(b, own.out, own.mass, label="single"), flush=True)


@pytest.mark.parametrize("nseq,lo,hi,rows,kind", [(2, 2, 70, None, 1), (63, 2, 60, None, 1), (66, 2, 40, None, 0), (130, 2, 20, None, 0),
                                                  (5, 300, 900, 40, 1), (7, 30, 500, 200, 0)])
def test_several_prompts_find_their_row_blocks(nseq, lo, hi, rows, kind):
    """Batches small enough to plan themselves: every row block is found exactly once, with single rows, empty and
    invalid sequences between the chunks (their rows stay untouched, their `mass` is zero)."""
    lens = [lo + (i * 7919) % (hi - lo + 1) for i in range(nseq)]
    qlens = [min(L, rows) if rows else L for L in lens]
    if kind == 0:
        qlens = [1 if i % 3 == 1 else 0 if i % 7 == 4 else n for i, n in enumerate(qlens)]
    b = W.random_batch(1450 + nseq, lens, qlens, 8, 2, 128, torch.bfloat16, num_probe_heads=3, max_sel_q=3, max_spans=2)
    call = _run(b, kind)
    assert call.device_status() == 0
    from helpers import valid_rows
    written = torch.isfinite(call.out.float()).all(dim=2).all(dim=1).cpu()
    assert bool((written == valid_rows(b)).all())
    print("      ", compare_with_oracle(b, call.out, call.mass, label="several"), flush=True)
    bad = b.to("cpu")
    bad.seq_lens = bad.seq_lens.clone()
    bad.seq_lens[1] = -3
    hit = _run(bad, kind, sentinel=7.0)
    cu = b.cu_q_lens.tolist()
    assert hit.device_status() == 4 and (hit.mass[1] == 0).all() and (hit.out[cu[1]:cu[2]] == 7.0).all()
    assert torch.equal(bits(hit.out[:cu[1]]), bits(call.out[:cu[1]])) and torch.equal(bits(hit.mass[0]), bits(call.mass[0]))


@pytest.mark.parametrize("Hq,Hkv,d,kv8", [(8, 2, 128, False), (16, 2, 64, False), (4, 1, 128, True), (8, 2, 64, True)])
def test_row_blocks_whose_keys_are_shared(Hq, Hkv, d, kv8):
    """Few row blocks, whose four waves share the keys they fetch.  Lengths around the tile borders (one to five tiles, a last
    tile that some rows do not reach), spans across the middle, several sequences of unlike depth in one call; against the
    oracle and the planned call."""
    for lens, qlens in (([129], [129]), ([192], [2]), ([193], [193]), ([256], [33]), ([257], [257]), ([320, 40, 150], [320, 40, 31]),
                        ([1000, 65, 64], [40, 65, 64])):
        print(f"[case] shared keys Hq={Hq} d={d} kv8={kv8} L={lens} n={qlens}", flush=True)
        b = W.random_batch(1460 + lens[0], lens, qlens, Hq, Hkv, d, torch.bfloat16, num_probe_heads=3, max_sel_q=8, max_spans=3)
        for i, (L, n) in enumerate(zip(lens, qlens)):
            b.query_sel[i, 0], b.query_sel[i, 1] = max(0, n - 5), n
            b.key_spans[i] = torch.tensor([(0, L), (L // 2 - 5, L // 2 + 70), (60, 68)], dtype=torch.int32)
        if kv8:
            b = W.fp8_cache_variant(b, 1461)
        own, planned = _run(b, binding.BATCH_PREFILL_ONLY), planned_reference(b, batch_kind=binding.BATCH_PREFILL_ONLY)
        assert torch.equal(bits(own.out), bits(planned.out)) and torch.equal(bits(own.mass), bits(planned.mass))
        print("      ", compare_with_oracle(b, own.out, own.mass, label="shared"), flush=True)


def _widened(b, factor):
    """The same batch behind a block table `factor` times as wide."""
    v = b.to("cpu")
    v.block_table = torch.cat([v.block_table] + [torch.full_like(v.block_table, W.PAD_BLOCK_ID)] * (factor - 1), dim=1).contiguous()
    v.max_blocks_per_seq *= factor
    return v


@pytest.mark.parametrize("lens,qlens,Hq,Hkv,d,kv8", [([1500], [1500], 32, 8, 128, False), ([1024], [1024], 32, 8, 128, False),
                                                    ([700], [300], 32, 8, 64, False), ([1100], [1100], 32, 8, 128, True),
                                                    ([512] * 4, [512] * 4, 16, 4, 128, False)])
def test_results_depend_on_neither_the_table_width_nor_the_rest_of_the_batch(lens, qlens, Hq, Hkv, d, kv8):
    """A row block's result is a matter of its rows and keys: bit for bit the same behind a wider block table and in a
    batch with more sequences than it was alone."""
    b = W.random_batch(1480 + lens[0], lens, qlens, Hq, Hkv, d, torch.bfloat16, num_probe_heads=3, max_sel_q=4, max_spans=2)
    for i, n in enumerate(qlens):
        b.query_sel[i, 0], b.query_sel[i, 1] = n - 4, n
    if kv8:
        b = W.fp8_cache_variant(b, 1481)
    ref = _run(b, binding.BATCH_PREFILL_ONLY)
    print("      ", compare_with_oracle(b, ref.out, ref.mass, label="alone"), flush=True)
    for factor in (2, 8):
        got = _run(_widened(b, factor), binding.BATCH_PREFILL_ONLY)
        assert torch.equal(bits(got.out), bits(ref.out)) and torch.equal(bits(got.mass), bits(ref.mass)), f"table x {factor}"
    times = 4                                  # the same sequences several times over (their caches are only read)
    v = b.to("cpu")
    for name in ("seq_lens", "block_table", "query_sel", "key_spans", "q"):
        t = getattr(v, name)
        setattr(v, name, torch.cat([t] * times).contiguous())
    n = v.cu_q_lens[1:] - v.cu_q_lens[:-1]
    v.cu_q_lens = torch.cat([v.cu_q_lens[:1], torch.cumsum(torch.cat([n] * times), 0).to(torch.int32)])
    v.num_seqs, v.total_q = times * b.num_seqs, times * b.total_q
    got = _run(v, binding.BATCH_PREFILL_ONLY)
    for k in range(times):
        rows, seqs = slice(k * b.total_q, (k + 1) * b.total_q), slice(k * b.num_seqs, (k + 1) * b.num_seqs)
        assert torch.equal(bits(got.out[rows]), bits(ref.out)) and torch.equal(bits(got.mass[seqs]), bits(ref.mass)), f"copy {k}"


@pytest.mark.parametrize("d,kv8", [(128, False), (64, False), (128, True)])
def test_spans_that_end_at_the_integers_limits(d, kv8):
    """An end near the lowest integer makes an empty span, one near the largest reaches to the row's own key."""
    lo, hi = -2**31, 2**31 - 1
    for L, n in ((200, 200), (700, 40), (65, 2)):
        b = W.random_batch(1490 + L, [L], [n], 8, 2, d, torch.bfloat16, num_probe_heads=3, max_sel_q=4, max_spans=4)
        b.query_sel[0, 0], b.query_sel[0, 1] = max(0, n - 4), n
        b.key_spans[0] = torch.tensor([(0, lo), (lo, hi), (lo, lo + 1), (40, hi)], dtype=torch.int32)
        if kv8:
            b = W.fp8_cache_variant(b, 1491)
        got = _run(b, binding.BATCH_PREFILL_ONLY)
        assert (got.mass[:, :, :, 0] == 0).all() and (got.mass[:, :, :, 2] == 0).all()
        print("      ", compare_with_oracle(b, got.out, got.mass, label="limits"), flush=True)
