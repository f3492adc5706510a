"""Query chunks take a row's maximum over its first 64 keys as softmax reference.  It is raised where the sums under it grow large,
and rows whose sums leave the range of fp32 before that are done over (needs an MI355X)."""
import pytest
import torch

import oracle
from paper_2603_06588_amd import binding, workloads as W
from helpers import MASS_ATOL, OUT_RTOL_MAX, bits, plan_header, planned_reference

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
FIRST = 96        # first key with large scores


def _run(b_cpu, batch_kind=binding.BATCH_PREFILL_ONLY):
    b = b_cpu.to(DEV)
    call = binding.call_from_batch(b, batch_kind=batch_kind)
    call.out.fill_(float("nan"))
    call.mass.fill_(float("nan"))
    call.launch()
    torch.cuda.synchronize()
    return call


def _rows_of(b, seq, first):
    """(block, row) of the keys first .. L - 1 of a sequence."""
    keys = torch.arange(first, int(b.seq_lens[seq]))
    return b.block_table[seq, keys // 16].long(), keys % 16


def _batch(seed, lens, n, G, d, kv8):
    b = W.random_batch(seed, lens, n, 2 * G, 2, d, torch.bfloat16, num_probe_heads=2 * G, max_sel_q=max(n), max_spans=3)
    b.query_sel[:, 0], b.query_sel[:, 1] = 0, max(n)
    return W.fp8_cache_variant(b, seed + 1) if kv8 else b


def _heat(b, times, head=1, first=FIRST):
    """The batch with keys from `first` on `times` larger for one kv head of sequence 0."""
    hot = b.to("cpu")
    hot.k_cache = b.k_cache.clone()
    blk, row = _rows_of(b, 0, first)
    if b.k_cache.dtype == torch.uint8:      # (the format's largest is 448)
        k = b.k_cache[blk, head, row].view(torch.float8_e4m3fn).float() * times
        hot.k_cache[blk, head, row] = k.clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
    else:
        hot.k_cache[blk, head, row] = (b.k_cache[blk, head, row].float() * times).to(torch.bfloat16)
    return hot


def _check(b, got, rows=None):
    """Against the oracle; the outputs' bound is relative to the largest output of the row (one key can hold all the mass)."""
    ref, ref_mass = oracle.attn_probe_batch(b, rows=rows)
    out = got.out.cpu().double()
    if rows is not None:
        ref, out = ref[rows], out[rows]
    assert torch.isfinite(out).all()
    bound = OUT_RTOL_MAX * ref.abs().amax(dim=-1, keepdim=True).clamp_min(1e-30)
    assert bool(((out - ref).abs() <= bound).all())
    assert (got.mass.cpu().double() - ref_mass).abs().max() <= MASS_ATOL


@pytest.mark.parametrize("G,d,kv8", [(4, 128, False), (8, 128, False), (1, 128, False), (2, 64, False), (4, 64, False), (4, 128, True), (1, 64, True)])
@pytest.mark.parametrize("times", [8.0, 40.0])
def test_scores_far_above_the_first_tile(G, d, kv8, times):
    """Keys from FIRST on are `times` larger for one kv head: scores of some 20 or some 100 natural units, below and above
    what fp32 sums hold.  Everything else keeps its bits."""
    lens, n = [300, 161], [300, 70]
    b = _batch(4100 + d + G, lens, n, G, d, kv8)
    clean = _run(b)
    hot = _heat(b, times)
    clean_head = None if kv8 else FIRST
    if kv8:      # three more powers of two of exponent in the format, one in the scale
        hot.k_scale = b.k_scale.clone()
        hot.k_scale[1] *= 2.0
    got = _run(hot)
    _check(hot, got)
    assert torch.equal(bits(got.out[:, :G]), bits(clean.out[:, :G]))
    if clean_head is not None:
        assert torch.equal(bits(got.out[:FIRST]), bits(clean.out[:FIRST])) and torch.equal(bits(got.out[lens[0]:]), bits(clean.out[lens[0]:]))


@pytest.mark.parametrize("d", [64, 128])
def test_large_values_under_a_low_reference(d):
    """Values of 2^110 with weights that reach 2^20 and more relative to the first tile: finite, as the definition says."""
    b = _batch(4300 + d, [300], [300], 4, d, False)
    blk, row = _rows_of(b, 0, FIRST)
    b.k_cache[blk, 1, row] = (b.k_cache[blk, 1, row].float() * 8).to(torch.bfloat16)
    blk, row = _rows_of(b, 0, 0)
    b.v_cache[blk, 1, row] = (b.v_cache[blk, 1, row].float() * 2.0 ** 110).to(torch.bfloat16)
    _check(b, _run(b))


@pytest.mark.parametrize("G,d", [(4, 128), (1, 128), (8, 64), (2, 64)])
@pytest.mark.parametrize("later", [-1.2e-17, -4e-18, -6e-19])
def test_first_tile_of_minus_infinity(G, d, later):
    """Rows whose scores over the first tile all leave the range of fp32 downwards, so that no maximum is there to refer to:
    the keys behind it, at some -150, -50 and -8 powers of two, get the mass."""
    b = _batch(4400 + d + G, [300, 161], [300, 70], G, d, False)
    b.query_sel[:, 0] = 64
    clean = _run(b)
    b.q[:300, G:], b.k_cache = 0, b.k_cache.clone()
    b.q[:300, G:, 0] = 1e20
    blk, row = _rows_of(b, 0, 0)
    key = torch.arange(300)
    b.k_cache[blk, 1, row, 0] = torch.where(key < 64, -1e20, later * d ** 0.5 / 128 ** 0.5 * (1.0 + (key % 7) / 50.0)).to(torch.bfloat16)
    got = _run(b)
    ref, ref_mass = oracle.attn_probe_batch(b)
    out = got.out.cpu().double()[64:]
    assert (out - ref[64:]).abs().max() <= OUT_RTOL_MAX * ref[64:].abs().max()
    assert (got.mass.cpu().double() - ref_mass).abs().max() <= MASS_ATOL
    assert torch.equal(bits(got.out[:, :G]), bits(clean.out[:, :G])) and torch.equal(bits(got.out[300:]), bits(clean.out[300:]))


@pytest.mark.parametrize("Hq,Hkv,kv8", [(64, 16, False), (64, 8, False), (64, 16, True), (64, 8, True)])
@pytest.mark.parametrize("times", [8.0, 40.0])
def test_late_scores_with_eight_waves(Hq, Hkv, kv8, times):
    """Workgroups of eight waves (groups of 4: two row blocks to a workgroup, groups of 8: one), whose rows are done over elsewhere
    in LDS: against the oracle, and the bits of the planned form with four waves."""
    G, L = Hq // Hkv, 2100
    print(f"[case] late scores, eight waves: heads {Hq}/{Hkv} kv8 {kv8} times {times}", flush=True)
    b = W.random_batch(4500 + G, [L], [L], Hq, Hkv, 128, torch.bfloat16, num_probe_heads=Hq, max_sel_q=40, max_spans=3)
    b.query_sel[:, 0], b.query_sel[:, 1] = FIRST - 20, FIRST + 20
    if kv8:
        b = W.fp8_cache_variant(b, 4501)
    clean = _run(b)
    hot = _heat(b, times)
    if kv8:
        hot.q[:, G:2 * G] = (b.q[:, G:2 * G].float() * times / 2).to(torch.bfloat16)
    got = _run(hot)
    assert plan_header(got)[0] == (L + 32 * 8 // G - 1) // (32 * 8 // G)       # (the number of row blocks says how many waves)
    _check(hot, got, rows=[0, 31, 32, 63, 64, 94, 95, 96, 97, 100, 127, 128, 511, 1023, 1100, 2047, 2048, 2070, 2099]
           + list(range(FIRST - 20, FIRST + 20)))
    others = [h for h in range(Hq) if h // G != 1]
    assert torch.equal(bits(got.out[:, others]), bits(clean.out[:, others]))
    four = planned_reference(hot, batch_kind=binding.BATCH_PREFILL_ONLY)
    assert plan_header(four)[0] == (L + 32 * 4 // min(G, 4) - 1) // (32 * 4 // min(G, 4))
    assert torch.equal(bits(got.out), bits(four.out)) and torch.equal(bits(got.mass), bits(four.mass))


@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("times", [8.0, 40.0])
def test_late_scores_beside_single_rows(kv8, times):
    """A chunk and single rows in one batch: the oracle's results, and for the chunk the bits of the planned form."""
    b = W.random_batch(4600, [300, 700, 64, 1290], [300, 1, 1, 65], 32, 8, 128, torch.bfloat16, num_probe_heads=32, max_sel_q=40, max_spans=3)
    b.query_sel[0, 0], b.query_sel[0, 1] = 200, 240
    if kv8:
        b = W.fp8_cache_variant(b, 4601)
    hot = _heat(b, times)
    if kv8:
        hot.q[:, 4:8] = (b.q[:, 4:8].float() * times / 2).to(torch.bfloat16)
    got = _run(hot, binding.BATCH_MIXED)
    _check(hot, got)
    alone = planned_reference(hot)
    assert torch.equal(bits(got.out[:300]), bits(alone.out[:300])) and torch.equal(bits(got.out[302:]), bits(alone.out[302:]))


@pytest.mark.parametrize("G,d,kv8", [(4, 128, False), (1, 128, False), (4, 64, False), (4, 128, True)])
def test_a_row_that_rises_leaves_its_neighbours_alone(G, d, kv8):
    """Two query rows of a block are 12 and 60 times larger, so that their references rise by some tens and some hundreds of powers of
    two along the context: the other rows of the block keep their bits."""
    b = _batch(4700 + d + G, [600, 161], [600, 70], G, d, kv8)
    clean = _run(b)
    hot = b.to("cpu")
    hot.q = b.q.clone()
    big = [401, 410]
    for row, times in zip(big, (12.0, 60.0)):
        hot.q[row] = (b.q[row].float() * times).to(torch.bfloat16)
    got = _run(hot)
    _check(hot, got)
    rest = [r for r in range(670) if r not in big]
    assert torch.equal(bits(got.out[rest]), bits(clean.out[rest]))


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("times,bound", [(12.0, 1.6), (40.0, 4.7)])
def test_what_late_scores_cost(d, times, bound):
    """Keys of 12 times the first tile's spread take the fast path (1.02-1.2 times the plain prompt's time; done over, it was 5.8 and 4.2 times),
    keys that leave the range of fp32 within a few tiles are done over (3.6 and 3.1)."""
    b = W.random_batch(4800 + d, [2048], [2048], 32, 8, d, torch.bfloat16, num_probe_heads=8, max_sel_q=1, max_spans=2)
    hot = _heat(b, times, head=slice(None))
    calls = [binding.call_from_batch(x.to(DEV), batch_kind=binding.BATCH_PREFILL_ONLY) for x in (b, hot)]
    us = [[], []]
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for _ in range(7):
        for c, t in zip(calls, us):
            c.launch()
            e[0].record()
            for _ in range(20):
                c.launch()
            e[1].record()
            torch.cuda.synchronize()
            t.append(e[0].elapsed_time(e[1]) * 50)
    plain, late = (sorted(t)[3] for t in us)
    print(f"[case] d {d} times {times}: {plain:.1f} and {late:.1f} us", flush=True)
    assert late <= bound * plain
