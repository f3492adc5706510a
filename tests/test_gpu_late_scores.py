"""Query chunks take a row's maximum over its first 64 keys as softmax reference and keep it.  Rows whose later scores lie so
far above it that their sums leave the range of fp32 are done over from their true maximum (needs an MI355X)."""
import pytest
import torch

import oracle
from paper_2603_06588_amd import binding, workloads as W
from helpers import MASS_ATOL, OUT_RTOL_MAX, bits

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
FIRST = 96        # first key with large scores


def _run(b_cpu):
    b = b_cpu.to(DEV)
    call = binding.call_from_batch(b, batch_kind=binding.BATCH_PREFILL_ONLY)
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


def _check(b, got):
    """Against the oracle; the outputs' bound is relative to the largest output of the row (one key can hold all the mass)."""
    ref, ref_mass = oracle.attn_probe_batch(b)
    out = got.out.cpu().double()
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
    hot = b.to("cpu")
    hot.k_cache = b.k_cache.clone()
    blk, row = _rows_of(b, 0, FIRST)
    if kv8:      # three more powers of two of exponent (the format's largest is 448)
        k = b.k_cache[blk, 1, row].view(torch.float8_e4m3fn).float() * times
        hot.k_cache[blk, 1, row] = k.clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
        hot.k_scale = b.k_scale.clone()
        hot.k_scale[1] *= 2.0
        clean_head = None
    else:
        hot.k_cache[blk, 1, row] = (b.k_cache[blk, 1, row].float() * times).to(torch.bfloat16)
        clean_head = FIRST
    got = _run(hot)
    _check(hot, got)
    assert torch.equal(bits(got.out[:, :G]), bits(clean.out[:, :G]))
    if clean_head is not None:
        assert torch.equal(bits(got.out[:FIRST]), bits(clean.out[:FIRST])) and torch.equal(bits(got.out[lens[0]:]), bits(clean.out[lens[0]:]))


@pytest.mark.parametrize("d", [64, 128])
def test_large_values_under_a_low_reference(d):
    """Values of 2^100 with weights that reach 2^20 and more relative to the first tile: finite, as the definition says."""
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
