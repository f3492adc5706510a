"""Shared comparison helpers for the GPU parity tests (HIP library vs CPU oracle)."""
from __future__ import annotations

from typing import Optional, Sequence

import torch

import oracle

# Tolerances of the parity bar for bf16 inputs: attention output within 2e-2 max-abs of the
# oracle and, because the literal value distribution makes |out| ~ 1e-2, also within 2e-2 of
# max|out_ref|; span masses within 1e-3 absolute.  fp32 inputs are held to 1e-4 / 1e-5.
OUT_ATOL = 2e-2
OUT_RTOL_MAX = 2e-2
MASS_ATOL = 1e-3
F32_OUT_ATOL = 1e-4
F32_MASS_ATOL = 1e-5


def run_hip(b, probe: bool = True):
    from paper_2603_06588_amd import binding
    out, mass = binding.hook_attn_probe_batch(b, probe=probe)
    torch.cuda.synchronize()
    return out, mass


def beyond_self_planning(b_cpu):
    """The batch on the GPU with empty sequences appended until there are too many of them for the kernels to find their
    work themselves: its work lists come from the planning kernel."""
    b = b_cpu.to("cuda:0")
    more = max(513 - b.num_seqs, 0)

    def grow(t):
        return torch.cat([t, t[-1:].expand(more, *t.shape[1:])]).contiguous()

    b.num_seqs += more
    b.seq_lens, b.block_table, b.cu_q_lens = grow(b.seq_lens), grow(b.block_table), grow(b.cu_q_lens)
    b.query_sel, b.key_spans = grow(b.query_sel), grow(b.key_spans)
    return b


def plan_header(call):
    """[row blocks, single-row items, keys per item, status]; a batch without a planner has 0 keys per item."""
    return call.workspace[:16].view(torch.int32).tolist()


def planned_reference(b_cpu, **kw):
    """The call by way of the planning kernel; `mass` is cut back to the batch's own sequences."""
    from paper_2603_06588_amd import binding
    call = binding.call_from_batch(beyond_self_planning(b_cpu), **kw)
    call.workspace.fill_(0xFF)
    call.out.fill_(float("nan"))
    call.mass.fill_(float("nan"))
    call.launch()
    torch.cuda.synchronize()
    assert plan_header(call)[2] >= 256, f"no planner ran: {plan_header(call)}"
    call.mass = call.mass[:b_cpu.num_seqs]
    return call


def valid_rows(b) -> torch.Tensor:
    """Global q rows that belong to a sequence with n_i >= 1 (all rows, normally)."""
    cu = b.cu_q_lens.tolist()
    m = torch.zeros(b.total_q, dtype=torch.bool)
    for i in range(b.num_seqs):
        m[cu[i]:cu[i + 1]] = True
    return m


def compare_with_oracle(b_cpu, out_gpu: torch.Tensor, mass_gpu: torch.Tensor,
                        rows: Optional[Sequence[int]] = None, label: str = ""):
    """Element-by-element comparison; returns the error figures."""
    ref_out, ref_mass = oracle.attn_probe_batch(b_cpu, rows=rows)
    got = out_gpu.detach().cpu().double()
    if rows is None:
        sel = valid_rows(b_cpu)
    else:
        sel = torch.zeros(b_cpu.total_q, dtype=torch.bool)
        sel[torch.tensor(list(rows), dtype=torch.long)] = True
    r, g = ref_out[sel], got[sel]
    assert torch.isfinite(g).all(), f"{label}: non-finite attention output"
    err = (r - g).abs().max().item() if r.numel() else 0.0
    ref_max = r.abs().max().item() if r.numel() else 1.0
    f32 = b_cpu.dtype == torch.float32
    atol = F32_OUT_ATOL if f32 else OUT_ATOL
    assert err <= atol, f"{label}: out max-abs error {err:.3e} > {atol}"
    if not f32:
        assert err <= OUT_RTOL_MAX * ref_max, f"{label}: out error {err:.3e} vs max|ref| {ref_max:.3e}"
    merr = 0.0
    if b_cpu.num_probe_heads:
        gm = mass_gpu.detach().cpu().double()
        assert torch.isfinite(gm).all(), f"{label}: non-finite mass"
        merr = (gm - ref_mass).abs().max().item()
        matol = F32_MASS_ATOL if f32 else MASS_ATOL
        assert merr <= matol, f"{label}: mass error {merr:.3e} > {matol}"
    return {"out_err": err, "out_ref_max": ref_max, "mass_err": merr}


def bits(t: torch.Tensor) -> torch.Tensor:
    t = t.detach().cpu().contiguous()
    return t.view(torch.int16) if t.dtype == torch.bfloat16 else t.view(torch.int32)
