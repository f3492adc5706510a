"""Mixed batches of few sequences: row blocks and single rows share a launch.  Row blocks give the bits they have by
themselves, single rows (other ranges, other partial sums) the oracle's results, on both sides of the line on the number of
sequences, of the one on self-planning and of the ones on the workgroups per compute unit.  That the launch is one is read from a
captured graph (needs an MI355X)."""
import ctypes

import pytest
import torch

from paper_2603_06588_amd import binding, workloads as W
from helpers import bits, compare_with_oracle, plan_header, planned_reference

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # seed, single rows' contexts, chunks (context, new rows), q heads, kv heads, head size, 8-bit cache, shared
    (6001, [1], [(2, 2)], 4, 1, 128, False, True),                                        # the smallest
    (6002, [17, 1290, 64], [(300, 300), (700, 65)], 32, 8, 128, False, True),             # groups of 4
    (6003, [1029, 333], [(130, 129), (40, 2)], 64, 8, 128, True, True),                   # groups of 8, 8-bit cache
    (6004, [900, 15, 2100], [(257, 33)], 16, 4, 64, False, True),                         # head size 64
    (6005, [500, 1200], [(97, 97), (64, 64)], 24, 3, 64, True, True),                     # ranges that are no multiple of eight
    (6006, [40 + 37 * i for i in range(30)], [(90, 70), (33, 31)], 32, 8, 128, False, True),       # as many sequences as ranges
    (6007, [40 + 37 * i for i in range(31)], [(90, 70), (33, 31)], 32, 8, 128, False, False),      # one more
    (6008, [700, 30, 1, 513], [(2100, 2080), (2100, 2063)], 32, 8, 128, False, True),             # row blocks behind the planner
    (6009, [2500, 77, 640], [(1700, 1650), (900, 900), (1650, 1640)], 32, 8, 128, True, True),     # the same over an 8-bit cache
    (6010, [100, 50], [(300, 300)], 8, 4, 128, False, False),                             # groups of 2
    # two workgroups of single rows to a compute unit ...
    (6011, [1500, 2900, 800, 1700], [(200, 33)], 64, 8, 128, True, True),
    (6012, [1500, 2900, 800, 1700], [(200, 33)], 64, 8, 128, False, True),
    (6013, [1500, 2900, 800, 1700], [(200, 33)], 32, 8, 64, False, True),
    (6014, [2900, 1100, 60, 40], [(60, 60)], 32, 8, 128, True, True),
    # ... unless the row blocks weigh more than contexts of these lengths, which only the kernel sees
    (6015, [2900, 100, 60, 40], [(60, 60)], 32, 8, 128, True, True),
    (6016, [2900, 100, 60, 40], [(60, 60)], 64, 8, 128, False, True),
    # no row blocks at all: two workgroups; one sequence: one
    (6017, [500, 1200, 64], [], 32, 8, 128, False, True),
    (6018, [500, 1200, 64], [], 64, 8, 128, True, True),
    (6019, [1290], [], 32, 8, 128, False, True),
]


def _kernels(call):
    """Launches of the call: the nodes of a graph that captures it."""
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        call.launch(torch.cuda.current_stream())
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    nodes = ctypes.c_size_t(0)
    get = ctypes.CDLL(path).hipGraphGetNodes
    get.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t)]
    assert get(g.raw_cuda_graph(), None, ctypes.byref(nodes)) == 0
    return nodes.value


@pytest.mark.parametrize("seed,ctx,chunks,Hq,Hkv,D,kv8,shared", CASES)
def test_row_blocks_and_single_rows_together(seed, ctx, chunks, Hq, Hkv, D, kv8, shared):
    print(f"[case] one launch: {ctx} and {chunks} heads {Hq}/{Hkv} d {D} kv8 {kv8}", flush=True)
    lens, n = [L for L, _ in chunks[:1]], [x for _, x in chunks[:1]]        # a chunk, the single rows, the other chunks
    lens, n = lens + ctx + [L for L, _ in chunks[1:]], n + [1] * len(ctx) + [x for _, x in chunks[1:]]
    b = W.random_batch(seed, lens, n, Hq, Hkv, D, torch.bfloat16, num_probe_heads=min(5, Hq), max_sel_q=6, max_spans=3)
    b.query_sel[:, 0], b.query_sel[:, 1] = 0, 6
    if kv8:
        b = W.fp8_cache_variant(b, seed + 1)
    call = binding.call_from_batch(b.to(DEV))
    for _ in range(2):
        call.workspace.fill_(0xFF)
        call.out.fill_(float("nan"))
        call.mass.fill_(float("nan"))
        call.launch()
    torch.cuda.synchronize()
    alone = planned_reference(b)
    first, rows = 0, []
    for x in n:
        if x > 1:
            assert torch.equal(bits(call.out[first:first + x]), bits(alone.out[first:first + x]))
        rows += range(first, first + min(x, 6))       # (what is selected)
        first += x
    print("      ", compare_with_oracle(b, call.out, call.mass, rows=rows), flush=True)
    planned = plan_header(call)[2] != 0
    assert _kernels(call) == (2 if shared else 3) + planned       # (planner), row blocks and single rows, merge
