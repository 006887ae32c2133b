"""GPU parity of the single-pass dispatch and return path (the library's default).

Each token row is read once and stored to its rows of STAGE and of FINAL; on the way back each row of y is read once,
stored to its row of y_stage and added.  Bar: every table, STAGE, FINAL (canary intact above R), y_stage and out are
bit for bit what the two passes give (pipeline mode 2, itself held against the oracle elsewhere), and STAGE / FINAL are
the oracle's.  The shapes sit on the edges of the kernels: fewer lanes per row than choices, rows shared by part of a
wave, by one wave, by whole workgroups and by more than one pass; workgroups of several rows; token counts that no
group of rows divides; the padded layout; histogram tables that every workgroup of the mover rebuilds (at most 2048
counters), that only the plan's own workgroups rebuild (at most 4096), and that a kernel scans first.
"""
import numpy as np
import pytest

import oracle
from workloads import BF16, FP32, Workload, make_inputs

pytestmark = pytest.mark.gpu

SHAPES = [
    Workload("row16", 640, 8, BF16, 32, 20, 4, 2, 2, 0.5, zipf_s=0.8),              # 1 lane a row, 20 choices
    Workload("row128", 96, 64, BF16, 16, 12, 4, 1, 1, 0.0),                         # 8 lanes a row, 12 choices
    Workload("row272", 330, 136, BF16, 5, 3, 5, 2, 3, 0.7, zipf_s=0.8),             # 17 vectors on 32 lanes
    Workload("row1k", 4096, 256, FP32, 8, 2, 4, 2, 4, 1.25, zipf_s=0.5),            # a wave a row, four rows a workgroup
    Workload("row1040", 777, 260, FP32, 7, 7, 7, 7, 3, 0.9, zipf_s=0.8, renorm=0),  # 65 vectors: 128 lanes a row
    Workload("row16k", 520, 8192, BF16, 8, 2, 8, 1, 1, 0.6, zipf_s=1.0),            # exactly one pass of a workgroup
    Workload("row32k", 65, 8196, FP32, 4, 2, 2, 1, 5, 0.8, zipf_s=0.5),             # three passes, the last one vector
    Workload("one", 1, 4096, BF16, 8, 2, 8, 1, 1, 0.0),
    Workload("odd", 37, 2048, BF16, 8, 2, 8, 1, 1, 0.0),
    Workload("rounds", 12288, 1024, BF16, 4, 2, 4, 1, 3, 0.9, zipf_s=0.5),          # more than one round: rows per workgroup
    Workload("wide", 2048, 128, BF16, 64, 8, 8, 4, 8, 0.5, zipf_s=1.2),             # 2048 counters: the most a mover rebuilds
    Workload("plan", 4096, 128, BF16, 64, 8, 8, 1, 1, 0.5, zipf_s=1.2),             # 4096: plan and rows in two kernels
    Workload("scan", 2048, 128, BF16, 256, 8, 8, 4, 8, 0.5, zipf_s=1.2),            # 8192: scanned, plan and rows in one
    Workload("scanpad", 2100, 264, FP32, 100, 3, 4, 5, 6, 0.6, zipf_s=0.8, padded=1),
    Workload("scanlong", 8192, 2048, BF16, 64, 8, 8, 4, 4, 0.7, zipf_s=0.5),        # scanned, above 320 MiB: in two
    Workload("padded", 600, 264, BF16, 7, 3, 7, 5, 2, 0.5, zipf_s=0.8, padded=1),
    Workload("padded16", 512, 4096, BF16, 8, 2, 8, 1, 1, 2.0, padded=1),
]


@pytest.fixture(scope="module")
def m():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_00662_amd as mod
    mod.binding.lib()
    return mod


def run(m, w, mode, fused, logits, x, plan_mode=-1):
    import torch
    cfg = m.make_cfg(w.tokens, w.hidden, w.dtype, w.experts, w.top_k, w.ep, w.tp, w.slices, w.capacity_factor, w.renorm, w.padded)
    b = m.alloc_buffers(cfg, logits, x, canary=0xA5)
    y_stage = b.stage.clone()
    m.monta_set_pipeline_mode(mode)
    m.monta_set_plan_mode(plan_mode)
    if fused:
        m.monta_route_dispatch_regather(cfg, b.logits, b.x, b.topk_idx, b.gates, b.stage, b.final, b.ws)
    else:
        m.monta_route(cfg, b.logits, b.topk_idx, b.gates, b.ws)
        m.monta_dispatch_regather(cfg, b.x, b.stage, b.final, b.ws)
    m.monta_unregather_combine(cfg, b.final, y_stage, b.gates, b.out, b.ws)
    torch.cuda.synchronize()
    return cfg, b, y_stage, m.read_tables(cfg, b.ws)


def same_bytes(a, b):
    import torch
    return torch.equal(a.view(torch.uint8), b.view(torch.uint8))


# plan mode 0 scans the table whatever its size
@pytest.mark.parametrize("plan_mode", [-1, 0], ids=["plan-by-size", "plan-scanned"])
@pytest.mark.parametrize("w", SHAPES, ids=lambda w: w.name)
def test_single_pass_equals_two_passes(m, w, plan_mode):
    from paper_2411_00662_amd import buffers as bufs
    logits, x = make_inputs(w)
    cfg, b2, ys2, t2 = run(m, w, 2, False, logits, x)
    ref = oracle.forward(logits, x, k=w.top_k, ep=w.ep, tp=w.tp, S=w.slices, cf=w.capacity_factor, renorm=w.renorm, padded=w.padded)
    for fused in (False, True):
        _, b, ys, t = run(m, w, -1, fused, logits, x, plan_mode)
        R = t["R"]
        for name in ("counts", "kept", "offsets", "n", "stage_off", "unit_base", "send_rows", "unit_rows", "pos_final", "pos_stage"):
            assert np.array_equal(t[name], t2[name]), name
        assert np.array_equal(t["row_map"][:R], t2["row_map"][:R]) and t["alive"] == t2["alive"]
        for name in ("stage", "final", "out", "gates", "topk_idx"):
            assert same_bytes(getattr(b, name), getattr(b2, name)), name
        assert same_bytes(ys, ys2)
        assert np.array_equal(bufs.to_host_act(cfg, b.stage, R), ref.stage[:R])
        assert np.array_equal(bufs.to_host_act(cfg, b.final, t["final_rows"]), ref.final[:t["final_rows"]])


ALIASED = [
    Workload("alias1", 1024, 512, BF16, 8, 2, 4, 2, 1, 0.0),
    Workload("alias4", 1024, 512, BF16, 8, 2, 4, 2, 4, 0.0),                        # plan and pack of all slices in one grid
    Workload("aliasdrop", 1320, 264, BF16, 6, 3, 3, 5, 4, 0.7, zipf_s=0.8),         # plan and pack in two
    Workload("aliaspad", 600, 264, BF16, 7, 3, 7, 5, 2, 0.5, zipf_s=0.8, padded=1),
]


def shared_memory(first, second, where):
    """One allocation for two buffers of so many rows that starts with the first: (rows in all, start of the second)."""
    at = {"start": 0, "second": 1, "inside": max(first - second, 1), "straddling": first - second // 2}[where]
    return max(first, at + second), at


@pytest.mark.parametrize("fused", [False, True], ids=["plan-apart", "plan-fused"])
@pytest.mark.parametrize("where", ["start", "inside", "straddling"])
@pytest.mark.parametrize("w", ALIASED, ids=lambda w: w.name)
def test_final_in_the_memory_of_x(m, w, where, fused):
    """By default FINAL may reuse the memory of x, whatever the number of slices: all of x is packed first."""
    import torch
    logits, x = make_inputs(w)
    cfg, want, _, t2 = run(m, w, 2, False, logits, x)
    b = m.alloc_buffers(cfg, logits, x, canary=0xA5)
    rows = b.layout.max_rows
    total, at = shared_memory(rows, w.tokens, where)
    mem = torch.zeros((total, w.hidden), dtype=b.x.dtype, device="cuda:0")
    shared_x, shared_final = mem[at:at + w.tokens], mem[:rows]
    shared_x.copy_(b.x)
    m.monta_set_pipeline_mode(-1)
    if fused:
        m.monta_route_dispatch_regather(cfg, b.logits, shared_x, b.topk_idx, b.gates, b.stage, shared_final, b.ws)
    else:
        m.monta_route(cfg, b.logits, b.topk_idx, b.gates, b.ws)
        m.monta_dispatch_regather(cfg, shared_x, b.stage, shared_final, b.ws)
    torch.cuda.synchronize()
    n = t2["final_rows"]
    assert same_bytes(shared_final[:n], want.final[:n]) and same_bytes(b.stage, want.stage)


@pytest.mark.parametrize("where", ["second", "inside", "straddling"])
@pytest.mark.parametrize("w", ALIASED, ids=lambda w: w.name)
def test_out_in_the_memory_of_y(m, w, where):
    """By default out may reuse the memory of y, whatever the number of slices: all of y is fetched first."""
    import torch
    logits, x = make_inputs(w)
    cfg, want, want_stage, _ = run(m, w, 2, False, logits, x)
    b = m.alloc_buffers(cfg, logits, x, canary=0xA5)
    rows = b.layout.max_rows
    total, at = shared_memory(rows, w.tokens, where)
    mem = torch.zeros((total, w.hidden), dtype=b.x.dtype, device="cuda:0")
    y, out = mem[:rows], mem[at:at + w.tokens]
    y.copy_(want.final)
    m.monta_set_pipeline_mode(-1)
    m.monta_unregather_combine(cfg, y, b.stage, want.gates, out, want.ws)
    torch.cuda.synchronize()
    assert same_bytes(out, want.out) and same_bytes(b.stage, want_stage)
