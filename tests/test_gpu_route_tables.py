"""Routing and plan tables against the oracle over the expert counts where the selection changes shape: lanes per token
(1, 2, 4, 8), elements per lane around the group sizes (2, 4, 8), more than one run of 64 experts in the scan, and enough
route workgroups that the scan's waves take several rows each, or none.  Indices and tables bit for bit, with and without
ties; gates to one rounding of a 64-bit value whose exp() is not the oracle's (1e-6 relative)."""
import numpy as np
import pytest

import oracle
import workloads
from workloads import BF16, Workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def m():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_00662_amd as mod
    mod.binding.lib()
    return mod


# experts, top-k, tokens, tp, slices
SHAPES = [(1, 1, 70, 1, 1), (2, 2, 70, 1, 1), (7, 3, 300, 1, 1), (8, 8, 300, 2, 1), (9, 4, 300, 1, 2), (15, 2, 300, 1, 1),
          (16, 16, 300, 1, 1), (17, 5, 300, 1, 1), (31, 32 - 1, 300, 1, 1), (32, 4, 300, 3, 1), (33, 8, 300, 1, 1),
          (63, 6, 300, 1, 1), (64, 8, 4200, 7, 2), (65, 8, 300, 1, 1), (100, 3, 520, 1, 1), (127, 8, 300, 1, 1),
          (128, 32, 300, 1, 1), (129, 1, 300, 1, 1), (255, 8, 300, 1, 1), (256, 32, 2100, 1, 3), (256, 8, 1, 1, 1),
          (32, 2, 16384, 16, 16)]


@pytest.mark.parametrize("tied", [False, True])
@pytest.mark.parametrize("E,k,T,tp,S", SHAPES)
def test_route_tables(m, E, k, T, tp, S, tied):
    import torch
    w = Workload("rt", T, 8, BF16, E, k, 1, tp, S, 0.6, renorm=E % 2, zipf_s=0.7)
    logits = workloads.make_tied_logits(w) if tied else workloads.make_logits(w)
    x = np.zeros((T, 8), np.uint16)
    ref = oracle.forward(logits, x, k=k, ep=1, tp=tp, S=S, cf=w.capacity_factor, renorm=w.renorm)
    cfg = m.make_cfg(T, 8, BF16, E, k, 1, tp, S, w.capacity_factor, w.renorm)
    for mode in (-1, 0):
        m.monta_set_plan_mode(mode)
        b = m.alloc_buffers(cfg, logits, x)
        m.monta_route(cfg, b.logits, b.topk_idx, b.gates, b.ws)
        torch.cuda.synchronize()
        t = m.read_tables(cfg, b.ws)
        assert np.array_equal(b.topk_idx.cpu().numpy(), ref.topk_idx)
        np.testing.assert_allclose(b.gates.cpu().numpy(), ref.gates, rtol=1e-6)
        pl = ref.plan
        assert t["R"] == pl.R and t["alive"] == int((pl.pos_final.reshape(T, k) >= 0).any(axis=1).sum())
        for name in ("counts", "kept", "offsets", "n", "stage_off", "unit_base", "send_rows", "pos_final", "pos_stage"):
            assert np.array_equal(t[name].reshape(-1), np.asarray(getattr(pl, name)).reshape(-1)), (name, mode)
        assert np.array_equal(t["unit_rows"], np.concatenate([[0], np.cumsum(pl.n.sum(axis=1))]))
        kept = pl.pos_stage.reshape(-1) >= 0
        row_map = np.empty(pl.R, np.int32)
        row_map[pl.pos_stage.reshape(-1)[kept]] = pl.pos_final.reshape(-1)[kept]
        assert np.array_equal(t["row_map"][:pl.R], row_map)


# every count of choices that is found by networks, over lanes per token and keys per lane, rows that are not whole fours and logits that are
# aligned to their elements only; ties among the chosen and at their end in some tokens, masked experts (the type's lowest value) in others
@pytest.mark.parametrize("offset", [0, 1, 3])
@pytest.mark.parametrize("E", [3, 5, 8, 13, 16, 30, 64, 101, 129, 254, 255, 256])
def test_route_choices(m, E, offset):
    import torch
    T = 700
    rng = np.random.default_rng(E + offset)
    logits = rng.standard_normal((T, E)).astype(np.float32)
    logits[100:300] = np.round(logits[100:300] * 4) / 4
    logits[200:400, rng.permutation(E)[:E // 2]] = np.finfo(np.float32).min
    logits[650:] = logits[650:, :1]
    x = np.zeros((T, 8), np.uint16)
    for k in range(1, min(E, 9) + 1):
        w = Workload("choices", T, 8, BF16, E, k, 1, 1, 1, 0.9, renorm=k % 2)
        ref = oracle.forward(logits, x, k=k, ep=1, tp=1, S=1, cf=w.capacity_factor, renorm=w.renorm)
        cfg = m.make_cfg(T, 8, BF16, E, k, 1, 1, 1, w.capacity_factor, w.renorm)
        b = m.alloc_buffers(cfg, logits, x)
        flat = torch.empty(T * E + 4, device="cuda:0")
        view = flat[offset:offset + T * E].view(T, E)
        view.copy_(b.logits)
        m.monta_route(cfg, view, b.topk_idx, b.gates, b.ws)
        torch.cuda.synchronize()
        t = m.read_tables(cfg, b.ws)
        assert np.array_equal(b.topk_idx.cpu().numpy(), ref.topk_idx), k
        np.testing.assert_allclose(b.gates.cpu().numpy(), ref.gates, rtol=1e-6)
        assert np.array_equal(t["pos_final"].reshape(-1), np.asarray(ref.plan.pos_final).reshape(-1)), k
