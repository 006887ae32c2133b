"""The combine and the single-pass return at the lines between their forms: rows of a few vectors, of one wave's 64 and just beyond, of 192 and
256 vectors, rows that leave more or less than three tenths of the lanes' vectors unused; up to 1024 tokens and more; one to nine choices;
some of them dropped.  Rows, sums and what lies past them bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
import workloads
from workloads import BF16, FP32, Workload

pytestmark = pytest.mark.gpu

# tokens, vectors per row, top-k
SHAPES = [(1, 1, 1), (37, 3, 2), (70, 5, 4), (130, 33, 3), (300, 63, 8), (300, 64, 2), (65, 65, 9), (40, 128, 8), (90, 192, 2), (90, 193, 2),
          (25, 256, 1), (25, 257, 1), (25, 257, 2), (30, 358, 5), (30, 359, 8), (20, 512, 2), (20, 516, 3), (1025, 257, 2), (1026, 358, 3),
          (1026, 359, 3), (1030, 516, 2), (1024, 512, 3), (4097, 7, 3), (5000, 64, 3)]


@pytest.mark.parametrize("dtype", [BF16, FP32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("T,vectors,k", SHAPES)
def test_combine_and_return(T, vectors, k, dtype):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_00662_amd as m
    from paper_2411_00662_amd import buffers as bufs
    H = vectors * (8 if dtype == BF16 else 4)
    w = Workload("units", T, H, dtype, 12, k, 3, 1, 1, 0.8, zipf_s=0.5)
    logits, x = workloads.make_inputs(w, seed=T)
    ref = oracle.forward(logits, x, k=k, ep=3, tp=1, S=1, cf=w.capacity_factor)
    R = ref.plan.R
    y = np.random.default_rng(vectors).standard_normal((R, H), dtype=np.float32) * 2
    if dtype == BF16:
        y = workloads.f32_to_bf16_bits(y)
    ys_ref = oracle.unregather(y, ref.plan, 1, 1)
    out_ref = oracle.combine(y, ref.gates, ref.plan.pos_final)
    cfg = m.make_cfg(T, H, dtype, 12, k, 3, 1, 1, w.capacity_factor, w.renorm)
    b = m.alloc_buffers(cfg, logits, x)
    m.monta_route(cfg, b.logits, b.topk_idx, b.gates, b.ws)
    b.gates.copy_(torch.from_numpy(ref.gates).cuda())
    ydev = torch.empty_like(b.final)
    ydev.view(torch.uint8).fill_(0x5A)
    ydev[:R].copy_(bufs.to_device_act(cfg, y))
    ys = torch.empty_like(b.final)
    out = torch.empty((2, T + 1, H), dtype=b.out.dtype, device="cuda:0")
    for t in (ys, out):
        t.view(torch.uint8).fill_(0xA5)
    m.monta_combine(cfg, ydev, b.gates, out[0, :T], b.ws)
    m.monta_unregather_combine(cfg, ydev, ys, b.gates, out[1, :T], b.ws)
    torch.cuda.synchronize()
    ys_h = bufs.to_host_act(cfg, ys)
    np.testing.assert_array_equal(ys_h[:R], ys_ref)
    assert (ys_h[R:].view(np.uint8) == 0xA5).all()
    for i in (0, 1):
        got = bufs.to_host_act(cfg, out[i])
        np.testing.assert_array_equal(got[:T], out_ref)
        assert (got[T].view(np.uint8) == 0xA5).all()
