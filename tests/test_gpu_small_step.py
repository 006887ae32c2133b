"""Small problems in one launch (every workgroup routes all tokens) against the same calls in several (which an explicit cache
policy or plan mode asks for, and which are held against the oracle elsewhere): choices, gates, every plan table, STAGE, FINAL
and the output, bit for bit.  The shapes sit on the edges: one token, a token more or less than a mask word, the most tokens,
lanes per token from 1 to 16 and up to 8 and up to 16 experts a lane, fewer lanes per row than choices, several rows per wave and
several passes per row, units of one token, padding, drops, and sizes just outside."""
import numpy as np
import pytest

import workloads
from workloads import BF16, FP32, Workload

pytestmark = pytest.mark.gpu

SHAPES = [
    Workload("one", 1, 4096, BF16, 8, 2, 8, 1, 1, 0.0),
    Workload("word", 64, 512, BF16, 8, 2, 8, 1, 1, 0.0),
    Workload("word+1", 65, 4096, FP32, 9, 3, 3, 1, 1, 0.7, zipf_s=0.8, renorm=0),
    Workload("units", 60, 264, BF16, 10, 3, 5, 12, 5, 0.7, zipf_s=0.8),                 # a unit is one token
    Workload("most", 512, 1024, BF16, 15, 4, 5, 4, 8, 0.5, zipf_s=1.0, renorm=0),
    Workload("most16", 512, 8192, BF16, 16, 2, 4, 1, 1, 0.9, zipf_s=0.5),               # two lanes a token
    Workload("many", 100, 2048, BF16, 256, 32, 8, 1, 4, 0.6, zipf_s=0.6),               # too many for one launch
    Workload("lds", 88, 64, FP32, 255, 8, 5, 4, 2, 0.0, renorm=0),
    Workload("four", 200, 136, BF16, 33, 6, 11, 2, 4, 1.25, zipf_s=1.2),                # four lanes a token
    Workload("eight", 128, 520, FP32, 64, 8, 8, 2, 2, 0.5, zipf_s=1.2),
    Workload("row16", 320, 8, BF16, 32, 20, 4, 2, 2, 0.5, zipf_s=0.8),                  # one lane a row, 20 choices
    Workload("row128", 96, 64, BF16, 16, 12, 4, 1, 1, 0.0),                             # eight lanes a row, 12 choices
    Workload("row48", 77, 12, FP32, 7, 7, 7, 7, 11, 0.9, zipf_s=0.8, renorm=0),         # four lanes a row, seven choices
    Workload("row32k", 65, 8196, FP32, 4, 2, 2, 1, 5, 0.8, zipf_s=0.5),                 # three passes, the last one vector
    Workload("padded", 300, 264, BF16, 7, 3, 7, 5, 2, 0.5, zipf_s=0.8, padded=1),
    Workload("padded64", 64, 4096, BF16, 64, 1, 8, 1, 1, 2.0, padded=1),
    Workload("dropall", 256, 128, FP32, 2, 1, 2, 2, 2, 0.01, zipf_s=3.0),               # most tokens lose every choice
    Workload("sixteen", 64, 1024, BF16, 128, 8, 8, 1, 1, 0.0),                          # sixteen lanes a token, four tokens a wave
    Workload("sixteen-drops", 63, 520, FP32, 200, 6, 8, 3, 3, 0.6, zipf_s=1.2, renorm=0),   # 13 experts a lane, the last ones 12
    Workload("sixteen-most", 64, 512, BF16, 256, 32, 8, 2, 2, 0.8, zipf_s=0.6, padded=1),
    Workload("sixteen-few", 3, 264, BF16, 255, 7, 5, 1, 3, 0.8, zipf_s=1.0, renorm=0),
    Workload("outside", 513, 1024, BF16, 8, 2, 8, 1, 1, 0.0),
    Workload("logits", 65, 64, BF16, 126, 4, 6, 5, 1, 0.0),                             # 8190 logits; rows 32760 per choice
    Workload("outside-logits", 65, 64, BF16, 127, 4, 1, 5, 1, 0.9, zipf_s=0.5),         # routing in one launch no longer
    Workload("outside-choices", 130, 64, BF16, 51, 5, 3, 5, 2, 0.9, zipf_s=0.5),        # routing yes, rows no
    Workload("outside-units", 512, 64, BF16, 16, 2, 1, 64, 8, 0.0),                     # too many units
]
TABLES = ("counts", "kept", "offsets", "n", "stage_off", "unit_base", "send_rows", "unit_rows", "pos_final", "pos_stage")


@pytest.fixture(scope="module")
def m():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_00662_amd as mod
    mod.binding.lib()
    return mod


def one_way(m, w, logits, x, several, call):
    import torch
    cfg = m.make_cfg(w.tokens, w.hidden, w.dtype, w.experts, w.top_k, w.ep, w.tp, w.slices, w.capacity_factor, w.renorm, w.padded)
    b = m.alloc_buffers(cfg, logits, x, canary=0xA5)
    b.ws.fill_(0x7F)                     # nothing may depend on what the workspace held
    b.topk_idx.fill_(-7)
    b.gates.fill_(-7.0)
    m.monta_set_cache_policy(42 if several else -1)
    m.monta_set_plan_mode(0 if several else -1)
    try:
        if call == "route":
            m.monta_route(cfg, b.logits, b.topk_idx, b.gates, b.ws)
        elif call == "dispatch":
            m.monta_route_dispatch_regather(cfg, b.logits, b.x, b.topk_idx, b.gates, b.stage, b.final, b.ws)
        else:
            m.monta_route_dispatch_combine_static(cfg, b.logits, b.x, b.topk_idx, b.gates, b.stage, b.final, b.out)
    finally:
        m.monta_set_cache_policy(-1)
        m.monta_set_plan_mode(-1)
    torch.cuda.synchronize()
    got = {"idx": b.topk_idx, "gates": b.gates.view(torch.int32), "stage": b.stage, "final": b.final, "out": b.out}
    got = {n: t.contiguous().view(torch.uint8).cpu().numpy() for n, t in got.items()}
    if call != "static":
        t = m.read_tables(cfg, b.ws)
        got.update({n: np.asarray(t[n]).reshape(-1) for n in TABLES})
        got["row_map"] = np.asarray(t["row_map"])[:t["R"]]
        got["meta"] = np.array([t["R"], t["alive"]])
    return got


@pytest.mark.parametrize("call", ["route", "dispatch", "static"])
@pytest.mark.parametrize("tied", [False, True], ids=["", "tied"])
@pytest.mark.parametrize("w", SHAPES, ids=lambda w: w.name)
def test_one_launch_equals_several(m, w, tied, call):
    logits, x = workloads.make_inputs(w)
    if tied:
        logits = workloads.make_tied_logits(w)
        logits.reshape(-1)[:: max(3, w.experts)] = np.float32("nan")
        logits.reshape(-1)[1:: max(5, w.experts + 2)] = np.float32("-inf")
    one, several = (one_way(m, w, logits, x, s, call) for s in (False, True))
    for name in several:
        np.testing.assert_array_equal(one[name], several[name], err_msg=name)


def test_launch_counts(m):
    """One launch up to 512 tokens, the several beyond; and no launch that reads rows others overwrite."""
    import torch
    for T, names in ((512, {"small_step": 1}), (513, {"route_plan": 1, "plan_place": 1})):
        cfg = m.make_cfg(T, 512, m.BF16, 8, 2, 1, 1, 1, 0.0)
        b = m.alloc_buffers(cfg, np.random.default_rng(0).normal(size=(T, 8)).astype(np.float32))
        m.monta_profile_reset()
        m.monta_profile_enable(True)
        m.monta_route_dispatch_regather(cfg, b.logits, b.x, b.topk_idx, b.gates, b.stage, b.final, b.ws)
        m.monta_profile_enable(False)
        got = {n: m.monta_profile_read(kid)[1] for kid, n in enumerate(m.KERNEL_NAMES)}
        m.monta_profile_reset()
        assert {n: c for n, c in got.items() if c} == names
    torch.cuda.synchronize()


@pytest.mark.parametrize("shared", ["final-x", "gates-logits", "stage-x", "out-x", "out-stage"])
def test_shared_memory_takes_several_launches(m, shared):
    """Where a stored buffer lies in the memory of one that is read, the result is that of the launches one after the other."""
    import torch
    T, H, E, k = 96, 512, 8, 2
    cfg = m.make_cfg(T, H, m.BF16, E, k, 1, 1, 1, 0.0)
    rng = np.random.default_rng(3)
    logits = rng.normal(size=(T, E)).astype(np.float32)

    def step(policy):
        b = m.alloc_buffers(cfg, logits)
        g = torch.Generator(device="cuda").manual_seed(1)
        rows = int(b.stage.shape[0])
        pool = torch.randn((rows + T, H), generator=g, device="cuda").bfloat16()
        lg, gates = b.logits.clone(), b.gates
        x, stage, final, out = pool[:T].clone(), b.stage, b.final, b.out
        if shared == "final-x":
            x, final = pool[8:8 + T], pool[:rows]
        elif shared == "stage-x":
            x, stage = pool[:T], pool[4:4 + rows]
        elif shared == "gates-logits":
            gates = lg.view(-1)[:T * k].view(T, k)
        elif shared == "out-x":
            x, out = pool[:T], pool[2:2 + T]
        elif shared == "out-stage":
            stage, out = pool[:rows], pool[rows - 8:rows - 8 + T]
        m.monta_set_cache_policy(policy)
        try:
            if shared.startswith("out"):
                m.monta_route_dispatch_combine_static(cfg, lg, x, b.topk_idx, gates, stage, final, out)
            else:
                m.monta_route_dispatch_regather(cfg, lg, x, b.topk_idx, gates, stage, final, b.ws)
        finally:
            m.monta_set_cache_policy(-1)
        torch.cuda.synchronize()
        return [t.clone() for t in (b.topk_idx, final, stage) + ((out,) if shared.startswith("out") else ())]

    if shared in ("stage-x", "gates-logits"):
        # several launches race over these themselves beyond one routing workgroup's tokens: it is enough that the call is one of them
        m.monta_profile_reset()
        m.monta_profile_enable(True)
        step(-1)
        m.monta_profile_enable(False)
        assert m.monta_profile_read(m.KERNEL_NAMES.index("small_step"))[1] == 0
        m.monta_profile_reset()
        return
    for a, b in zip(step(-1), step(42)):
        assert torch.equal(a, b)


# what the launches one after the other define: the choices or gates of at most one routing workgroup's tokens anywhere in the logits'
# memory, and with top-k = experts, where a token's gates are stored in place of its own logits, those of any number of tokens.  The
# second shape's units are not divided by its rows per workgroup, so that its dispatch, too, routes by the call that monta_route makes.
@pytest.mark.parametrize("call", ["route", "dispatch"])
@pytest.mark.parametrize("T,E,k,tp,what,at", [(64, 8, 2, 1, "gates", 0), (64, 8, 2, 1, "gates", 37), (64, 8, 2, 1, "idx", 0),
                                             (64, 8, 2, 1, "idx", 384), (62, 4, 4, 2, "gates", 0)])
def test_routing_in_the_logits_memory(m, T, E, k, tp, what, at, call):
    in_the_logits_memory(m, T, E, k, tp, what, at, call, 1)


# the same where several waves route together (two, four and eight lanes a token), and where the logits are read again for the sums
# of their exponentials: choices in front of the first logits, in the middle and behind
@pytest.mark.parametrize("renorm", [0, 1])
@pytest.mark.parametrize("call", ["route", "dispatch"])
@pytest.mark.parametrize("T,E,k,what,at", [(64, 64, 2, "idx", 0), (64, 64, 2, "idx", 1999), (64, 64, 2, "gates", 0), (64, 16, 1, "idx", 0),
                                          (63, 33, 8, "idx", 512), (64, 256, 4, "idx", 0), (50, 256, 6, "idx", 12500), (64, 128, 9, "idx", 3)])
def test_routing_of_several_waves_in_the_logits_memory(m, T, E, k, what, at, call, renorm):
    in_the_logits_memory(m, T, E, k, 1, what, at, call, renorm)


def in_the_logits_memory(m, T, E, k, tp, what, at, call, renorm):
    import torch
    cfg = m.make_cfg(T, 512, m.BF16, E, k, 1, tp, 1, 0.5, renorm)
    rng = np.random.default_rng(T + at)
    logits = rng.normal(size=(T, E)).astype(np.float32)
    x = workloads.f32_to_bf16_bits(rng.normal(size=(T, 512)).astype(np.float32))

    def one(shared):
        b = m.alloc_buffers(cfg, logits, x, canary=0xA5)
        idx, gates = b.topk_idx, b.gates
        if shared:
            mem = b.logits.view(-1)[at:at + T * k]
            if what == "gates":
                gates = mem.view(T, k)
            else:
                idx = mem.view(torch.int32).view(T, k)
        m.monta_profile_reset()
        m.monta_profile_enable(True)
        if call == "route":
            m.monta_route(cfg, b.logits, idx, gates, b.ws)
        else:
            m.monta_route_dispatch_regather(cfg, b.logits, b.x, idx, gates, b.stage, b.final, b.ws)
        m.monta_profile_enable(False)
        assert m.monta_profile_read(m.KERNEL_NAMES.index("small_step"))[1] == (0 if shared else 1)
        m.monta_profile_reset()
        torch.cuda.synchronize()
        t = m.read_tables(cfg, b.ws)
        got = {n: np.asarray(t[n]).reshape(-1) for n in TABLES}
        got.update(idx=idx.cpu().numpy(), gates=gates.view(torch.int32).cpu().numpy(), row_map=np.asarray(t["row_map"])[:t["R"]],
                   stage=b.stage.view(torch.int16).cpu().numpy(), final=b.final.view(torch.int16).cpu().numpy())
        return got

    apart, shared = one(False), one(True)
    for name in apart:
        np.testing.assert_array_equal(shared[name], apart[name], err_msg=name)


# Four tokens whose strongest choice is dropped and whose three kept gates are 2^24 to 2^28 apart: (bf16 value of the row, logits of the
# kept choices; that of the dropped one is 0).  The sum of the three products lies within 2^-53 of the middle between two bf16
# numbers: added one after the other in 64 bits it falls on the middle or on one side, the value times the sum of the gates on another.
FAR_GATES = [(246 / 128, (-0.9775711894035339, -17.92718505859375, -18.063194274902344)),
             (151 / 128, (-1.1030322313308716, -18.03681182861328, -18.30622100830078)),
             (225 / 128, (-1.1926922798156738, -18.10735511779785, -18.39781951904297)),
             (210 / 128, (-0.2344007045030594, -19.29912567138672, -19.637168884277344))]


def test_gates_far_apart(m):
    """The one-launch step adds the products of a token's choices as the combine does, where the order of the roundings shows."""
    import torch
    n, E, k, H = len(FAR_GATES), 8, 4, 512
    logits = np.full((2 * n, E), -60.0, np.float32)
    logits[:n, [0, 4, 5, 6]] = np.float32([0.0, -1.0, -2.0, -3.0])      # these fill expert 0
    logits[n:, 0] = 0.0
    logits[n:, 1:4] = np.float32([far for _, far in FAR_GATES])
    x = np.ones((2 * n, H), np.float32)
    x[n:] = np.float32([v for v, _ in FAR_GATES])[:, None]
    cfg = m.make_cfg(2 * n, H, m.BF16, E, k, 1, 1, 1, 1.0)              # four rows per expert
    got = []
    for static in (True, False):
        b = m.alloc_buffers(cfg, logits, workloads.f32_to_bf16_bits(x), canary=0xA5)
        if static:
            m.monta_route_dispatch_combine_static(cfg, b.logits, b.x, b.topk_idx, b.gates, b.stage, b.final, b.out)
        else:
            m.monta_route_dispatch_regather(cfg, b.logits, b.x, b.topk_idx, b.gates, b.stage, b.final, b.ws)
            m.monta_combine(cfg, b.final, b.gates, b.out, b.ws)
        torch.cuda.synchronize()
        got.append(b.out.view(torch.int16).cpu().numpy())
    g = b.gates.cpu().numpy().astype(np.float64)[n:, 1:]
    v = x[n:, 0].astype(np.float64)
    chain = (g[:, 0] * v + g[:, 1] * v) + g[:, 2] * v                   # products are exact in 64 bits
    assert np.all(chain != ((g[:, 0] + g[:, 1]) + g[:, 2]) * v)         # the case is what it is meant to be
    np.testing.assert_array_equal(got[0], got[1])


def test_replayed_from_a_hip_graph(m):
    import torch
    w = Workload("graph", 256, 1024, BF16, 8, 2, 4, 2, 2, 0.8, zipf_s=0.6)
    cfg = m.make_cfg(w.tokens, w.hidden, w.dtype, w.experts, w.top_k, w.ep, w.tp, w.slices, w.capacity_factor)
    inputs = [workloads.make_inputs(w, seed=s) for s in (1, 2, 3)]
    b = m.alloc_buffers(cfg, *inputs[0], canary=0)
    stream = torch.cuda.Stream()

    def step():
        m.monta_route_dispatch_regather(cfg, b.logits, b.x, b.topk_idx, b.gates, b.stage, b.final, b.ws, stream)
        m.monta_combine(cfg, b.final, b.gates, b.out, b.ws, stream)
        m.monta_route_dispatch_combine_static(cfg, b.logits, b.x, b.topk_idx, b.gates, b.stage, b.final, b.out, stream)

    def load(i):
        b.logits.copy_(torch.from_numpy(inputs[i][0]).cuda())
        b.x.copy_(torch.from_numpy(inputs[i][1].view(np.int16)).cuda().view(torch.bfloat16))
        torch.cuda.synchronize()

    def shot():
        torch.cuda.synchronize()
        return [t.clone() for t in (b.topk_idx, b.gates.view(torch.int32), b.out.view(torch.int16))]

    eager = []
    for i in range(3):
        load(i)
        step()
        eager.append(shot())
    with torch.cuda.stream(stream):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            step()
    for i in (2, 0, 1, 2):
        load(i)
        b.out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        for a, e in zip(shot(), eager[i]):
            assert torch.equal(a, e)
