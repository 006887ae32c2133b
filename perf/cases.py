"""The work whose speed counts: what a program that uses this library has it do, as cases with sizes.

A case is one pass of one kind of call through the public binding:

  step    routing, dispatch and re-gather, then the combine with identity experts: the whole path
          (`static`: through the entry point that keeps its plan tables in the library)
  return  the mirrored second exchange: expert output back to unit-major order, and combined
  route   routing and the plan tables alone (a program that moves rows itself, or plans ahead)
  gate    the gate projection ahead of the path
  expert  the expert layer on an expert-major buffer that is already filled
  layer   routing, dispatch, the expert layer and the combine: one MoE layer from logits to output

`listed()` names the shapes of the repository's own workloads and, where those are all large or all in one data type,
a small, a ragged and a 32-bit one beside them; `draw()` spreads the same kinds over the ranges in between.
"""
import math

import torch

import paper_2411_00662_amd as m

FP32, BF16 = m.FP32, m.BF16


def _case(kind, T, H, dtype, E, k, ep, tp, S, cf, name=None, N=0, zipf=0.0, renorm=1, padded=0, static=0):
    c = {"kind": kind, "tokens": T, "hidden": H, "dtype": "f32" if dtype == FP32 else "bf16", "experts": E, "top_k": k,
         "ep": ep, "tp": tp, "slices": S, "capacity_factor": float(cf), "out_features": N, "zipf": float(zipf),
         "renorm": renorm, "padded": padded, "static": static}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest named workload: launches and host work are all there is
        _case("step", 256, 128, FP32, 4, 2, 2, 2, 2, 0.0, "step_tiny"),
        # one decoding step of a serving loop: 64 sequences, through the entry point made for such loops
        _case("step", 64, 4096, BF16, 8, 2, 8, 1, 1, 0.0, "step_decode", static=1),
        # a sparse layer of 8 experts on an 8K batch
        _case("step", 8192, 4096, BF16, 8, 2, 8, 1, 4, 2.0, "step_mixtral"),
        # fine-grained experts, skewed load, more than half of the pairs dropped: the largest named workload
        _case("step", 65536, 7168, BF16, 64, 8, 8, 4, 8, 1.25, "step_skewed", zipf=1.2),
        # the paper's evaluation shape, on the way back
        _case("return", 8192, 8192, BF16, 2, 1, 2, 8, 4, 0.0, "return_2x70b"),
        # routing at the library's limit of 256 experts
        _case("route", 32768, 64, BF16, 256, 8, 8, 8, 4, 1.25, "route_256", zipf=1.2),
        # gate projections: few experts, many experts
        _case("gate", 8192, 4096, BF16, 8, 2, 8, 1, 1, 0.0, "gate_mixtral"),
        _case("gate", 65536, 7168, BF16, 64, 8, 8, 1, 1, 0.0, "gate_skewed"),
        # the expert layer with long segments (prefill, training) ...
        _case("expert", 8192, 4096, BF16, 8, 2, 8, 1, 4, 2.0, "expert_mixtral", N=4096),
        # ... and with the short, uneven ones of fine-grained experts on an odd batch
        _case("expert", 1532, 7168, BF16, 64, 8, 8, 1, 1, 0.0, "expert_fine", N=2048),
        # one decoding step through a whole layer: the experts' weights are read for a few rows each
        _case("layer", 64, 4096, BF16, 8, 2, 8, 1, 1, 0.0, "layer_decode", N=4096),
        # 32-bit activations, odd sizes, drops and the capacity-padded layout through a whole layer
        _case("layer", 1155, 516, FP32, 10, 3, 5, 3, 5, 0.7, "layer_f32_odd", N=516, renorm=0, padded=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _max_rows(c):
    T, E, k = c["tokens"], c["experts"], c["top_k"]
    C = _capacity(c)
    return E * C if c["padded"] else min(T * k, E * C)


def draw(rng):
    while True:
        kind = rng.choice(["step", "step", "return", "route", "gate", "expert", "expert", "layer"])
        dtype = FP32 if rng.random() < 0.2 else BF16
        E = rng.choice([2, 4, 8, 8, 16, 32, 64, 64, 128, 256, rng.randint(2, 256)])
        k = min(E, rng.choice([1, 2, 2, 4, 6, 8]))
        ep = rng.choice([d for d in (1, 2, 4, 8, 16) if E % d == 0])
        tp, S = rng.choice([1, 1, 2, 4, 8]), rng.choice([1, 2, 4, 4, 8])
        if kind in ("gate", "layer"):
            S = 1 if kind == "gate" else S
            tp = 1
        T = _log(rng, 1, 65536 if kind in ("step", "return", "route", "gate") else 16384)
        T = max(1, T // (tp * S)) * tp * S
        unit = 8 if dtype == BF16 else 4
        H = unit * max(1, _log(rng, 64, 8192) // unit) if rng.random() < 0.4 else rng.choice([512, 1024, 2048, 4096, 5120, 7168, 8192])
        N = 0
        cf, zipf = rng.choice([(0.0, 0.0), (2.0, 0.0), (1.25, 0.0), (1.25, 1.2), (0.7, 0.8)])
        c = _case(kind, T, H, dtype, E, k, ep, tp, S, cf, zipf=zipf, renorm=rng.choice([1, 1, 0]),
                  padded=int(kind in ("step", "layer") and cf > 0 and rng.random() < 0.15),
                  static=int(kind == "step" and rng.random() < 0.2))
        bpe = 4 if dtype == FP32 else 2
        if kind == "route":
            c["hidden"] = 64
        if kind in ("expert", "layer"):
            N = H if kind == "layer" else unit * max(1, _log(rng, 128, 8192) // unit)
            c["out_features"] = N
            flops = 2.0 * T * k * H * N
            # no more than the largest listed case, in 32 bits no more than a test-sized layer takes
            if flops > (5.5e11 if dtype == BF16 else 2e10) or E * H * N * bpe > 2 << 30:
                continue
        # plan tables of the static entry point, and the largest listed case's rows
        if c["static"] and T * (3 * k * 4 + 8) + _max_rows(c) * 4 + T * E // 8 > 8 << 20:
            c["static"] = 0
        if _max_rows(c) * H * bpe > 4 << 30 or T * H * bpe > 1 << 30:
            continue
        return c


# ------------------------------------------------------------------------------------------------ inputs


def _dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _cfg(c):
    return m.make_cfg(c["tokens"], c["hidden"], FP32 if c["dtype"] == "f32" else BF16, c["experts"], c["top_k"], c["ep"],
                      c["tp"], c["slices"], c["capacity_factor"], c["renorm"], c["padded"])


def _inputs(c, seed):
    """Standard-normal logits (with the Zipf bias of a skewed load) and activations, weights scaled by 1/sqrt(H)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    T, H, E, N, dt = c["tokens"], c["hidden"], c["experts"], c["out_features"], _dtype(c)
    d = {}
    d["logits"] = torch.randn((T, E), generator=g, device="cuda")
    if c["zipf"] > 0:
        d["logits"] -= c["zipf"] * torch.log(torch.arange(1, E + 1, device="cuda", dtype=torch.float32))
    if c["kind"] != "route":
        rows = _max_rows(c) if c["kind"] == "return" else T
        d["x"] = torch.randn((rows, H), generator=g, device="cuda", dtype=dt)
    if c["kind"] == "gate":
        d["w"] = torch.randn((E, H), generator=g, device="cuda", dtype=dt).mul_(H ** -0.5)
    if N:
        d["w"] = torch.randn((E, N, H), generator=g, device="cuda", dtype=dt).mul_(H ** -0.5)
    return d


class _State:
    pass


_TABLES = ("pos_final", "pos_stage", "row_map", "offsets", "n", "stage_off", "unit_base", "send_rows", "unit_rows")


def prepare(case, seed):
    c, s = case, _State()
    s.kind, s.cfg, s.static = c["kind"], _cfg(c), c["static"]
    d = _inputs(c, seed)
    T, H, E, k, N, dt = c["tokens"], c["hidden"], c["experts"], c["top_k"], c["out_features"], _dtype(c)
    s.logits, s.x, s.w, s.N = d["logits"], d.get("x"), d.get("w"), N
    if s.kind == "gate":
        return s
    L = m.monta_ws_layout_query(s.cfg)
    rows = L.max_rows

    def zeros(n, w, t=dt):
        return torch.zeros((n, w), dtype=t, device="cuda")

    s.idx, s.gates = zeros(T, k, torch.int32), zeros(T, k, torch.float32)
    s.ws = torch.zeros(L.ws_bytes, dtype=torch.uint8, device="cuda")
    m.monta_ws_init(s.cfg, s.ws)
    if s.kind == "route":
        ints = s.ws.view(torch.int32)
        U = L.units
        size = {"pos_final": T * k, "pos_stage": T * k, "row_map": rows, "offsets": E + 1, "n": U * E, "stage_off": U * E,
                "unit_base": U * E, "send_rows": U * c["ep"], "unit_rows": U + 1}
        s.tables = {t: ints[getattr(L, "off_" + t) // 4:getattr(L, "off_" + t) // 4 + size[t]] for t in _TABLES}
    elif s.kind == "return":
        s.y, s.x = s.x, None
        s.y_stage, s.out = zeros(rows, H), zeros(T, H)
        m.monta_route(s.cfg, s.logits, s.idx, s.gates, s.ws)
    else:
        s.stage, s.final = zeros(rows, H), zeros(rows, H)
        if N:
            s.y = zeros(rows, N)
        if s.kind == "expert":
            m.monta_route_dispatch_regather(s.cfg, s.logits, s.x, s.idx, s.gates, s.stage, s.final, s.ws)
            s.stage = s.x = None
        else:
            s.out = zeros(T, H)
    return s


def run(s):
    if s.kind == "gate":
        m.monta_gate(s.cfg, s.x, s.w, s.logits)
        return s.logits
    if s.kind == "route":
        m.monta_route(s.cfg, s.logits, s.idx, s.gates, s.ws)
        return dict(s.tables, idx=s.idx, gates=s.gates)
    if s.kind == "return":
        m.monta_unregather_combine(s.cfg, s.y, s.y_stage, s.gates, s.out, s.ws)
        return {"y_stage": s.y_stage, "out": s.out}
    if s.kind == "expert":
        m.monta_expert_linear(s.cfg, s.final, s.w, s.N, s.y, s.ws)
        return s.y
    if s.kind == "layer":
        m.monta_route_dispatch_expert(s.cfg, s.logits, s.x, s.idx, s.gates, s.stage, s.final, s.w, s.N, s.y, s.ws, overlap=0)
        m.monta_combine(s.cfg, s.y, s.gates, s.out, s.ws)
        return {"idx": s.idx, "gates": s.gates, "stage": s.stage, "final": s.final, "y": s.y, "out": s.out}
    if s.static:
        m.monta_route_dispatch_combine_static(s.cfg, s.logits, s.x, s.idx, s.gates, s.stage, s.final, s.out)
    else:
        m.monta_route_dispatch_regather(s.cfg, s.logits, s.x, s.idx, s.gates, s.stage, s.final, s.ws)
        m.monta_combine(s.cfg, s.final, s.gates, s.out, s.ws)
    return {"idx": s.idx, "gates": s.gates, "stage": s.stage, "final": s.final, "out": s.out}


# --------------------------------------------------------------------------------- what a pass cannot do without


def _capacity(c):
    T = c["tokens"]
    cf = float(torch.tensor(c["capacity_factor"], dtype=torch.float32))
    return T if cf <= 0 else min(T, math.ceil(cf * T * c["top_k"] / c["experts"]))


def _kept(c):
    """Expected kept pairs and tokens with one: a sample of logits routed on the host and scaled."""
    T, E, k = c["tokens"], c["experts"], c["top_k"]
    n = min(T, 4096)
    lg = torch.randn((n, E), generator=torch.Generator().manual_seed(1))
    if c["zipf"] > 0:
        lg -= c["zipf"] * torch.log(torch.arange(1, E + 1, dtype=torch.float32))
    top = lg.topk(k, dim=1).indices
    counts = torch.bincount(top.flatten(), minlength=E).double() * T / n
    keep = (_capacity(c) / counts.clamp(min=1e-9)).clamp(max=1.0)          # share of an expert's pairs that survive
    alive = 1.0 - (1.0 - keep[top]).prod(dim=1)
    return float((counts * keep).sum()), float(alive.mean()) * T


def work(case):
    c = case
    T, H, E, k, N = c["tokens"], c["hidden"], c["experts"], c["top_k"], c["out_features"]
    bpe = 4 if c["dtype"] == "f32" else 2
    row = H * bpe
    if c["kind"] == "gate":
        return {"bytes": (T + E) * row + T * E * 4, "flops": 2.0 * T * E * H}
    R, alive = _kept(c)
    routing = T * E * 4 + T * k * 8
    if c["kind"] == "route":
        return {"bytes": routing + 2 * T * k * 4 + R * 4, "flops": 0.0}
    if c["kind"] == "return":            # y read, y_stage written, out written
        return {"bytes": (2 * R + T) * row + T * k * 8, "flops": 2.0 * R * H}
    final_rows = E * _capacity(c) if c["padded"] else R
    touched = E * min(1.0, 1.0 - (1.0 - k / E) ** T)                       # experts with at least one token
    if c["kind"] == "expert":
        return {"bytes": R * row + touched * N * row + R * N * bpe, "flops": 2.0 * R * H * N}
    moved = alive * row + R * row + final_rows * row                       # x read, STAGE and FINAL written
    if c["kind"] == "layer":             # and FINAL read by the experts, their output written, read and combined
        return {"bytes": routing + moved + R * row + touched * N * row + 2 * R * N * bpe + T * row,
                "flops": 2.0 * R * H * N + 2.0 * R * H}
    return {"bytes": routing + moved + R * row + T * row, "flops": 2.0 * R * H}


def tolerance(case):
    """Rows are copied and indices counted, so those are the same to the bit; gates are one rounding of a 64-bit value,
    and the combine is one rounding of a 64-bit sum."""
    c = case
    if c["kind"] in ("step", "return", "route"):
        return {"rel": 1e-6, "max": 1e-5 if c["dtype"] == "f32" else 8e-3}
    if c["kind"] == "gate":              # 32-bit sums over the hidden axis, of bf16 or 32-bit products
        return {"rel": 4e-6, "max": 4e-5}
    if c["dtype"] == "f32":              # 32-bit sums over the hidden axis, one after the other: 1.6e-6 off at 8192
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 7e-3, "max": 3e-2}    # one rounding to bf16 per stage


# ------------------------------------------------------------------------------------------ the same in 64 bits


def _plan(c, logits):
    T, E, k = c["tokens"], c["experts"], c["top_k"]
    C = _capacity(c)
    idx = torch.sort(logits, dim=1, descending=True, stable=True).indices[:, :k]
    top = torch.gather(logits.double(), 1, idx)
    w = torch.exp(top - top[:, :1])
    den = w.sum(1, keepdim=True) if c["renorm"] else torch.exp(logits.double() - top[:, :1]).sum(1, keepdim=True)
    e = idx.flatten()
    t = torch.arange(T, device=e.device).repeat_interleave(k)
    order = torch.sort(e, stable=True).indices                              # by expert, then token
    counts = torch.bincount(e, minlength=E)
    start = torch.cumsum(counts, 0) - counts
    rank = torch.empty_like(e)
    rank[order] = torch.arange(T * k, device=e.device) - start[e[order]]
    kept = counts.clamp(max=C)
    off = torch.arange(E, device=e.device) * C if c["padded"] else torch.cumsum(kept, 0) - kept
    live = rank < C
    pos_final = torch.where(live, off[e] + rank, -1)
    U = c["tp"] * c["slices"]
    unit = t // (T // U)
    sent = torch.sort(torch.where(live, unit * E + e, U * E), stable=True).indices[:int(live.sum())]
    pos_stage = torch.full_like(e, -1)
    pos_stage[sent] = torch.arange(sent.numel(), device=e.device)
    return idx, w / den, t, e, live, pos_final, pos_stage, off, kept


def exact(case, seed):
    c = case
    d = _inputs(c, seed)
    T, H, E, k, N = c["tokens"], c["hidden"], c["experts"], c["top_k"], c["out_features"]
    if c["kind"] == "gate":
        return torch.cat([x.double() @ d["w"].double().t() for x in d["x"].split(8192)])
    idx, gates, t, e, live, pos_final, pos_stage, off, kept = _plan(c, d["logits"])
    if c["kind"] == "route":
        return dict({n: None for n in _TABLES}, idx=None, gates=gates)
    rows = _max_rows(c)

    def combined(y):                     # sum over the kept choices of gate * row
        out = torch.zeros((T, H), dtype=torch.float64, device="cuda")
        pf, g = pos_final.view(T, k), gates * live.view(T, k)
        for j in range(k):
            for lo in range(0, T, 8192):
                out[lo:lo + 8192] += g[lo:lo + 8192, j:j + 1] * y[pf[lo:lo + 8192, j].clamp(min=0)].double()
        return out

    if c["kind"] == "return":
        y_stage = torch.zeros_like(d["x"])
        y_stage[pos_stage[live]] = d["x"][pos_final[live]]
        return {"y_stage": y_stage, "out": combined(d["x"])}
    stage, final = (torch.zeros((rows, H), dtype=_dtype(c), device="cuda") for _ in range(2))
    for lo in range(0, T * k, 65536):
        p = live[lo:lo + 65536].nonzero().flatten() + lo
        stage[pos_stage[p]] = d["x"][t[p]]
        final[pos_final[p]] = d["x"][t[p]]
    if c["kind"] == "step":
        return {"idx": None, "gates": gates, "stage": stage, "final": final, "out": combined(final)}
    y = torch.zeros((rows, N), dtype=torch.float64, device="cuda")
    for i in range(E):
        lo, n = int(off[i]), int(kept[i])
        if n:
            y[lo:lo + n] = final[lo:lo + n].double() @ d["w"][i].double().t()
    if c["kind"] == "expert":
        return y
    return {"idx": None, "gates": gates, "stage": stage, "final": final, "y": y, "out": combined(y)}
