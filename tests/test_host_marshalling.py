"""The native half of the binding refuses what binding.py's own functions refuse, in the same words and order, and passes
addresses and tensors on alike."""
import ctypes

import pytest

import paper_2411_00662_amd as m

B = m.binding
CFG = dict(tokens=8, hidden=16, dtype=m.FP32, experts=4, top_k=2, ep=2, tp=2, slices=2)


def _calls():
    """The buffers of each call in the order in which they are looked at."""
    return {
        "monta_route": ["logits", "topk_idx", "gates", "ws"],
        "monta_route_dispatch_regather": ["logits", "x", "topk_idx", "gates", "stage", "final_", "ws"],
        "monta_route_dispatch_combine_static": ["logits", "x", "topk_idx", "gates", "stage", "final_", "out"],
        "monta_combine": ["y", "gates", "out", "ws"],
        "monta_unregather_combine": ["y", "y_stage", "gates", "out", "ws"],
        "monta_gate": ["x", "w_gate", "logits"],
        "monta_expert_linear": ["x_final", "w_exp", "y", "ws"],
        "monta_route_dispatch_expert": ["logits", "x", "topk_idx", "gates", "stage", "final", "w_exp", "y", "ws"],
    }


def _addresses(names):
    return {n: 4096 * (i + 1) for i, n in enumerate(names)}


def _call(name, cfg, bufs, n=16, **kw):
    if name in ("monta_expert_linear", "monta_route_dispatch_expert"):
        kw["out_features"] = n
    return getattr(m, name)(cfg, **bufs, **kw)


@pytest.mark.parametrize("name", sorted(_calls()))
def test_refusals(name):
    import torch
    names = _calls()[name]
    cfg = m.make_cfg(**CFG)
    for i, bad in enumerate(names):                     # an address, as it is; a host tensor; something else
        bufs = _addresses(names)
        bufs[bad] = torch.zeros(4096)
        with pytest.raises(ValueError, match=f"^{bad}: expected a device tensor$"):
            _call(name, cfg, bufs, stream=0)
        for later in names[i + 1:]:                     # the first in order is the one that is named
            bufs[later] = torch.zeros(1)
        with pytest.raises(ValueError, match=f"^{bad}: expected a device tensor$"):
            _call(name, cfg, bufs, stream=0)
        bufs = dict(_addresses(names), **{bad: "text"})
        with pytest.raises(AttributeError, match="is_cuda"):
            _call(name, cfg, bufs, stream=0)
        bufs[bad] = None
        with pytest.raises(m.MontaError, match=f"^{name}: ") as e:
            _call(name, cfg, bufs, stream=0)
        assert e.value.code == -3
        bufs[bad] = 3                                   # misaligned
        with pytest.raises(m.MontaError, match=f"^{name}: ") as e:
            _call(name, cfg, bufs, stream=0)
        assert e.value.code == -5
    bufs = _addresses(names)
    with pytest.raises(AttributeError, match="cuda_stream"):
        _call(name, cfg, bufs, stream="text")
    with pytest.raises(m.MontaError) as e:              # a configuration that the library refuses, before any buffer is looked at
        _call(name, m.make_cfg(**dict(CFG, top_k=5)), _addresses(names), stream=0)
    assert e.value.code == -1
    for no_cfg in (None, 5, m.monta_ws_layout(), ctypes.pointer(cfg)):
        with pytest.raises(TypeError):
            _call(name, no_cfg, bufs, stream=0)
    with pytest.raises(TypeError):
        getattr(m, name)(cfg)


def test_out_features_beyond_its_type():
    import torch
    bufs = {"x_final": 256, "w_exp": torch.zeros(64), "y": 256, "ws": 256}
    for n in (1 << 40, 1 << 70, -(1 << 70)):
        with pytest.raises(ValueError, match="^w_exp: "):
            _call("monta_expert_linear", m.make_cfg(**CFG), bufs, n, stream=0)


@pytest.mark.gpu
def test_tensors_addresses_and_subclasses():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")

    class Other(torch.Tensor):                          # not one of torch's own classes: looked at by binding.py's function
        pass

    cfg = m.make_cfg(64, 128, m.FP32, 4, 2, 2, 2, 2)
    L = m.monta_ws_layout_query(cfg)
    g = torch.Generator(device="cuda").manual_seed(3)
    logits, x = (torch.randn((64, w), generator=g, device="cuda") for w in (4, 128))
    got = []
    for kind in (lambda t: t, lambda t: t.data_ptr(), lambda t: t.as_subclass(Other), torch.nn.Parameter):
        own = [torch.zeros((64, 2), dtype=torch.int32, device="cuda"), torch.zeros((64, 2), device="cuda"),
               torch.zeros((L.max_rows, 128), device="cuda"), torch.zeros((L.max_rows, 128), device="cuda"),
               torch.zeros((64, 128), device="cuda"), torch.zeros(L.ws_bytes, dtype=torch.uint8, device="cuda")]
        idx, gates, stage, fin, out, ws = [t if kind is torch.nn.Parameter and not t.is_floating_point() else kind(t) for t in own]
        side = torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):                   # without a stream: the current one
            m.monta_route_dispatch_regather(cfg, kind(logits), kind(x), idx, gates, stage, fin, ws)
            m.monta_combine(cfg, fin, gates, out, ws)
        side.synchronize()
        got.append(own[:5])
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert torch.equal(a, b)
    with pytest.raises(ValueError, match="^x: expected a contiguous tensor$"):
        m.monta_route_dispatch_regather(cfg, logits, x.t(), *own[:4], own[5])
    with pytest.raises(ValueError, match="^x: tensor holds 32764 bytes, the shapes in cfg need 32768$"):
        m.monta_route_dispatch_regather(cfg, logits, x.flatten()[1:], *own[:4], own[5])
