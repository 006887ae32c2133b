"""The kernel classes of the profile: the binding names every id the header declares, in its order."""
import os
import re

import numpy as np
import pytest

import paper_2411_00662_amd as m

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_kernel_id_has_a_name():
    header = open(os.path.join(ROOT, "include", "monta.h")).read()
    ids = {n.lower(): int(v) for n, v in re.findall(r"MONTA_K_([A-Z_]+) = (\d+)", header)}
    count = ids.pop("count")
    assert sorted(ids.values()) == list(range(count)) and len(m.KERNEL_NAMES) == count
    named_otherwise = {"route": "route_plan", "scan": "block_scan"}
    for name, kid in ids.items():
        assert m.KERNEL_NAMES[kid] == named_otherwise.get(name, name)


@pytest.mark.gpu
def test_scan_and_positions_are_counted_apart():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = m.make_cfg(1024, 64, m.BF16, 8, 2, 1, 1, 1, 0.0)
    b = m.alloc_buffers(cfg, np.random.default_rng(0).normal(size=(1024, 8)).astype(np.float32))
    for plan_mode, scans in ((0, 1), (-1, 0)):
        m.monta_set_plan_mode(plan_mode)
        m.monta_profile_reset()
        m.monta_profile_enable(True)
        m.monta_route(cfg, b.logits, b.topk_idx, b.gates, b.ws)
        m.monta_profile_enable(False)
        launches = {name: m.monta_profile_read(kid)[1] for kid, name in enumerate(m.KERNEL_NAMES)}
        assert {n: c for n, c in launches.items() if c} == dict({"route_plan": 1, "positions": 1}, **({"block_scan": 1} if scans else {}))
    m.monta_profile_reset()
