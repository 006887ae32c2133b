"""The single pass where most tokens lose all their choices.  From 16 MiB of x on their rows are not read, the others' are, whatever
share of a wave or of a workgroup they are, with one row per workgroup and with several; below that every row is read."""
import math

import pytest

from test_gpu_single_pass import m, test_single_pass_equals_two_passes as check        # noqa: F401  (m: the fixture)
from workloads import BF16, FP32, Workload

pytestmark = pytest.mark.gpu

SHAPES = [
    Workload("eighths", 1000, 64, BF16, 16, 1, 4, 1, 1, 0.1, zipf_s=1.5),           # 8 rows a wave, some of them read
    Workload("halves", 6006, 136, FP32, 8, 1, 4, 2, 3, 0.2, zipf_s=1.2),            # 34 vectors on 64 lanes
    Workload("waves", 4096, 1024, BF16, 32, 2, 4, 2, 2, 0.15, zipf_s=1.2),          # 128 lanes a row
    Workload("several", 16384, 2048, BF16, 4, 1, 4, 1, 4, 0.3, zipf_s=1.0),         # more rows than workgroups at once
    Workload("apart", 8192, 520, BF16, 64, 1, 8, 4, 8, 0.3, zipf_s=1.2),            # plan and rows in kernels of their own
    Workload("scanned", 60000, 1032, BF16, 64, 2, 8, 1, 4, 0.9, zipf_s=1.2),        # the same with the table scanned, above 320 MiB
    Workload("passes", 600, 8196, FP32, 8, 1, 4, 1, 1, 0.2, zipf_s=1.0),            # three passes a row
    Workload("padded", 700, 264, BF16, 7, 1, 7, 5, 2, 0.2, zipf_s=1.0, padded=1),
]


@pytest.mark.parametrize("w", SHAPES, ids=lambda w: w.name)
def test_rows_of_dropped_tokens(m, w):              # noqa: F811
    check(m, w, -1)


# 16 MiB of x and more: every number of lanes that share a row, the tables rebuilt by the rows' own workgroups (up to 2048 counters),
# finished ahead of them, and scanned
UNREAD = [
    Workload("lanes8", 131072, 64, BF16, 4, 1, 4, 1, 2, 0.2, zipf_s=1.5),           # 8 rows a wave
    Workload("lanes16", 65536, 128, BF16, 4, 2, 4, 1, 4, 0.1, zipf_s=1.5),
    Workload("lanes16-apart", 70000, 128, BF16, 16, 1, 4, 2, 5, 0.1, zipf_s=1.5),
    Workload("lanes32", 40000, 256, BF16, 8, 3, 4, 2, 2, 0.1, zipf_s=1.5),
    Workload("lanes32-odd", 40001, 132, FP32, 5, 2, 5, 1, 1, 0.1, zipf_s=1.2),      # 33 vectors on 64 lanes, a last wave of one row
    Workload("lanes32-scanned", 33000, 256, BF16, 200, 2, 8, 5, 6, 0.15, zipf_s=1.2),
    Workload("lanes64", 16500, 512, BF16, 8, 2, 4, 2, 2, 0.15, zipf_s=1.2),
    Workload("lanes128", 16384, 1024, BF16, 32, 2, 4, 2, 2, 0.15, zipf_s=1.2),
    Workload("passes", 1000, 8196, FP32, 8, 1, 4, 1, 1, 0.2, zipf_s=1.0),           # three passes a row
    Workload("padded16", 70000, 128, BF16, 7, 1, 7, 5, 2, 0.2, zipf_s=1.0, padded=1),
    Workload("padded128", 16500, 520, BF16, 7, 2, 7, 5, 2, 0.2, zipf_s=1.0, padded=1),
]


@pytest.mark.parametrize("w", UNREAD, ids=lambda w: w.name)
def test_rows_that_are_not_read(m, w):              # noqa: F811
    capacity = math.ceil(w.capacity_factor * w.tokens * w.top_k / w.experts)
    assert w.tokens * w.hidden * (4 if w.dtype == FP32 else 2) >= 16 << 20
    assert capacity < w.tokens and capacity * w.experts < 2 * w.tokens * w.top_k
    check(m, w, -1)
