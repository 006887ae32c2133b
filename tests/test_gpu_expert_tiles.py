"""Expert layer with segment sizes on the edges of its kernels' tiles, fixed by the logits (top-1, one expert per token
run).  Small-integer inputs: every partial sum is an integer below 2^24, so any order of additions gives the oracle's
value and the comparison is exact."""
import numpy as np
import pytest

import oracle
import workloads
from workloads import BF16, FP32, Workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def m():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_00662_amd as mod
    mod.binding.lib()
    return mod


def check(m, sizes, H, N, dtype):
    import torch
    from paper_2411_00662_amd import buffers as bufs
    T, E = sum(sizes), len(sizes)
    w = Workload("tiles", T, H, dtype, E, 1, 1, 1, 1, 0.0)
    rng = np.random.default_rng(T + H + N)
    logits = rng.uniform(-0.25, 0.25, size=(T, E)).astype(np.float32)
    logits[np.arange(T), np.repeat(np.arange(E), sizes)] += 4.0
    to_act = (lambda a: a) if dtype == FP32 else workloads.f32_to_bf16_bits
    x = to_act(rng.integers(-4, 5, size=(T, H)).astype(np.float32))
    we = to_act(rng.integers(-4, 5, size=(E, N, H)).astype(np.float32))
    cfg = m.make_cfg(T, H, dtype, E, 1, 1, 1, 1, 0.0)
    b = m.alloc_buffers(cfg, logits, x)
    m.monta_route_dispatch_regather(cfg, b.logits, b.x, b.topk_idx, b.gates, b.stage, b.final, b.ws)
    y = torch.empty((T + 1, N), dtype=b.final.dtype, device="cuda:0")
    y.view(torch.uint8).fill_(0x5A)
    m.monta_expert_linear(cfg, b.final, bufs.to_device_act(cfg, we.reshape(E * N, H)), N, y[:T], b.ws)
    torch.cuda.synchronize()
    got = bufs.to_host_act(cfg, y)
    ref = oracle.forward(logits, x, k=1, ep=1, tp=1, S=1, cf=0.0)
    assert [int(v) for v in ref.plan.kept] == list(sizes)
    lo, hi = oracle.expert_ranges(ref.plan, 1, 1)
    np.testing.assert_array_equal(got[:T], oracle.expert(ref.final, we, lo, hi))
    assert np.all(got[T].view(np.uint8) == 0x5A)


# many experts on short rows: the register-staged tiles
def test_short_rows_many_experts(m):
    check(m, [120 + (37 * e) % 33 for e in range(64)], 128, 1032, BF16)


def check_on_gpu(m, sizes, H, N, dtype):
    """Large weights: made, and multiplied for the reference, on the GPU (fp32 products and sums of these integers are exact in any
    order; one rounding to bf16)."""
    import torch
    t = torch.float32 if dtype == FP32 else torch.bfloat16
    T, E = sum(sizes), len(sizes)
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randint(-4, 5, (T, H), generator=g, device="cuda").to(t)
    w = torch.randint(-4, 5, (E, N, H), generator=g, device="cuda", dtype=torch.int8).to(t)
    logits = torch.zeros((T, E), device="cuda")
    expert = torch.repeat_interleave(torch.arange(E, device="cuda"), torch.tensor(sizes, device="cuda"))
    logits[torch.arange(T, device="cuda"), expert] = 4.0
    cfg = m.make_cfg(T, H, dtype, E, 1, 1, 1, 1, 0.0)
    b = m.alloc_buffers(cfg, logits.cpu().numpy())
    m.monta_route_dispatch_regather(cfg, b.logits, x, b.topk_idx, b.gates, b.stage, b.final, b.ws)
    y = torch.full((T + 1, N), float("nan"), dtype=t, device="cuda")
    m.monta_expert_linear(cfg, b.final, w, N, y[:T], b.ws)
    assert bool(torch.isnan(y[T]).all())
    for e in range(E):
        rows = expert == e
        if bool(rows.any()):
            assert torch.equal(y[:T][rows], (x[rows].float() @ w[e].float().t()).to(t))


def test_long_rows_full_rounds(m):
    """Close to 1 GB of weights."""
    check_on_gpu(m, [40, 1, 0, 100, 33, 64, 65, 17], 4096, 57 * 256 + 8, BF16)


# 57 to 76 rows in the mean on long rows, large tiles beside ragged ones of up to 64 rows; and fp32 in 783 and 957
# tiles of 16 x 32, where those of 32 x 64 are up to one per CU and more, and in 32 x 64
@pytest.mark.parametrize("H", [4096, 4104])
def test_long_rows(m, H):
    check_on_gpu(m, [70, 64, 65, 100, 33, 129, 40, 60], H, 63 * 256 + 8, BF16)


@pytest.mark.parametrize("H", [800, 1300])
@pytest.mark.parametrize("N", [836, 1028, 1412])
def test_fp32_many_split_tiles(m, H, N):
    check_on_gpu(m, [50, 1, 130, 64, 0, 47, 33, 80], H, N, FP32)


# weights of 128 MiB, which are not streamed, and of 256 MiB and more, all but 96 MiB of which are where an expert's rows fit one tile
# and not where they take two: the line lies inside an expert, on a column tile's edge or beside it
@pytest.mark.parametrize("sizes,H,N,dtype", [
    ([16, 1, 0, 17, 33, 5, 32, 40], 4096, 2056, BF16),                                   # 32 x 64
    ([40, 64, 65, 1, 0, 33, 48, 50] * 2, 4096, 2056, BF16),                              # 64 x 128
    ([40, 64, 65, 1, 0, 33, 48, 50] * 8, 1472, 2056, BF16),                              # plain on rows below 1536
    ([40, 64, 65, 1, 0, 33, 48, 50] * 8, 1536, 2056, BF16),
    ([150, 256, 257, 65, 0, 64, 300, 255, 33] * 2, 4096, 2056, BF16),                    # 256 x 256: plain up to rows of 4096
    ([150, 256, 257, 65, 0, 64, 300, 255] * 4, 2048, 2056, BF16),
    ([150, 256, 257, 65, 0, 64, 300, 255, 33] * 2, 4160, 2056, BF16),                    # the ragged tiles last
    ([150, 256, 257, 65, 0, 64, 300, 255] * 4, 4160, 2056, BF16),                        # in place
    ([16, 1, 0, 17, 33, 5, 32, 40], 2048, 2052, FP32),
    ([40, 64, 65, 1, 0, 33, 48, 50] * 2, 1024, 2052, FP32),
    ([16, 1, 0, 17, 33, 5, 32, 40], 4096, 4112, BF16),
    ([1, 0, 0, 0, 9], 8192, 8200, BF16),                                                 # 4.5 of 5 experts counted
    ([1, 0, 0, 1], 8192, 8200, BF16),                                                    # 1.75 of 4: below the line
    ([16, 1, 0, 17, 33, 5, 32, 40], 2048, 4104, FP32),
    ([40, 64, 65, 1, 0, 33, 48, 50] * 2, 1024, 4104, FP32),
], ids=["32x64-plain", "64x128", "64x128-plain", "64x128-short", "last-plain", "inplace-plain", "last", "inplace", "fp32-plain", "fp32-64x64-plain", "32x64", "32x64-few", "32x64-two", "fp32", "fp32-64x64"])
def test_streamed_weights(m, sizes, H, N, dtype):
    check_on_gpu(m, sizes, H, N, dtype)


# rows of a ragged tile around its 32-row steps (two halves of 16-row blocks), around the 64 rows of the short tile and around
# whole tiles; columns of one lane group and of one and of two tiles
@pytest.mark.parametrize("H", [64, 128, 192])
@pytest.mark.parametrize("N", [8, 248, 264])
def test_long_segments(m, H, N):
    check(m, [65, 96, 97, 0, 129, 224, 225, 240, 255, 256, 257, 321, 64], H, N, BF16)


# so many tiles that they are 256 x 256: ragged tiles last (2056 and 4104 features) or in place (6664), up to 256 rows per expert
# on average or more; one step of the hidden axis, fewer than the stages, and more
@pytest.mark.parametrize("H", [64, 128, 320])
@pytest.mark.parametrize("sizes,N", [
    ([65, 96, 97, 0, 129, 224, 225, 240, 255, 256, 257, 513, 64, 700], 2056),
    ([577, 320, 61, 257], 4104),
    ([65, 96, 97, 0, 129, 224, 225, 240, 255, 256, 257, 321, 64], 6664),
    ([300, 512, 769, 33, 255], 6664 * 2),
], ids=["last-short", "last-long", "inplace-short", "inplace-long"])
def test_big_tiles(m, sizes, N, H):
    check(m, sizes, H, N, BF16)


# few rows per expert: row counts around the 16-row blocks and past one tile, hidden sizes of fewer steps than waves and
# of several turns of the registers in flight, columns of one lane group and of several workgroups
@pytest.mark.parametrize("sizes", [[1], [1, 0, 2, 0], [16, 1, 7], [17, 33, 4, 31, 0, 15], [64, 65, 20, 1, 129, 40]], ids=str)
@pytest.mark.parametrize("H,N", [(64, 8), (192, 72), (256, 520), (2176, 40), (4096, 264)])
def test_few_rows(m, sizes, H, N):
    check(m, sizes, H, N, BF16)


# one row of x in a tile, the smallest descriptor, with about as many steps as there are stages in flight, so that loads past
# the row's end are issued (tiles of 32 x 64, and of 64 x 128 where the columns are many; ragged tiles of one row of the
# 256 x 256 form are among its own cases above)
@pytest.mark.parametrize("H", [64, 128, 192, 256])
@pytest.mark.parametrize("sizes,N", [([1, 33], 8), ([65], 16264)], ids=["32x64", "64x128"])
def test_one_row_tiles(m, sizes, N, H):
    check(m, sizes, H, N, BF16)


def test_few_rows_many_columns(m):
    """More column tiles than one round of workgroups; segments of several row tiles."""
    check(m, [5, 30, 1, 12], 128, 8200, BF16)
    check(m, [5, 30, 1, 12], 128, 4104, BF16)


# 64 x 64 tiles of fp32: rows and columns on both sides of the 32-row halves and of the tile, hidden sizes that are not
# whole 32-element steps
@pytest.mark.parametrize("H", [4, 32, 36, 100])
@pytest.mark.parametrize("N", [4, 32, 64, 132])
def test_fp32_tiles(m, H, N):
    check(m, [1, 31, 32, 33, 0, 64, 65, 130], H, N, FP32)


# rows that are not whole steps: a last step of one, of some and of all but one pieces of 16 bytes, alone, after fewer steps than
# there are stages and after more; the pieces past a row's end belong to the next row (integers as well) or to nothing
@pytest.mark.parametrize("H", [8, 56, 72, 184, 200, 328])
@pytest.mark.parametrize("sizes,N", [
    ([1, 17, 33, 0, 16], 72),                                                  # 32 x 64
    ([65, 64, 1], 16264),                                                      # 64 x 128
    ([65, 96, 97, 0, 129, 224, 225, 240, 255, 256, 257, 513, 64, 700], 2056),  # 256 x 256, the ragged tiles last ...
    ([577, 320, 61, 257, 500], 4104),                                          # ... with the third stage of weights or without
    ([65, 96, 97, 0, 129, 224, 225, 240, 255, 256, 257, 321, 64], 6664),       # in place
    ([480, 512, 769, 33, 512], 6664 * 2),
    ([300, 290, 310, 257, 384, 280, 1, 320], 1032),                            # register-staged
], ids=["32x64", "64x128", "last-short", "last-long", "inplace-short", "inplace-long", "staged"])
def test_ragged_steps(m, sizes, N, H):
    check(m, sizes, H, N, BF16)


# such rows of up to 448 elements and just beyond: both sides of the lines between 32 x 64, 64 x 128 and the register-staged tiles
@pytest.mark.parametrize("H", [8, 56, 72, 440, 456])
@pytest.mark.parametrize("sizes,N", [([16, 17, 15, 16] * 16, 1280), ([16, 17, 15, 16] * 16, 1288), ([17, 18, 16, 17] * 16, 648),
                                     ([8, 9, 7, 8] * 16, 4104), ([9, 10, 8, 9] * 16, 4104), ([56, 57, 55, 56] * 4, 7624),
                                     ([57, 58, 57, 56] * 4, 7624), ([130, 1, 128, 129, 77, 255, 0, 31] * 3, 5128)],
                         ids=["16", "16-many", "17", "8", "9", "56", "57", "many"])
def test_short_ragged_steps(m, sizes, N, H):
    check_on_gpu(m, sizes, H, N, BF16)


@pytest.mark.parametrize("H,N", [(520, 248), (520, 256), (1096, 256), (520, 264), (1112, 256)])
def test_ragged_steps_one_column_tile(m, H, N):
    check_on_gpu(m, [130, 1, 128, 129, 577, 455, 0, 231] * 12, H, N, BF16)


# fp32 tiles of 64 x 64, and several levels of sums
@pytest.mark.parametrize("H", [4, 36, 60, 260, 1100])
def test_fp32_one_tile_per_expert(m, H):
    check(m, [33, 40, 64, 1, 65, 48, 0, 47], H, 4100, FP32)


@pytest.mark.parametrize("H", [508, 516, 1100])
def test_fp32_levels(m, H):
    check(m, [1, 16, 17, 33, 200], H, 132, FP32)


# both sides of the longest row whose tiles fit the 31-bit offsets of the direct loads, 2^20 elements: the register-staged forms beyond
@pytest.mark.parametrize("H,dtype", [(2 ** 20 - 8, BF16), (2 ** 20, BF16), (2 ** 20 + 8, BF16), (2 ** 20 - 4, FP32), (2 ** 20, FP32),
                                     (2 ** 20 + 4, FP32)])
@pytest.mark.parametrize("sizes", [[3, 1], [33, 0, 65]], ids=str)
def test_longest_rows(m, sizes, H, dtype):
    check_on_gpu(m, sizes, H, 72, dtype)


# rows a multiple of 4096 bytes apart, whose tiles start their walk at different steps: a start in every step, an expert without rows, experts
# of one tile and of two; both sides of the lines at seven eighths of a tile's rows on average, 28 of 32 and 56 of 64
@pytest.mark.parametrize("sizes,H,N,dtype", [
    ([28, 1, 0, 33, 16, 40, 27, 32] * 3, 2048, 2056, BF16),
    ([28, 1, 0, 33, 16, 40, 27, 32] * 3, 6144, 2056, BF16),
    ([56, 1, 0, 65, 48, 64, 33, 40] * 4, 2048, 2056, BF16),
    ([28, 29, 28, 28] * 2, 2048, 2056, BF16),
    ([29, 30, 28, 29] * 2, 2048, 2056, BF16),
    ([56, 57, 55, 56] * 6, 2048, 2056, BF16),
    ([57, 58, 56, 57] * 6, 2048, 2056, BF16),
    ([28, 1, 0, 33, 16, 40, 27, 32] * 3, 1024, 2052, FP32),
], ids=["32x64", "32x64-long", "64x128", "28", "29", "56", "57", "fp32"])
def test_spread_starts(m, sizes, H, N, dtype):
    check_on_gpu(m, sizes, H, N, dtype)


# few tiles, their steps dealt to four or eight waves: rows around the 16-row blocks, one row, none; 8 steps, whole and not, two a wave; 23 and
# 24, and shares of unequal length and of several levels of sums; columns of one lane group, of a block and more.  [40, 100, ...] take
# 16 x 32 tiles and, with more columns, 32 x 32
@pytest.mark.parametrize("H", [456, 512, 1024, 1472, 1480, 2568, 8192, 8200])
@pytest.mark.parametrize("sizes,N", [([1], 8), ([16, 1, 7, 0, 17], 40), ([33, 31, 15, 32], 264), ([40, 100, 65, 0, 33], 136), ([40, 100, 65, 0, 33], 392)],
                         ids=["one", "few", "32", "16x32", "32x32"])
def test_split_tiles(m, sizes, N, H):
    check_on_gpu(m, sizes, H, N, BF16)


@pytest.mark.parametrize("H", [252, 256, 516, 740, 1284, 4096, 4100])
@pytest.mark.parametrize("sizes,N", [([1], 4), ([16, 1, 7, 0, 17], 20), ([33, 31, 15, 32], 264), ([40, 100, 65, 0, 33], 132), ([40, 100, 65, 0, 33], 392)],
                         ids=["one", "few", "32", "16x32", "32x32"])
def test_split_tiles_fp32(m, sizes, N, H):
    check_on_gpu(m, sizes, H, N, FP32)


# fewer rows than half a tile's: both sides of the line at one column tile per CU, 256, counted by experts, and both forms on the near side
@pytest.mark.parametrize("dtype", [BF16, FP32])
@pytest.mark.parametrize("sizes,N", [([5, 4, 6, 5], 2048), ([5, 4, 6, 5], 2056), ([12, 10, 14, 0, 12], 2048), ([12, 11, 13, 12], 2056),
                                     ([1] * 16, 640)], ids=["16x32", "16x32-more", "32x32", "32x32-more", "one"])
def test_split_tiles_of_few_rows(m, sizes, N, dtype):
    check_on_gpu(m, sizes, 1544, N, dtype)
