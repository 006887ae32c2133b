"""Gate projection on the edges of its tiles: token, expert and hidden counts around the 16 x 16 tiles with a split hidden
axis (fewer steps than waves, steps that do not divide among them, rows that end inside a step) and around the larger tiles
of a few thousand tokens.  Small-integer inputs: every partial sum is an integer below 2^24, so any order of additions gives
the same fp32 value and the comparison is exact."""
import numpy as np
import pytest
import torch

import workloads
from workloads import BF16, FP32

pytestmark = pytest.mark.gpu

SPLIT = [(1, 4, 1), (16, 28, 16), (17, 32, 17), (31, 60, 33), (40, 64, 9), (5, 224, 255), (48, 480, 48), (300, 448, 256), (260, 2044, 10)]
# fp32 with at most four experts: a wave per token; rows shorter than a wave, and with a remainder; both sides of its limit
FEW = [(1, 4, 1), (2, 252, 4), (7, 256, 2), (5, 260, 3), (1025, 1028, 4), (33, 8196, 1), (3072, 516, 4), (3073, 516, 4),
       (13000, 512, 3)]
TILES = [(2049, 64, 80), (4128, 128, 65), (8161, 64, 32), (8192, 192, 129), (16383, 64, 200), (4100, 320, 64), (4097, 64, 16)]


def check(T, H, E, dtype):
    import paper_2411_00662_amd as m
    from paper_2411_00662_amd import buffers as bufs
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(T + H + E)
    x = rng.integers(-4, 5, size=(T, H)).astype(np.float32)
    w = rng.integers(-4, 5, size=(E, H)).astype(np.float32)
    act = workloads.f32_to_bf16_bits if dtype == BF16 else np.ascontiguousarray
    cfg = m.make_cfg(T, H, dtype, E, 1, 1, 1, 1, 0.0)
    out = torch.full((T + 1, E), float("nan"), device="cuda:0")
    m.monta_gate(cfg, bufs.to_device_act(cfg, act(x)), bufs.to_device_act(cfg, act(w)), out[:T])
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.all(np.isnan(got[T]))
    np.testing.assert_array_equal(got[:T], (x.astype(np.float64) @ w.astype(np.float64).T).astype(np.float32))


@pytest.mark.parametrize("T,H,E", SPLIT + FEW + TILES)
def test_gate_fp32(T, H, E):
    check(T, H, E, FP32)


# both sides of the lines between the forms: one and two rounds of split tiles, 4096 and 8192 tokens, 16 / 17, 32 / 33 and 48 / 49
# experts on short, middling, 8-KiB and long rows, two and three short tiles per CU
RULE = [(2048, 128, 48), (2560, 128, 40), (1024, 192, 65), (1536, 192, 65), (8192, 320, 16), (8193, 320, 16), (5000, 2112, 16),
        (5000, 2112, 17), (6144, 2048, 32), (6144, 2048, 33), (6144, 4096, 48), (6145, 4096, 48), (8192, 3072, 48), (8193, 3072, 48),
        (8192, 3072, 49), (5000, 4160, 24), (5000, 200, 24), (16385, 64, 64), (24576, 128, 33), (24577, 128, 64), (24577, 64, 16),
        (6200, 8192, 65), (6144, 8192, 128)]


@pytest.mark.parametrize("T,H,E", [(T, (H + 7) // 8 * 8, E) for T, H, E in SPLIT] + TILES + RULE)
def test_gate_bf16(T, H, E):
    check(T, H, E, BF16)


# few tiles, their steps dealt to four or eight waves: one token, seven steps (other forms) and eight, the last of them one piece and whole, steps
# that do not divide, pieces past a row's end, both sides of the lines between 16 x 16 (200 tiles, eight waves up to 128), 16 x 32, 32 x 32
# and 32 x 64 (256 tiles); activations of 96 MiB and of more, which split tiles in registers take in 16 x 16 and 16 x 32
FEW_BF16 = [(1, 448, 9), (1, 456, 9), (1, 504, 9), (1, 512, 9), (17, 520, 33), (16, 1032, 16), (3199, 512, 5), (3200, 520, 16), (3201, 512, 16),
            (2048, 8192, 16), (2049, 8200, 16), (4096, 600, 32), (4097, 1024, 32), (8192, 1024, 32), (8193, 1024, 32), (5120, 1000, 30),
            (5121, 1000, 30), (8192, 2048, 64), (8193, 2048, 64), (8192, 2040, 33), (2000, 2056, 250), (100, 4104, 256), (6144, 8192, 16),
            (6145, 8192, 16), (8193, 8184, 9), (4095, 12296, 17), (4096, 12296, 17)]


@pytest.mark.parametrize("T,H,E", FEW_BF16)
def test_gate_few_tiles(T, H, E):
    check(T, H, E, BF16)


# bf16: rows that are not whole steps in the direct-to-LDS tiles of each shape, and the lines drawn for them; short rows on up to 8
# experts; two persistent workgroups per CU; and activations of 256 MiB, which are not streamed yet, and of 300 MiB, which are
RAGGED = [(4100, 520, 33), (8161, 72, 9), (9000, 2056, 64), (12000, 1096, 200), (16353, 2056, 24), (16352, 2056, 24), (6000, 8, 100),
          (8200, 200, 128), (3000, 1032, 256), (33000, 1016, 32), (33000, 1032, 32)]
SHORT_ROWS = [(2049, 8, 2), (2048, 64, 8), (5000, 1024, 8), (4097, 520, 5), (40001, 16, 1), (2049, 1088, 8)]
PERSISTENT = [(5000, 1536, 7), (9001, 2048, 8), (4095, 1088, 3)]
STREAMED = [(32768, 4096, 40), (32801, 4096, 65), (38400, 4096, 40), (38433, 4096, 65), (38480, 4088, 64)]


# both sides of the lines between the direct-to-LDS tiles: one, two and three rounds of 32 x 64 and 32 x 128 on rows of up to 2 KiB, of
# up to 4 KiB, of 8 KiB and others, with columns that fill their tiles or not; split tiles on some rows of 1 to 2 KiB
LINES = [(2730, 64, 129), (5461, 1024, 129), (5473, 64, 129), (8192, 512, 256), (8193, 64, 256), (8192, 1536, 128), (8193, 1536, 128),
         (3072, 1536, 129), (4096, 2112, 129), (4113, 2112, 129), (5473, 2112, 129), (8192, 4096, 192), (8193, 4096, 192), (8192, 4096, 128),
         (8193, 2112, 256), (24576, 1088, 33), (24577, 1088, 33), (24577, 1024, 64), (4096, 520, 17), (4097, 520, 17), (4096, 512, 17),
         (6188, 1784, 192), (4096, 576, 17), (4096, 1024, 24), (4096, 1024, 25), (4096, 952, 24)]


@pytest.mark.parametrize("T,H,E", RAGGED + SHORT_ROWS + PERSISTENT + STREAMED + LINES)
def test_gate_bf16_further(T, H, E):
    check(T, H, E, BF16)


# fp32 in the direct-to-LDS tiles: 32 x 64 and 64 x 64, and both sides of their lines
@pytest.mark.parametrize("T,H,E", [(8161, 896, 17), (8160, 892, 17), (8161, 1000, 64), (8160, 900, 33), (16001, 1004, 65), (15969, 1004, 65),
                                   (2017, 1124, 256), (31970, 900, 64)])
def test_gate_fp32_tiles(T, H, E):
    check(T, H, E, FP32)


# both sides of the longest row whose tiles fit the 31-bit offsets of the direct loads; made and multiplied for the reference on the GPU
# (fp32 products and sums of these integers are exact in any order)
@pytest.mark.parametrize("H,dtype", [(2 ** 20 - 8, BF16), (2 ** 20, BF16), (2 ** 20 + 8, BF16), (2 ** 20 - 4, FP32), (2 ** 20 + 4, FP32)])
@pytest.mark.parametrize("T,E", [(5, 9), (272, 256)])
def test_gate_longest_rows(T, E, H, dtype):
    import paper_2411_00662_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(T)
    x, w = (torch.randint(-4, 5, (n, H), generator=g, device="cuda", dtype=torch.int8).to(torch.float32 if dtype == FP32 else torch.bfloat16)
            for n in (T, E))
    out = torch.full((T + 1, E), float("nan"), device="cuda")
    m.monta_gate(m.make_cfg(T, H, dtype, E, 1, 1, 1, 1, 0.0), x, w, out[:T])
    assert bool(torch.isnan(out[T]).all())
    assert torch.equal(out[:T], x.float() @ w.float().t())


# rows 4096 bytes or a multiple of it apart in the direct-to-LDS tiles of each shape, and in the forms around them
@pytest.mark.parametrize("T,H,E", [(16384, 2048, 64), (12000, 8192, 64), (12001, 4096, 128), (9001, 6144, 100), (4097, 2048, 9), (33, 4096, 40),
                                   (40000, 2048, 20), (40000, 2048, 100), (9001, 2048, 8), (6145, 8192, 16), (300, 7168, 256)])
def test_equal_tokens_have_equal_logits(T, H, E):
    """Bit for bit, wherever in the batch they stand."""
    import paper_2411_00662_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn((1, H), generator=g, device="cuda").to(torch.bfloat16).repeat(T, 1)
    w = torch.randn((E, H), generator=g, device="cuda", dtype=torch.bfloat16) * H ** -0.5
    out = torch.empty((T, E), device="cuda")
    m.monta_gate(m.make_cfg(T, H, BF16, E, 1, 1, 1, 1, 0.0), x, w, out)
    assert bool((out == out[0]).all())
