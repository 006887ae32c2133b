"""Many tokens are projected as exactly as few: the forms that serve them differ, the error against 64 bits must not grow.  A call of
512 tokens or fewer splits the hidden axis over the waves of a workgroup; the logits of a larger call are held to those of such
calls on its parts, token by token the same sums.  2 % stand for the spread of the error itself: it is a root mean square over at
least 36,000 logits, whose relative deviation is below 1 / sqrt(2 * 36000) = 0.4 %."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,E", [(4096, 1024, 17), (4096, 768, 32), (2048, 768, 64), (2574, 592, 32), (2733, 640, 20), (800, 1024, 128),
                                   (5444, 384, 16), (3654, 360, 20), (1544, 320, 64), (2955, 320, 20), (2100, 256, 20), (2048, 512, 40),
                                   (3000, 448, 24), (6000, 504, 12), (3000, 520, 20), (4096, 960, 24), (4096, 896, 17), (4096, 704, 25)])
def test_error_of_many_tokens(T, H, E):
    import paper_2411_00662_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(T + H + E)
    x = torch.randn((T, H), generator=g, device="cuda", dtype=torch.bfloat16)
    w = torch.randn((E, H), generator=g, device="cuda", dtype=torch.bfloat16) * H ** -0.5
    exact = x.double() @ w.double().t()

    def error(tokens):
        logits = torch.empty((T, E), device="cuda")
        for lo in range(0, T, tokens):
            part = x[lo:lo + tokens]
            m.monta_gate(m.make_cfg(part.shape[0], H, m.BF16, E, 1, 1, 1, 1, 0.0), part, w, logits[lo:lo + tokens])
        return float((logits.double() - exact).norm() / exact.norm())

    assert error(T) <= 1.02 * error(512)
