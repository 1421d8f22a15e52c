"""The expert forward gives a row the same bits whatever the capacity of its buffers: the capacity picks the kernel (few rows or
256x256 tiles, or the row counts pick between the two), and both add an output up along ascending k."""
import pytest
import torch

from paper_2605_11005_amd import binding as B

pytestmark = pytest.mark.gpu


# 1, 2 and 4 groups of 16 rows and a second block of 64; contractions of 2 steps of 32, of a last round with 2 of its 4 steps and
# of whole rounds; columns past the end of a block of 128; empty experts; more experts than lanes
@pytest.mark.parametrize("d,f,rows", [(64, 64, [1]), (192, 320, [16, 17]), (1088, 64, [33, 0, 31]), (256, 192, [64, 65, 127]),
                                      (2048, 1408, [0, 3, 40, 0, 17, 1, 100, 70]), (448, 704, [5, 0] * 40), (4096, 1536, [4, 2, 1, 1, 0, 0]),
                                      # at most 64 tiles, which are halved, and one more; a last round with 2 of its 4 steps
                                      (2112, 2048, [1, 33]), (2112, 2048, [1, 33, 64]),
                                      # more than 256 MB of weights: with the middle capacity the counts decide, for few rows and for tiles
                                      (2048, 2304, [9, 0, 0, 17, 1, 0, 2, 0, 0, 0]), (2048, 2304, [100, 90, 110, 120, 80, 100, 95, 60, 128, 99])])
def test_forward_bits_do_not_depend_on_the_capacity(d, f, rows):
    print(f"case capacity-{d}-{f}-{rows[:8]}", flush=True)
    e_cnt, R = len(rows), sum(rows)
    g = torch.Generator(device="cuda").manual_seed(d + f + R)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)  # noqa: E731
    x, w1, w3, w2 = randn(R, d), randn(e_cnt, d, f) * d ** -0.5, randn(e_cnt, d, f) * d ** -0.5, randn(e_cnt, f, d) * f ** -0.5
    offsets = torch.tensor([0] + rows, device="cuda").cumsum(0).to(torch.int32)
    results = []
    for cap in (R, max(R, 100 * e_cnt), 128 * e_cnt + R):         # the last is above every bound of the kernel for few rows
        xp = torch.full((cap, d), float("nan"), device="cuda", dtype=torch.bfloat16)
        xp[:R] = x
        h1, h3, o, a = (torch.full((cap, n), 3.0, device="cuda", dtype=torch.bfloat16) for n in (f, f, d, f))
        ws = torch.empty(B.moe_workspace_bytes(B.WS_EXPERT_FWD, B.MOE_BF16, R, 1, d, f, e_cnt, cap), dtype=torch.uint8, device="cuda")
        B.moe_expert_fwd(xp, offsets, w1, w3, w2, h1, h3, o, ws, a=a)
        torch.cuda.synchronize()
        for t in (h1, h3, a, o):
            assert torch.isfinite(t).all() and (t[R:] == 3.0).all()
        results.append([t[:R].view(torch.int16) for t in (h1, h3, a, o)])
    for name, *same in zip(("h1", "h3", "a", "o"), *results):
        assert all(torch.equal(t, same[0]) for t in same), name
