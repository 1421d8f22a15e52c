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


# Layers whose weights do not fit the 256 MB Infinity Cache read those that one tile uses once with nontemporal loads, single experts do not:
# same bits.  d, f, rows, cap: the kernel for few rows with whole tiles (8 experts, more than the seven that fit) and with halved ones (an
# expert that does not fit by itself); 256x256 tiles of one row tile with 1 to 256 rows, whose lower wavefronts have all, some or no
# rows, beside an expert of two row tiles and one without rows; the counts decide (few rows, tiles).
@pytest.mark.parametrize("d,f,rows,cap", [(4096, 1536, [1, 3, 17, 16, 1, 33, 2, 55], 128), (4096, 14336, [2], 2),
                                          (2048, 2304, [1, 64, 65, 129, 200, 256, 33, 0, 300, 96], 5000),
                                          (2048, 2304, [9, 1, 2, 17, 1, 4, 2, 1, 3, 5], 400), (2048, 2304, [100] * 10, 1280)])
def test_weights_beyond_the_cache(d, f, rows, cap):
    print(f"case beyond-cache-{d}-{f}-{rows[:4]}", flush=True)
    e_cnt, R = len(rows), sum(rows)
    g = torch.Generator(device="cuda").manual_seed(d + f + R)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)  # noqa: E731
    x, w1, w3, w2 = randn(R, d), randn(e_cnt, d, f) * d ** -0.5, randn(e_cnt, d, f) * d ** -0.5, randn(e_cnt, f, d) * f ** -0.5

    def forward(x, rows, weights, cap):
        n = sum(rows)
        offsets = torch.tensor([0] + rows, device="cuda").cumsum(0).to(torch.int32)
        xp = torch.full((cap, d), float("nan"), device="cuda", dtype=torch.bfloat16)
        xp[:n] = x
        h1, h3, o, a = (torch.full((cap, m), 3.0, device="cuda", dtype=torch.bfloat16) for m in (f, f, d, f))
        ws = torch.empty(B.moe_workspace_bytes(B.WS_EXPERT_FWD, B.MOE_BF16, n, 1, d, f, len(rows), cap), dtype=torch.uint8, device="cuda")
        B.moe_expert_fwd(xp, offsets, *weights, h1, h3, o, ws, a=a)
        assert all((t[n:] == 3.0).all() for t in (h1, h3, a, o))
        return [t[:n] for t in (h1, h3, a, o)]

    got = forward(x, rows, (w1, w3, w2), cap)
    first = 0
    for e, n in enumerate(rows):
        if n == 0:
            continue
        part = slice(first, first + n)
        first += n
        alone = forward(x[part], [n], [w[e:e + 1].contiguous() for w in (w1, w3, w2)], 129 + n)
        for name, t, ref in zip(("h1", "h3", "a", "o"), got, alone):
            assert torch.equal(t[part].view(torch.int16), ref.view(torch.int16)), (name, e)
        h1, h3 = x[part].float() @ w1[e].float(), x[part].float() @ w3[e].float()
        want = (torch.nn.functional.silu(h1) * h3) @ w2[e].float()
        # a is rounded once and o once: a few 2^-9 of the largest
        assert (got[3][part].float() - want).abs().max() < 2e-2 * want.abs().max(), e
