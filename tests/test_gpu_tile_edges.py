"""GPU parity at the edges of the expert kernels' tiles, against the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2605_11005_amd import binding as B
from paper_2605_11005_amd import workloads as W
from paper_2605_11005_amd.layer import run_backward
from tests.gpu_util import TOL, check_layer, gpu_layer, host, make_inputs, oracle_layer, rel_err

pytestmark = pytest.mark.gpu


# fp32 tiles are 64 x 64 with k-tiles of 32 (an odd number of them takes a path of its own); one expert: its rows are T
@pytest.mark.parametrize("T,d,f", [(1, 4, 4), (63, 36, 68), (64, 64, 32), (65, 100, 132), (130, 128, 60), (31, 196, 64)])
def test_fp32_experts_at_tile_edges(T, d, f):
    wl = W.TINY.scaled(name=f"fp32-edge-{T}-{d}-{f}", T=T, d=d, f=f, E=1, e_cnt=1, k=1)
    print(f"case {wl.name}", flush=True)
    inp = make_inputs(wl)
    fw, bw = oracle_layer(wl, inp)
    dev, buf = gpu_layer(wl, inp)
    check_layer(wl, inp, fw, bw, buf)
    run_backward(wl, dev, buf, accumulate=True)
    torch.cuda.synchronize()
    for got, ref in ((buf.dw1, bw["dw1"]), (buf.dw3, bw["dw3"]), (buf.dw2, bw["dw2"])):
        assert rel_err(host(got), 2.0 * ref) < TOL["f32"]


# numbers without three bf16 terms (infinities, what lies beyond 2^96) behave as fp32 products do, and so do sums of 1e-35
@pytest.mark.parametrize("T,d,f", [(70, 68, 132), (1, 36, 64)])
def test_fp32_experts_with_infinities(T, d, f):
    print(f"case fp32-inf-{T}-{d}-{f}", flush=True)
    g = torch.Generator().manual_seed(T)
    x = torch.randn((T, d), generator=g)
    w1, w3, w2 = (torch.randn(s, generator=g) * 1e-2 for s in ((d, f), (d, f), (f, d)))
    x[0, 3], x[T // 2, 35] = float("inf"), 3.4e38
    dev = lambda t: t.cuda().contiguous()  # noqa: E731
    h1, h3, o = (torch.empty((T, n), device="cuda") for n in (f, f, d))
    ws = torch.empty(B.moe_workspace_bytes(B.WS_EXPERT_FWD, B.MOE_F32, T, 1, d, f, 1, T), dtype=torch.uint8, device="cuda")
    offsets = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    B.moe_expert_fwd(dev(x), offsets, dev(w1[None]), dev(w3[None]), dev(w2[None]), h1, h3, o, ws)
    for got, w in ((h1, w1), (h3, w3)):
        ref, got = x.double() @ w.double(), got.cpu().double()
        assert torch.equal(torch.isinf(got), torch.isinf(ref)) and not torch.isnan(got).any()
        assert torch.equal(got[0], ref[0]) or T == 1           # the row of the infinity: its signs
        assert ((got - ref)[1:].norm(dim=1) <= 1e-5 * ref[1:].norm(dim=1)).all()
    x = torch.randn((T, d), generator=g) * 1e-33
    B.moe_expert_fwd(dev(x), offsets, dev(w1[None]), dev(w3[None]), dev(w2[None]), h1, h3, o, ws)
    for got, w in ((h1, w1), (h3, w3)):        # sums of up to 68 fp32 products
        ref = x.double() @ w.double()
        assert float((got.cpu().double() - ref).norm() / ref.norm()) < 68 ** 0.5 * 2.0 ** -24


def fp32_pass(rows, x, w1, w3, w2, d_o, h1=None, h3=None, a=None, cap=None):
    """Forward, then backward from the given h1, h3 and a where they are not the forward's, of experts with these rows."""
    R, (e_cnt, d, f) = sum(rows), w1.shape
    cap = cap or R
    up = lambda t: None if t is None else torch.cat([t, torch.zeros((cap - R, t.shape[1]))]).cuda()  # noqa: E731
    offsets = torch.tensor([0] + rows).cumsum(0).to(torch.int32).cuda()
    weights = [w.cuda() for w in (w1, w3, w2)]
    fh1, fh3, fa, o, dxp = (torch.zeros((cap, n), device="cuda") for n in (f, f, f, d, d))
    grads = [torch.zeros_like(w) for w in weights]
    wsf, wsb = (torch.empty(B.moe_workspace_bytes(which, B.MOE_F32, R, 1, d, f, e_cnt, cap), dtype=torch.uint8, device="cuda")
                for which in (B.WS_EXPERT_FWD, B.WS_EXPERT_BWD))
    B.moe_expert_fwd(up(x), offsets, *weights, fh1, fh3, o, wsf, a=fa)
    pick = lambda given, own: own if given is None else up(given)  # noqa: E731
    B.moe_expert_bwd(up(x), pick(h1, fh1), pick(h3, fh3), up(d_o), offsets, *weights, dxp, *grads, False, wsb, a=pick(a, fa))
    names = ("h1", "h3", "o", "dxp", "dw1", "dw3", "dw2")
    return dict(zip(names, [t[:R].cpu() for t in (fh1, fh3, o, dxp)] + [t.cpu() for t in grads]))


# numbers whose bf16 terms would lie below bf16's smallest ones, beside factors that make their sums ordinary; either operand of every
# GEMM, with one and two LDS buffers (the capacity decides)
@pytest.mark.parametrize("tiny,large", [(1e-33, 1e18), (1e-37, 1e22), (1e-41, 1e25), (2.0 ** -147, 1e28)])
@pytest.mark.parametrize("cap", [70, 40000])
def test_fp32_experts_hold_small_operands(tiny, large, cap):
    print(f"case fp32-small-{tiny}-{cap}", flush=True)
    T, d, f = 70, 68, 132
    g = torch.Generator().manual_seed(5)
    randn = lambda scale, *shape: torch.randn(shape, generator=g) * scale  # noqa: E731
    r = lambda t: t.double()  # noqa: E731
    for sx, sw in ((tiny, large), (large, tiny)):
        x, w1, w3, w2, d_o = randn(sx, T, d), randn(sw, 1, d, f), randn(sw, 1, d, f), randn(sw, 1, f, d), randn(sx, T, d)
        h1, h3, a = randn(1.0, T, f), randn(1.0, T, f), randn(sw, T, f)
        got = fp32_pass([T], x, w1, w3, w2, d_o, h1, h3, a, cap)
        sig = torch.sigmoid(r(h1))
        dA = r(d_o) @ r(w2[0]).T
        dh1, dh3 = dA * r(h3) * sig * (1 + r(h1) * (1 - sig)), dA * r(h1) * sig
        ref = {"h1": r(x) @ r(w1[0]), "h3": r(x) @ r(w3[0]), "dw2": r(a).T @ r(d_o)}
        # sums of up to 132 products, as fp32 makes them; dxp, dw1, dw3: of products with a rounded dh1, dh3 (a few roundings and expf)
        for name, want in ref.items():
            assert float((r(got[name]).reshape(want.shape) - want).norm() / want.norm()) < 132 ** 0.5 * 2.0 ** -24, (name, sx)
        ref = {"dxp": dh1 @ r(w1[0]).T + dh3 @ r(w3[0]).T, "dw1": r(x).T @ dh1, "dw3": r(x).T @ dh3}
        for name, want in ref.items():
            if float(want.norm()) / want.numel() ** 0.5 > 1e-30:          # (otherwise the results themselves are subnormal)
                assert float((r(got[name]).reshape(want.shape) - want).norm() / want.norm()) < TOL["f32"], (name, sx)


# what one row (for the weight gradients: one column) holds does not show in the bits of its neighbours in a tile
@pytest.mark.parametrize("what", [float("inf"), float("nan"), 3e38, 1e25, 1e-25, 1e-40])
@pytest.mark.parametrize("cap", [70, 40000])
def test_fp32_outputs_do_not_depend_on_their_neighbours(what, cap):
    print(f"case fp32-neighbours-{what}-{cap}", flush=True)
    T, d, f = 70, 68, 132
    g = torch.Generator().manual_seed(6)
    randn = lambda *shape: torch.randn(shape, generator=g)  # noqa: E731
    weights = (randn(1, d, f) * 0.1, randn(1, d, f) * 0.1, randn(1, f, d) * 0.1)
    acts = dict(x=randn(T, d), d_o=randn(T, d), h1=randn(T, f), h3=randn(T, f), a=randn(T, f))
    call = lambda c: fp32_pass([T], c["x"], *weights, c["d_o"], c["h1"], c["h3"], c["a"], cap)  # noqa: E731
    want = call(acts)
    rows, cols = torch.arange(T) != 5, torch.arange(f) != 7
    other = dict(acts, x=acts["x"].clone(), d_o=acts["d_o"].clone())
    other["x"][5], other["d_o"][5] = what, what
    got = call(other)
    for name in ("h1", "h3", "o", "dxp"):
        assert torch.equal(got[name][rows], want[name][rows]), name
    other = dict(acts, x=acts["x"].clone(), a=acts["a"].clone())
    other["x"][:, 7], other["a"][:, 7] = what, what
    got = call(other)
    for name in ("dw1", "dw3"):
        assert torch.equal(got[name][:, cols[:d]], want[name][:, cols[:d]]), name
    assert torch.equal(got["dw2"][:, cols], want["dw2"][:, cols])


# weight gradients of experts with one row are rounded products; of two rows, sums with a rounding per product and one of the sum
@pytest.mark.parametrize("d,f", [(4, 4), (68, 132), (260, 200)])
def test_fp32_weight_gradients_of_one_and_two_rows(d, f):
    print(f"case fp32-one-row-{d}-{f}", flush=True)
    rows, g = [1, 0, 2, 1, 3], torch.Generator().manual_seed(7)
    randn = lambda *shape: torch.randn(shape, generator=g)  # noqa: E731
    R, e_cnt = sum(rows), len(rows)
    x, d_o, a = randn(R, d), randn(R, d), randn(R, f)
    x[:, 0] = 1.0                              # row 0 of dw1 and dw3 then shows what the columns of x are multiplied by
    got = fp32_pass(rows, x, randn(e_cnt, d, f), randn(e_cnt, d, f), randn(e_cnt, f, d), d_o, randn(R, f), randn(R, f), a)
    off = [0] + list(np.cumsum(rows))
    for e in (0, 3):
        r = off[e]
        assert torch.equal(got["dw2"][e], a[r][:, None] * d_o[r][None, :])
        for name in ("dw1", "dw3"):
            assert torch.equal(got[name][e], x[r][:, None] * got[name][e][0][None, :]), name
    assert not any(got[name][1].any() for name in ("dw1", "dw3", "dw2"))
    a2, d2 = a[off[2]:off[3]].double(), d_o[off[2]:off[3]].double()
    assert ((got["dw2"][2].double() - a2.T @ d2).abs() <= 2.001 * 2.0 ** -24 * (a2.abs().T @ d2.abs())).all()


# launches of up to 512 blocks have two LDS buffers, larger ones one: the capacity decides for the forward, dA and dX, the widths for the
# weight gradients (576 blocks with 16 experts); one k-tile, odd and even numbers of them, empty experts
@pytest.mark.parametrize("d,f,rows", [(32, 64, [1]), (200, 520, [40, 0, 1, 33, 64, 65, 7, 0, 96, 3, 2, 1, 100, 0, 31, 32]), (100, 36, [70, 0, 33])])
def test_fp32_experts_with_one_and_two_buffers(d, f, rows):
    print(f"case fp32-buffers-{d}-{f}", flush=True)
    e_cnt, R = len(rows), sum(rows)
    g = torch.Generator().manual_seed(d + f)
    randn = lambda *shape: torch.randn(shape, generator=g)  # noqa: E731
    xp, d_o, w1, w3, w2 = randn(R, d), randn(R, d), randn(e_cnt, d, f) * d ** -0.5, randn(e_cnt, d, f) * d ** -0.5, randn(e_cnt, f, d) * f ** -0.5
    off = np.array([0] + rows).cumsum()
    args = [t.numpy().astype(np.float64) for t in (w1, w3, w2)]
    rh1, rh3, _, ro = O.expert_fwd(xp.numpy().astype(np.float64), off, *args)
    rdxp, rdw1, rdw3, rdw2 = O.expert_bwd(xp.numpy().astype(np.float64), rh1, rh3, d_o.numpy().astype(np.float64), off, *args)
    offsets, weights, results = torch.tensor(off, dtype=torch.int32, device="cuda"), [w.cuda() for w in (w1, w3, w2)], []
    for cap in (R, 40000):
        x, dy = (torch.zeros((cap, d), device="cuda") for _ in range(2))
        x[:R], dy[:R] = xp.cuda(), d_o.cuda()
        h1, h3, o, dxp = (torch.zeros((cap, n), device="cuda") for n in (f, f, d, d))
        dws = [torch.zeros_like(w) for w in weights]
        wsf, wsb = (torch.empty(B.moe_workspace_bytes(which, B.MOE_F32, R, 1, d, f, e_cnt, cap), dtype=torch.uint8, device="cuda")
                    for which in (B.WS_EXPERT_FWD, B.WS_EXPERT_BWD))
        B.moe_expert_fwd(x, offsets, *weights, h1, h3, o, wsf)
        B.moe_expert_bwd(x, h1, h3, dy, offsets, *weights, dxp, *dws, False, wsb)
        got = [t[:R] for t in (h1, h3, o, dxp)] + dws
        for t, ref in zip(got, (rh1, rh3, ro, rdxp, rdw1, rdw3, rdw2)):
            assert rel_err(host(t), ref) < TOL["f32"]
        results.append(got)
    assert all(torch.equal(a, b) for a, b in zip(*results))


# dA and dW2 share a launch where the forward's activation is kept, dX and dW1|dW3 always do: blocks beyond the tiles of the first GEMM,
# one and two LDS buffers and either GEMM first (the capacity decides), experts without rows, and the same bits as dA and dW2 in launches of
# their own
@pytest.mark.parametrize("d,f,rows", [(4, 4, [1]), (68, 132, [65, 0, 3, 64]), (200, 520, [40, 0, 129, 7] * 4)])
def test_fp32_gradients_that_share_launches(d, f, rows):
    print(f"case fp32-shared-{d}-{f}", flush=True)
    e_cnt, R = len(rows), sum(rows)
    g = torch.Generator().manual_seed(d * f)
    randn = lambda *shape: torch.randn(shape, generator=g)  # noqa: E731
    x, d_o, weights = randn(R, d), randn(R, d), [randn(e_cnt, d, f) * d ** -0.5, randn(e_cnt, d, f) * d ** -0.5, randn(e_cnt, f, d) * f ** -0.5]
    off, up = np.array([0] + rows).cumsum(), lambda t, cap: torch.cat([t, torch.zeros((cap - R, t.shape[1]))]).cuda()  # noqa: E731
    args = [t.numpy().astype(np.float64) for t in (x, *weights, d_o)]
    rh1, rh3, _, _ = O.expert_fwd(args[0], off, *args[1:4])
    refs = O.expert_bwd(args[0], rh1, rh3, args[4], off, *args[1:4])
    results = []
    for cap in (R, 40000):
        kept = fp32_pass(rows, x, *weights, d_o, cap=cap)
        results.append([kept[n] for n in ("dxp", "dw1", "dw3", "dw2")])
        dw, dxp = [torch.zeros_like(w).cuda() for w in weights], torch.zeros((cap, d), device="cuda")
        ws = torch.empty(B.moe_workspace_bytes(B.WS_EXPERT_BWD, B.MOE_F32, R, 1, d, f, e_cnt, cap), dtype=torch.uint8, device="cuda")
        B.moe_expert_bwd(up(x, cap), up(kept["h1"], cap), up(kept["h3"], cap), up(d_o, cap), torch.tensor(off, dtype=torch.int32, device="cuda"),
                         *[w.cuda() for w in weights], dxp, *dw, False, ws)
        for got, own, ref in zip(results[-1], (dxp[:R], *dw), refs):
            assert rel_err(host(got), ref) < TOL["f32"] and rel_err(host(own), ref) < TOL["f32"]
        assert all(torch.equal(got, own.cpu()) for got, own in zip(results[-1], (dxp[:R], *dw[:2])))
    assert all(torch.equal(a, b) for a, b in zip(*results))



# kernels for few rows: 16, 32 or 64 rows per block, wavefronts without a piece of the contraction (d = 64), columns past the end
@pytest.mark.parametrize("T,d,f", [(1, 64, 64), (16, 192, 320), (17, 1088, 64), (33, 64, 192), (64, 320, 128), (65, 128, 448), (127, 256, 64)])
def test_bf16_forward_with_few_rows(T, d, f):
    wl = W.QWEN.scaled(name=f"few-rows-{T}-{d}-{f}", T=T, d=d, f=f, E=1, e_cnt=1, k=1)
    print(f"case {wl.name}", flush=True)
    inp = make_inputs(wl)
    fw, bw = oracle_layer(wl, inp)
    dev, buf = gpu_layer(wl, inp)
    check_layer(wl, inp, fw, bw, buf)


# router logits: E = 8 n with column blocks of 128, row blocks of 16 to 64, contraction whole or cut into ranges: 8 equal ones
# (17, 4096, 128), 6 of 17 and 15 pieces (17, 3200, 128) and (40, 3200, 64); the 256x256 tiles from one block of 64 tokens by 128
# experts per CU on, their contraction cut into ranges of 5, 5, 5, 5 and 3 pairs of k-tiles (4100, 1472, 512) or whole (16500, 64, 64).
# fp32 sums of bf16 products: n products of N(0, 1/n) terms in any order are off by less than 1e-5 of the largest
@pytest.mark.parametrize("T,d,E", [(1, 64, 8), (15, 448, 24), (17, 4096, 128), (300, 2880, 136), (4100, 128, 192), (16500, 64, 64),
                                   (17, 3200, 128), (40, 3200, 64), (4100, 1472, 512)])
def test_router_logits_at_block_edges(T, d, E):
    print(f"case router-{T}-{d}-{E}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + d + E)
    x = torch.randn((T, d), generator=g, device="cuda", dtype=torch.bfloat16)
    wr = torch.randn((d, E), generator=g, device="cuda", dtype=torch.bfloat16).mul_(d ** -0.5)
    logits = torch.full((T, E), float("nan"), device="cuda")
    ws = torch.empty(B.moe_workspace_bytes(B.WS_ROUTER, B.MOE_BF16, T, 1, d, 0, E, 0), dtype=torch.uint8, device="cuda")
    B.moe_router_fwd(x, wr, logits, ws)
    assert rel_err(host(logits), host(x) @ host(wr)) < 1e-5


# plans of one block of 1024 slots and of several; up to 2048 slots the dispatch makes the plan itself
@pytest.mark.parametrize("T,k,e_cnt", [(1, 1, 1), (63, 1, 3), (64, 16, 64), (1024, 8, 7), (1025, 8, 7), (300, 4, 900), (300, 4, 901), (40, 2, 0)])
def test_plan_in_one_block_and_in_three_launches(T, k, e_cnt):
    print(f"case plan-{T}-{k}-{e_cnt}", flush=True)
    E, e_lo = 1024, 5
    ids = np.random.default_rng(T).permuted(np.tile(np.arange(E if e_cnt > 100 else 80), (T, 1)), axis=1)[:, :k].astype(np.int32)
    off_ref, perm_ref, inv_ref = O.plan(ids, e_lo, e_cnt)[:3]
    x = torch.zeros((T, 8), dtype=torch.bfloat16, device="cuda")
    idx = torch.from_numpy(ids).cuda()
    cap = T * k
    i32 = dict(dtype=torch.int32, device="cuda")
    off, perm, inv = torch.full((e_cnt + 1,), -7, **i32), torch.full((cap,), -7, **i32), torch.full((T, k), -7, **i32)
    ws = torch.empty(B.moe_workspace_bytes(B.WS_DISPATCH, B.MOE_BF16, T, k, 8, 8, e_cnt, cap), dtype=torch.uint8, device="cuda")
    B.moe_dispatch(x, k, idx, None, e_lo, e_cnt, off, perm, inv, False, torch.empty((cap, 8), dtype=torch.bfloat16, device="cuda"), ws)
    R = int(off_ref[-1])
    assert (host(off) == off_ref).all() and (host(inv) == inv_ref).all() and (host(perm)[:R] == perm_ref).all()
    assert int(ws[:4].view(torch.int32).item()) == 0


# one launch plans up to 16384 slots (32768 of 16 local experts or more, 65536 of 64 or more), several blocks of 1024; three beyond, and for
# more than 900 local experts
@pytest.mark.parametrize("T,k,e_cnt", [(1025, 2, 7), (4096, 4, 7), (4097, 4, 7), (8192, 4, 16), (8193, 4, 16), (8192, 8, 64), (8193, 8, 64), (1200, 8, 900), (600, 4, 900), (600, 4, 901), (1025, 2, 0)])
def test_plan_of_several_blocks(T, k, e_cnt):
    test_plan_in_one_block_and_in_three_launches(T, k, e_cnt)


# the same where most slots, or all, are one expert's, whose additions go to eight, four or one tables; other experts in between, slots that are
# not local, blocks whose first slots are
@pytest.mark.parametrize("T,k,e_cnt", [(2049, 1, 1), (5000, 1, 8), (16384, 1, 8), (3000, 3, 128), (3000, 3, 129), (2000, 8, 256), (2000, 8, 257)])
def test_plan_of_a_hot_expert(T, k, e_cnt):
    print(f"case hot-plan-{T}-{k}-{e_cnt}", flush=True)
    rng, e_lo, cap = np.random.default_rng(T + e_cnt), 3, T * k
    ids = rng.permuted(np.tile(np.arange(e_cnt + 20), (T, 1)), axis=1)[:, :k].astype(np.int32)
    hot = e_lo + e_cnt // 2
    ids[:, 0] = np.where((ids == hot).any(axis=1) | (rng.random(T) < 0.1), ids[:, 0], hot)
    off_ref, perm_ref, inv_ref = O.plan(ids, e_lo, e_cnt)[:3]
    i32 = dict(dtype=torch.int32, device="cuda")
    off, perm, inv = torch.full((e_cnt + 1,), -7, **i32), torch.full((cap,), -7, **i32), torch.full((T, k), -7, **i32)
    x, xp = torch.zeros((T, 8), dtype=torch.bfloat16, device="cuda"), torch.empty((cap, 8), dtype=torch.bfloat16, device="cuda")
    B.moe_dispatch_static(x, k, torch.from_numpy(ids).cuda(), None, e_lo, e_cnt, off, perm, inv, xp, torch.full((1,), -7, **i32))
    assert (host(off) == off_ref).all() and (host(inv) == inv_ref).all() and (host(perm)[:int(off_ref[-1])] == perm_ref).all()


# plan and move of few slots in one launch (up to 2048 slots, and 2**20 reads of slots by all blocks) and in two: one and several blocks
# per row, slots without a local expert, experts without rows, rows beyond the capacity, scaled rows of both types
@pytest.mark.parametrize("T,k,d,e_cnt,cap", [(1, 1, 8, 1, 1), (7, 3, 1032, 5, 21), (64, 16, 64, 64, 1024), (2048, 1, 72, 7, 2048), (2049, 1, 72, 7, 2049),
                                             (128, 2, 2056, 900, 256), (30, 64, 1024, 1000, 1920), (33, 4, 256, 8, 20), (9, 2, 64, 3, 0), (12, 2, 64, 0, 4)])
def test_plan_and_dispatch_of_few_slots(T, k, d, e_cnt, cap):
    print(f"case few-slots-{T}-{k}-{d}-{e_cnt}-{cap}", flush=True)
    E, e_lo = 1024, 2
    ids = np.random.default_rng(T + d).permuted(np.tile(np.arange(E if k > 20 or e_cnt > 100 else 24 if k <= 16 and e_cnt < 20 else 70), (T, 1)), axis=1)[:, :k].astype(np.int32)
    off_ref, perm_ref, inv_ref = O.plan(ids, e_lo, e_cnt)[:3]
    R = int(off_ref[-1])
    inv_ref = np.where(inv_ref < cap, inv_ref, -1)
    g = torch.Generator(device="cuda").manual_seed(T)
    i32 = dict(dtype=torch.int32, device="cuda")
    for dtype in (torch.bfloat16, torch.float32):
        x = torch.randn((T, d), generator=g, device="cuda").to(dtype)
        scale = torch.rand((T, k), generator=g, device="cuda")
        for rows in (None, scale):
            off, perm, inv = torch.full((e_cnt + 1,), -7, **i32), torch.full((max(cap, 1),), -7, **i32), torch.full((T, k), -7, **i32)
            xp, status = torch.full((max(cap, 1), d), 3.0, device="cuda", dtype=dtype), torch.full((1,), -7, **i32)
            B.moe_dispatch_static(x, k, torch.from_numpy(ids).cuda(), rows, e_lo, e_cnt, off, perm[:cap], inv, xp[:cap], status)
            n = min(R, cap)
            assert (host(off) == np.minimum(off_ref, cap)).all() and (host(inv) == inv_ref).all() and int(status) == int(R > cap)
            assert (host(perm)[:n] == perm_ref[:n]).all() and (perm[n:] == -7).all() and (xp[n:] == 3.0).all()
            s = torch.from_numpy(np.ascontiguousarray(perm_ref[:n])).cuda().long()
            want = x[s // k].float() * (1.0 if rows is None else rows.flatten()[s][:, None])
            assert torch.equal(xp[:n], want.to(dtype))



def _streams(T, d, E):
    """Whether the weight gradient of these sizes takes the streaming kernel: three planes of dlogits unless E % 64 == 0, and
    the operand and a sum per plane must fit where the sums of the cut product would go (rules of router.hip, expert_bf16.hip)."""
    up = lambda a, b: -(-a // b)  # noqa: E731
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    planes, sum_bytes = (1 if E % 64 == 0 else 3), 4 * d * E
    if planes == 1:
        tiles = up(d, 256) * up(E, 256)
        cost = lambda s: up(tiles * s, cus) * (up(up(T, s), 32) + 16)  # noqa: E731
        splits = min(range(1, min(32, up(T, 128)) + 1), key=cost)
    else:
        splits = max(1, min(up(4 * cus, up(d, 64) * up(E, 64)), (64 << 20) // sum_bytes, up(T, 64), 64))
    room, operand = up(splits * sum_bytes, 256) * 256, up(up(T, 32) * 64 * planes * E, 256) * 256
    large = planes == 1 and E > 64 and T * d > 1 << 26
    return T >= 32 and d % 64 == 0 and planes * E <= 128 and not large and room >= operand + planes * sum_bytes


# router backward: the streaming weight gradient (pieces of 32 tokens, the last one whole, of one token or of 31 with the overlap
# into the piece before it; one row block of planes, a second one, 128 rows), the kernels it leaves the rest to -- too few tokens
# for its operand to fit beside the sums, more than 128 rows of planes -- and the input gradient.
# bf16 dlogits (E % 64 == 0): one rounding, 2e-2 as everywhere; fp32 dlogits: bf16 stores only, 2**-8 of the largest
@pytest.mark.parametrize("T,d,E,streams", [
    (32, 64, 8, False), (33, 192, 8, False), (1000, 2048, 16, True), (31, 64, 8, False), (777, 320, 40, True), (500, 128, 48, False),
    (2049, 448, 64, True), (4000, 128, 128, True), (300, 64, 192, False),
    (288, 512, 8, True), (289, 512, 8, True), (319, 512, 8, True), (320, 512, 1, True), (1023, 128, 24, True), (256, 512, 64, True), (32, 64, 128, False)])
def test_router_backward_at_block_edges(T, d, E, streams):
    print(f"case router-bwd-{T}-{d}-{E}", flush=True)
    assert _streams(T, d, E) == streams
    g = torch.Generator(device="cuda").manual_seed(T + d + E)
    x = torch.randn((T, d), generator=g, device="cuda", dtype=torch.bfloat16)
    wr = torch.randn((d, E), generator=g, device="cuda", dtype=torch.bfloat16).mul_(d ** -0.5)
    dl = torch.randn((T, E), generator=g, device="cuda")
    dx = torch.randn((T, d), generator=g, device="cuda", dtype=torch.bfloat16)
    dx0 = host(dx)
    dwr = torch.full((d, E), float("nan"), device="cuda", dtype=torch.bfloat16)
    ws = torch.empty(B.moe_workspace_bytes(B.WS_ROUTER, B.MOE_BF16, T, 1, d, 0, E, 0), dtype=torch.uint8, device="cuda")
    B.moe_router_bwd(x, wr, dl, dwr, False, dx, True, ws)
    dwr_ref, dx_ref = O.router_bwd(host(x), host(wr), host(dl))
    tol = TOL["bf16"] if E % 64 == 0 else 2.0 ** -8
    assert rel_err(host(dwr), dwr_ref) < tol
    assert rel_err(host(dx), dx0 + dx_ref) < tol
    B.moe_router_bwd(x, wr, dl, dwr, True, None, False, ws)      # added to the gradient above, which was rounded once
    assert rel_err(host(dwr), 2.0 * dwr_ref) < tol


# router_dx.hip: rounded dlogits (E = 64, 128, 192, 256) and three terms of them (32, 96, 160); one token, tiles of 32 and 64 tokens with one
# more or less, several tiles and ranges per block; wavefronts past the last column.  Against the products of what the kernel is given
# (bf16 dlogits where E % 64 == 0), 2**-8 for the one rounding of a result, bit for bit without the products.  E = 320, 512 and 1024 are the
# grouped GEMM's
@pytest.mark.parametrize("T,d,E", [(1, 64, 32), (33, 192, 96), (65, 320, 32), (127, 256, 160), (31, 64, 64), (64, 576, 128), (129, 448, 192),
                                   (20011, 64, 96), (9001, 512, 64), (33, 320, 256), (1, 64, 320), (300, 576, 512), (129, 448, 1024)])
def test_router_input_gradient_stream(T, d, E):
    print(f"case router-dx-{T}-{d}-{E}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + d + E)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")  # noqa: E731
    x, wr, dl, dx0 = randn(T, d).bfloat16(), randn(d, E).bfloat16(), randn(T, E) * 0.1, randn(T, d).bfloat16()
    ws = torch.empty(B.moe_workspace_bytes(B.WS_ROUTER, B.MOE_BF16, T, 1, d, 0, E, 0), dtype=torch.uint8, device="cuda")
    ref = (dl.bfloat16() if E % 64 == 0 else dl).double() @ wr.double().t()
    for accumulate in (False, True):
        room = torch.full((T + 1, d), 3.0, device="cuda", dtype=torch.bfloat16)
        room[:T] = dx0
        B.moe_router_bwd(x, wr, dl, None, False, room[:T], accumulate, ws)
        want = ref + (dx0.double() if accumulate else 0.0)
        assert ((room[:T].double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5 * ref.abs().max()).all() and (room[T] == 3.0).all()
    dl[T // 2] = 0.0
    dl[T - 1, E - 1] = float("inf")
    B.moe_router_bwd(x, wr, dl, None, False, room[:T], False, ws)
    assert (room[T - 1] == wr[:, E - 1].float() * float("inf")).all() and (T < 3 or (room[T // 2] == 0.0).all())
    assert torch.isfinite(room[:T - 1]).all()


# the same with infinities, where the terms that are zero multiply an infinite weight: dlogits of one and two terms, a row that rounds up to
# infinity, and infinite weights in several columns of a wavefront
@pytest.mark.parametrize("T,d,E", [(33, 192, 96), (65, 320, 32), (127, 256, 160)])
def test_router_input_gradient_of_infinities(T, d, E):
    print(f"case router-dx-inf-{T}-{d}-{E}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + d + E)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")  # noqa: E731
    x, wr, dl, dx0 = randn(T, d).bfloat16(), randn(d, E).bfloat16(), randn(T, E), randn(T, d).bfloat16()
    dl[::2] = dl[::2].bfloat16().float()
    wr[3, 1] = wr[5, E - 1] = wr[d - 1, 7] = float("inf")
    wr[4, 0] = -float("inf")
    dl[7, 2], dl[8, 2], dl[9, 5], wr[:, 5] = float("inf"), -float("inf"), 3.4e38, 2.0 ** -30
    want, size = dl.double() @ wr.double().t(), dl.double().abs() @ wr.double().abs().t()
    ws = torch.empty(B.moe_workspace_bytes(B.WS_ROUTER, B.MOE_BF16, T, 1, d, 0, E, 0), dtype=torch.uint8, device="cuda")
    finite = torch.isfinite(want)
    for accumulate in (False, True):
        dx = dx0.clone()
        B.moe_router_bwd(x, wr, dl, None, False, dx, accumulate, ws)
        got, ref = dx.double(), want + (dx0.double() if accumulate else 0.0)
        assert torch.equal(got.nan_to_num(7.0)[~finite], want.nan_to_num(7.0)[~finite])
        assert ((got - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5 * size)[finite].all()


def _dw_ranges(T, d, E):
    """(ranges, offset of their sums in the workspace): into how many ranges of tokens the stream over x (router_dw.hip) cuts the weight
    gradient of a shape, 0 where it goes to another kernel (rules of router.hip and router_dw.hip)."""
    up = lambda a, b: -(-a // b)  # noqa: E731
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    planes, sum_bytes, pieces, x = (1 if E % 64 == 0 else 3), 4 * d * E, up(T, 32), T * d
    tiles = up(d, 256) * up(E, 256)
    splits = min(range(1, min(32, up(T, 128)) + 1), key=lambda s: up(tiles * s, cus) * (up(up(T, s), 32) + 16))
    if planes == 3:
        splits = max(1, min(up(4 * cus, up(d, 64) * up(E, 64)), (64 << 20) // sum_bytes, up(T, 64), 64))
    operand = up(pieces * 64 * planes * E, 256) * 256
    room = (up(splits * sum_bytes, 256) * 256 - operand) // sum_bytes
    least = {32: 1 << 22, 64: 1 << 22, 96: 7 << 15, 128: (1 << 23) + 1, 160: 5 << 16, 192: 1 << 22, 256: 1 << 22}.get(E)
    if T < 32 or d % 64 or room < 1 or least is None or x < least or (E in (192, 256) and x > 1 << 26):
        return 0, 0
    ranges = min(cus // up(d, 128), pieces // {1: 12, 3: 8 if E == 32 else 4}[planes])
    if ranges > room and splits > {32: 14, 64: 2.75, 96: 9, 160: 6}.get(E, 2.25) * room:
        return 0, 0
    ranges = max(1, min(ranges, room))
    return up(pieces, up(pieces, ranges)), 256 + (up(2 * T * E, 256) * 256 if planes == 1 else 0) + operand


# router_dw.hip, one plane (E = 64, 128, 192, 256) and three (32, 96, 160): fewer pieces than the ring holds, a last piece that overlaps
# the one before it, one and several ranges, as many as there are CUs or as the room holds, a last block of 64 columns; and shapes it leaves
# to others (ranges = 0), of small x, without room, with few long ranges beside those of big tiles (28000, 512, 256).  Against float64; the results
# are rounded to bf16 (2**-8), bf16 dlogits first (then: against what the kernel is given), sums of up to T products in fp32 (1e-5 of
# the largest)
@pytest.mark.parametrize("T,d,E,ranges", [
    (65, 3584, 96, 1), (300, 768, 96, 2), (1000, 1088, 96, 8), (100, 3328, 160, 1), (777, 448, 160, 5), (4100, 1024, 32, 15), (700, 7168, 32, 2),
    (4097, 1088, 64, 10), (600, 7168, 64, 1), (2100, 4096, 128, 5), (9001, 1024, 128, 22), (4100, 1024, 192, 10), (9000, 512, 192, 22),
    (4097, 1088, 256, 10), (32, 64, 96, 0), (33, 192, 160, 0), (65600, 64, 32, 0), (21900, 192, 64, 0), (6600, 640, 128, 0), (28000, 512, 256, 0)])
def test_router_weight_gradient_stream(T, d, E, ranges):
    print(f"case router-dw-{T}-{d}-{E}", flush=True)
    n, at = _dw_ranges(T, d, E)
    assert n == ranges
    g = torch.Generator(device="cuda").manual_seed(T + d + E)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")  # noqa: E731
    x, wr, dl, dw0 = randn(T, d).bfloat16(), randn(d, E).bfloat16(), randn(T, E) * 0.1, randn(d, E).bfloat16()
    ws = torch.empty(B.moe_workspace_bytes(B.WS_ROUTER, B.MOE_BF16, T, 1, d, 0, E, 0), dtype=torch.uint8, device="cuda")
    ref = x.double().t() @ (dl.bfloat16() if E % 64 == 0 else dl).double()
    for accumulate in (False, True):
        dwr = dw0.clone()
        ws.fill_(0x7b)
        B.moe_router_bwd(x, wr, dl, dwr, accumulate, None, False, ws)
        want = ref + (dw0.double() if accumulate else 0.0)
        assert ((dwr.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5 * ref.abs().max()).all()
        words = ws.view(torch.int32)
        if n:       # as many sums as ranges, and nobody drew a ticket
            sums = words[at // 4:]
            assert not (sums[:n * d * E] == 0x7b7b7b7b).any() and (sums[n * d * E:] == 0x7b7b7b7b).all()
            assert E % 64 or not words[:16].any()
        elif d * T > 1 << 23:
            assert words[:16].any()


# the sums of the weight gradient before they are rounded to bf16: every token has a partner whose products are the same with the other
# sign, so what comes out is the error of the sums.  Of sqrt(T) and the operands' size other kernels with these shapes are off by
# 0.9, 1.3, 0.9 and 1.8e-7, one chain of matrix instructions per range by 2.4, 2.6, 1.5 and 2.6e-7, several added up by 0.9, 1.2, 0.9 and 1.5e-7
@pytest.mark.parametrize("T,d,E,bound", [(8192, 2048, 32, 1.3e-7), (16384, 4096, 128, 1.6e-7), (16384, 1024, 64, 1.2e-7), (16384, 4096, 192, 2e-7)])
def test_router_weight_gradient_sums(T, d, E, bound):
    print(f"case router-dw-sums-{T}-{d}-{E}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + d + E)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")  # noqa: E731
    order = torch.randperm(T, generator=g, device="cuda")
    x, dl, wr = randn(T // 2, d).bfloat16(), randn(T // 2, E), randn(d, E).bfloat16()
    x, dl = torch.cat([x, -x])[order].contiguous(), torch.cat([dl, dl])[order].contiguous()
    ws = torch.empty(B.moe_workspace_bytes(B.WS_ROUTER, B.MOE_BF16, T, 1, d, 0, E, 0), dtype=torch.uint8, device="cuda")
    dwr = torch.empty_like(wr)
    B.moe_router_bwd(x, wr, dl, dwr, False, None, False, ws)
    assert float(dwr.double().norm()) < bound * (T * dwr.numel()) ** 0.5


# Infinities and numbers that round up to them, where the weight gradient's terms and the overlap of its last piece multiply by zeros that
# stand for nothing: every output is what one product per token gives, in one plane (E = 64, 192) and three.  Finite outputs as above
@pytest.mark.parametrize("T,d,E", [(777, 448, 160), (1001, 320, 96), (4100, 1024, 32), (4100, 1088, 64), (4100, 1024, 192)])
def test_router_weight_gradient_of_infinities(T, d, E):
    print(f"case router-dw-inf-{T}-{d}-{E}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + d + E)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")  # noqa: E731
    x, wr, dl = randn(T, d).bfloat16(), randn(d, E).bfloat16(), randn(T, E)
    x[20] *= 2.0 ** -30
    dl[20, 2] = 3.4e38
    x[10, 9], x[T - T % 32 - 1, 7] = -float("inf"), float("inf")       # the second one in the last piece's overlap
    dl[5, 3], dl[T - 1, 30] = float("inf"), -float("inf")
    seen = dl.bfloat16().double() if E % 64 == 0 else dl.double()
    want, size = x.double().t() @ seen, x.double().abs().t() @ seen.abs()
    dwr = torch.zeros_like(wr)
    ws = torch.empty(B.moe_workspace_bytes(B.WS_ROUTER, B.MOE_BF16, T, 1, d, 0, E, 0), dtype=torch.uint8, device="cuda")
    B.moe_router_bwd(x, wr, dl, dwr, False, None, False, ws)
    got, finite = dwr.double(), torch.isfinite(want)
    assert torch.equal(got.nan_to_num(7.0)[~finite], want.nan_to_num(7.0)[~finite])
    assert ((got - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5 * size)[finite].all()


# dlogits down to the smallest numbers keep their bits in three terms: both gradients, with x and weights that bring the results back among
# bf16's normal numbers.  Bounds as above
@pytest.mark.parametrize("T,d,E", [(777, 448, 160), (1001, 320, 96), (4100, 1024, 32)])
@pytest.mark.parametrize("exponent", [-112, -130, -143])
def test_router_gradients_of_tiny_dlogits(T, d, E, exponent):
    print(f"case router-tiny-{T}-{d}-{E}-{exponent}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + d + E)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")  # noqa: E731
    x, wr = (randn(T, d) * 2.0 ** 40).bfloat16(), (randn(d, E) * 2.0 ** 40).bfloat16()
    dl = (randn(T, E).double() * 2.0 ** exponent).float()
    dwr, dx = torch.empty_like(wr), torch.empty_like(x)
    ws = torch.empty(B.moe_workspace_bytes(B.WS_ROUTER, B.MOE_BF16, T, 1, d, 0, E, 0), dtype=torch.uint8, device="cuda")
    B.moe_router_bwd(x, wr, dl, dwr, False, dx, False, ws)
    for got, a, b in ((dwr, x.t(), dl), (dx, dl, wr.t())):
        want, size = a.double() @ b.double(), a.double().abs() @ b.double().abs()
        assert ((got.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5 * size).all()


# a token's selection and the counts, with one, two and four blocks per CU (the lines lie at 64 and 256 tokens per CU)
@pytest.mark.parametrize("T", [16385, 65537])
def test_route_of_many_tokens_equals_the_route_of_a_few(T):
    print(f"case route-{T}", flush=True)
    E, k, e_lo, e_cnt = 64, 4, 8, 24
    logits = torch.randn((T, E), generator=torch.Generator(device="cuda").manual_seed(T), device="cuda")

    def route(lg):
        n = lg.shape[0]
        idx, w = torch.full((n, k), -7, dtype=torch.int32, device="cuda"), torch.full((n, k), -7.0, device="cuda")
        counts = torch.full((e_cnt,), -7, dtype=torch.int32, device="cuda")
        B.moe_route(lg, k, W.GATE_SOFTMAX_RENORM, e_lo, e_cnt, idx, w, counts)
        return idx, w, counts
    idx, w, counts = route(logits)
    for t0 in (0, 4096, T - 100):
        idx2, w2, _ = route(logits[t0:t0 + 100].contiguous())
        assert torch.equal(idx[t0:t0 + 100], idx2) and torch.equal(w[t0:t0 + 100], w2)
    assert torch.equal(counts.long(), torch.bincount(idx.flatten().long(), minlength=E)[e_lo:e_lo + e_cnt])


# the router term of dx of 8 or 16 experts: a block per token, then 8, 16 and 32 tokens per block; a token's sum is the same
@pytest.mark.parametrize("T,d,E", [(1025, 1024, 8), (1027, 520, 16), (8209, 1032, 8), (8197, 1024, 16), (65545, 1032, 8)])
def test_router_input_gradient_does_not_depend_on_the_batch(T, d, E):
    print(f"case router-dx-{T}-{d}-{E}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + d + E)
    wr = torch.randn((d, E), generator=g, device="cuda", dtype=torch.bfloat16)
    dl, dx = torch.randn((T, E), generator=g, device="cuda"), torch.randn((T, d), generator=g, device="cuda", dtype=torch.bfloat16)

    def backward(t0, t1):
        n, out = t1 - t0, dx[t0:t1].clone()
        ws = torch.empty(B.moe_workspace_bytes(B.WS_ROUTER, B.MOE_BF16, n, 1, d, 0, E, 0), dtype=torch.uint8, device="cuda")
        B.moe_router_bwd(dx[t0:t1].contiguous(), wr, dl[t0:t1].contiguous(), None, False, out, True, ws)
        return out
    whole = backward(0, T)
    for t0, t1 in ((0, 40), (T // 2, T // 2 + 40), (T - 40, T)):
        assert torch.equal(whole[t0:t1], backward(t0, t1))


# weight gradients whose heavy experts are cut along the rows, by one of several plans or not at all: one expert, a hot one among
# empty ones, more experts than a wavefront has lanes (only the heaviest 64 may be cut), as heavy as each other
@pytest.mark.parametrize("d,f,rows", [(128, 192, [9000]), (256, 192, [300, 0, 12000, 10]), (512, 64, [7] * 66 + [4000, 3000, 9000]),
                                      (64, 320, [2500, 2500, 2500]), (320, 256, [100] * 70)])
def test_weight_gradients_of_heavy_experts(d, f, rows):
    print(f"case heavy-{d}-{f}-{rows[:4]}", flush=True)
    e_cnt, R = len(rows), sum(rows)
    g = torch.Generator(device="cuda").manual_seed(d + f + R)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)  # noqa: E731
    xp, h1, h3, a, d_o = randn(R, d), randn(R, f), randn(R, f), randn(R, f), randn(R, d)
    w1, w3, w2 = randn(e_cnt, d, f) * d ** -0.5, randn(e_cnt, d, f) * d ** -0.5, randn(e_cnt, f, d) * f ** -0.5
    offsets = torch.tensor([0] + rows, device="cuda").cumsum(0).to(torch.int32)
    dxp = torch.empty_like(xp)
    dw1, dw3, dw2 = (torch.full_like(w, float("nan")) for w in (w1, w3, w2))
    ws = torch.empty(B.moe_workspace_bytes(B.WS_EXPERT_BWD, B.MOE_BF16, R, 1, d, f, e_cnt, R), dtype=torch.uint8, device="cuda")
    B.moe_expert_bwd(xp, h1, h3, d_o, offsets, w1, w3, w2, dxp, dw1, dw3, dw2, False, ws, a=a)
    for e in range(e_cnt):
        r = slice(sum(rows[:e]), sum(rows[:e + 1]))
        if rows[e] == 0:
            assert not dw1[e].any() and not dw3[e].any() and not dw2[e].any()
            continue
        x, p, q, s, do = (t[r].double() for t in (xp, h1, h3, a, d_o))
        sig = p.sigmoid()
        da = do @ w2[e].double().t()
        for got, ref in ((dw2[e], s.t() @ do), (dw1[e], x.t() @ (da * q * sig * (1 + p * (1 - sig)))), (dw3[e], x.t() @ (da * p * sig))):
            assert rel_err(host(got), host(ref)) < TOL["bf16"]


# as many experts as a wavefront has lanes, and more: lists of tiles and pieces are then made 64 experts at a time
@pytest.mark.parametrize("d,f,rows", [(192, 64, [5, 0, 3000, 1] + [2] * 60), (128, 64, [1, 0] * 34 + [2500, 3, 700])])
def test_weight_gradients_of_more_experts_than_lanes(d, f, rows):
    test_weight_gradients_of_heavy_experts(d, f, rows)


# logits of 8 to 56 experts: eight fp32 sums per output and wavefront, added in pairs.  A block of 256 threads that adds the same
# products in 256 chains and a tree is off by 6.2e-8 / 7.3e-8 / 8.3e-8 of the logits' norm, chains of matrix instructions by
# 7.1e-8 / 1.03e-7 / 1.8e-7; the bounds are halfway for the longer contractions, 5 % above the first for the shortest
@pytest.mark.parametrize("E", [8, 16, 24, 32, 40, 56])
@pytest.mark.parametrize("d,bound", [(512, 6.5e-8), (2048, 8.8e-8), (7168, 1.3e-7)])
def test_logits_of_few_experts(E, d, bound):
    print(f"case few-experts-{E}-{d}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(E + d)
    x = torch.randn((5000, d), generator=g, device="cuda", dtype=torch.bfloat16)
    wr = torch.randn((d, E), generator=g, device="cuda", dtype=torch.bfloat16).mul_(d ** -0.5)

    def logits(rows):
        out = torch.full((rows.shape[0], E), float("nan"), device="cuda")
        ws = torch.empty(B.moe_workspace_bytes(B.WS_ROUTER, B.MOE_BF16, rows.shape[0], 1, d, 0, E, 0), dtype=torch.uint8, device="cuda")
        B.moe_router_fwd(rows.contiguous(), wr, out, ws)
        return out
    whole, ref = logits(x), x.double() @ wr.double()
    assert float((whole.double() - ref).norm() / ref.norm()) < bound
    # a token's logits do not depend on the batch: blocks of 1, 2, 8, 16 and 32 rows
    for t0, t1 in ((0, 1), (17, 320), (1000, 2999)):
        assert torch.equal(logits(x[t0:t1]), whole[t0:t1])
    assert torch.equal(logits(torch.cat([x[100:], x])), torch.cat([whole[100:], whole]))


# logits of 64 experts and more: blocks of 16, 32 and 64 tokens by 64 and 128 experts, the contraction whole and cut; one piece per wavefront and
# less, pieces that are no multiple of the wavefronts.  Every output is the sum of eight chains of d / 256 matrix instructions, whose sums are not
# rounded to nearest, so a bound per d: 2 % above what these chains are off by in relation to the logits' norm (3.85 / 5.65 / 7.45 / 7.57 / 7.93 /
# 8.39 / 10.4 / 11.8 / 13.7 / 18.0e-8 at d = 64 / 192 / 576 / 640 / 832 / 1088 / 2112 / 2880 / 4096 / 7168).  One instruction more in a chain of
# three to five would be 5 % more.
@pytest.mark.parametrize("d,E,bound", [(64, 64, 3.93e-8), (192, 72, 5.8e-8), (576, 72, 7.6e-8), (640, 136, 7.73e-8), (832, 128, 8.1e-8), (1088, 256, 8.56e-8),
                                       (2112, 520, 1.06e-7), (2880, 128, 1.2e-7), (4096, 192, 1.4e-7), (7168, 256, 1.84e-7)])
def test_logits_of_many_experts(d, E, bound):
    print(f"case many-experts-{E}-{d}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(E + d)
    most = 9001 if E <= 128 or E % 64 else 8000    # (above, 256x256 tiles take over)
    x = torch.randn((most, d), generator=g, device="cuda", dtype=torch.bfloat16)
    wr = torch.randn((d, E), generator=g, device="cuda", dtype=torch.bfloat16).mul_(d ** -0.5)
    ref = x.double() @ wr.double()
    whole = None
    for T in (most, 7000, 4000, 2700, 1500, 300, 33, 15, 1):
        x[T:] = float("nan")
        out = torch.full((T + 64, E), float("nan"), device="cuda")
        ws = torch.empty(B.moe_workspace_bytes(B.WS_ROUTER, B.MOE_BF16, T, 1, d, 0, E, 0), dtype=torch.uint8, device="cuda")
        B.moe_router_fwd(x[:T], wr, out[:T], ws)
        assert out[T:].isnan().all()
        off = float((out[:T].double() - ref[:T]).norm() / ref[:T].norm())
        whole = out if whole is None else whole
        assert off < bound or T < 1500             # (few tokens scatter)
        # a token's logits do not depend on the batch where the contraction is not cut: too short, experts that fill no blocks of 64, many tokens
        if d < 1536 or E % 64 or T >= 1500:
            assert torch.equal(out[:T].view(torch.int32), whole[:T].view(torch.int32)), T


# a plan that does not fit its buffers, with the kernels for few rows: the rows that fit are those of the whole plan
def test_few_rows_with_more_rows_than_the_capacity():
    wl = W.QWEN.scaled(name="few-rows-overflow", T=40, d=128, f=192, E=8, e_cnt=8, k=4)
    print(f"case {wl.name}", flush=True)
    inp = make_inputs(wl)
    fw, _ = oracle_layer(wl, inp)
    cap, R = 101, int(fw["offsets"][-1])
    assert R > cap
    dev, buf = gpu_layer(wl, inp, cap=cap)
    assert buf.status() == 1
    assert (host(buf.offsets) == np.minimum(fw["offsets"], cap)).all()
    for name, got in (("h1", buf.h1), ("h3", buf.h3), ("o", buf.o)):
        assert got.shape[0] == cap and rel_err(host(got), fw[name][:cap]) < TOL["bf16"], name


# GEMMs all of 128x128 tiles and all of 256x256 ones (both kinds in one launch: the last test); one k-tile, an odd number of them,
# widths that are no multiples of either tile, 1 to 129 rows in the last row tile, empty experts
@pytest.mark.parametrize("d,f,rows", [(64, 192, [129, 0, 128, 1, 65]), (192, 64, [300, 257, 33]), (320, 448, [140] * 9),
                                      (512, 1472, [3000, 1700, 900, 130, 129, 128, 127, 1]), (1088, 512, [5000, 0, 1400, 290, 2])])
def test_bf16_gemms_that_end_in_quarter_tiles(d, f, rows):
    print(f"case quarters-{d}-{f}-{rows[:4]}", flush=True)
    e_cnt, R = len(rows), sum(rows)
    g = torch.Generator(device="cuda").manual_seed(d + f + R)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)  # noqa: E731
    cap = max(R, 129 * e_cnt)                      # above every bound of the kernel for few rows
    xp, d_o, w1, w3, w2 = randn(cap, d), randn(cap, d), randn(e_cnt, d, f) * d ** -0.5, randn(e_cnt, d, f) * d ** -0.5, randn(e_cnt, f, d) * f ** -0.5
    h1, h3, a, o, dxp = (torch.full((cap, n), float("nan"), device="cuda", dtype=torch.bfloat16) for n in (f, f, f, d, d))
    dw1, dw3, dw2 = (torch.full_like(w, float("nan")) for w in (w1, w3, w2))
    offsets = torch.tensor([0] + rows, device="cuda").cumsum(0).to(torch.int32)
    for keep_a in (a, None):                       # without the kept activation dA is a launch of its own
        wsf, wsb = (torch.empty(B.moe_workspace_bytes(which, B.MOE_BF16, R, 1, d, f, e_cnt, cap), dtype=torch.uint8, device="cuda")
                    for which in (B.WS_EXPERT_FWD, B.WS_EXPERT_BWD))
        B.moe_expert_fwd(xp, offsets, w1, w3, w2, h1, h3, o, wsf, a=keep_a)
        B.moe_expert_bwd(xp, h1, h3, d_o, offsets, w1, w3, w2, dxp, dw1, dw3, dw2, False, wsb, a=keep_a)
        off = np.array([0] + rows).cumsum()
        args = [host(t) for t in (w1, w3, w2)]
        rh1, rh3, _, ro = O.expert_fwd(host(xp[:R]), off, *args)
        rdxp, rdw1, rdw3, rdw2 = O.expert_bwd(host(xp[:R]), rh1, rh3, host(d_o[:R]), off, *args)
        for name, got, ref in (("h1", h1, rh1), ("h3", h3, rh3), ("o", o, ro), ("dxp", dxp, rdxp)):
            assert torch.isnan(got[R:]).all() and rel_err(host(got[:R]), ref) < TOL["bf16"], name
        for name, got, ref in (("dw1", dw1, rdw1), ("dw3", dw3, rdw3), ("dw2", dw2, rdw2)):
            for e in range(e_cnt):
                assert rel_err(host(got[e]), ref[e]) < TOL["bf16"], (name, e)
        for t in (h1, h3, o, dxp, dw1, dw3, dw2):
            t.fill_(float("nan"))


def bf16_pass(rows, weights, xp, d_o, cap):
    """Forward and backward of experts with these rows; outputs, and which tiles each ragged GEMM drew tickets for: (256x256, 128x128).
    The capacity keeps dX in a launch of its own, and so does the activation that is not kept with dA."""
    R, (e_cnt, d, f) = sum(rows), weights[0].shape
    empty = lambda n: torch.empty((cap, n), device="cuda", dtype=torch.bfloat16)  # noqa: E731
    x, dy, h1, h3, o, dxp = empty(d), empty(d), empty(f), empty(f), empty(d), empty(d)
    x[:R], dy[:R] = xp, d_o
    grads = [torch.empty_like(w) for w in weights]
    offsets = torch.tensor([0] + rows).cumsum(0).to(torch.int32).cuda()
    wsf, wsb = (torch.empty(B.moe_workspace_bytes(which, B.MOE_BF16, R, 1, d, f, e_cnt, cap), dtype=torch.uint8, device="cuda")
                for which in (B.WS_EXPERT_FWD, B.WS_EXPERT_BWD))
    B.moe_expert_fwd(x, offsets, *weights, h1, h3, o, wsf)
    B.moe_expert_bwd(x, h1, h3, dy, offsets, *weights, dxp, *grads, False, wsb)
    kinds = {}
    for ws, scratch, names in ((wsf, cap * f * 2, ("up", "down")), (wsb, 3 * cap * f * 2, ("da", "dx"))):
        first = (scratch + 255) // 256 * 256             # the ticket counters lie behind the scratch matrices, 16 words per GEMM
        for i, name in enumerate(names):
            words = ws[first + 64 * i:first + 64 * (i + 1)].view(torch.int32)
            kinds[name] = (bool(words[:8].any()), bool(words[8:].any()))
    return dict(h1=h1[:R], h3=h3[:R], o=o[:R], dxp=dxp[:R]), kinds


# 256x256 tiles and then 128x128 ones: of what whole rounds of 256 CUs leave, the list cut inside an expert; of the row tiles of which
# half is empty (third case, up); of both (fourth case, dA).  Alone an expert's rows go to other tiles, with the same bits.
@pytest.mark.parametrize("d,f,rows,both", [(2048, 1024, [5000, 3500, 1400, 290, 2], ("up", "dx")),
                                           (2048, 2048, [5000, 0, 3700, 290, 2], ("down", "da", "dx")),
                                           (2112, 1024, [20, 2916, 2204, 2716], ("up", "down", "dx")),
                                           (1664, 2176, [2048, 511, 356, 1024, 1556, 1024, 1436], ("up", "da"))])
def test_bf16_gemms_with_both_kinds_of_tiles(d, f, rows, both):
    print(f"case both-kinds-{d}-{f}", flush=True)
    e_cnt, R, cap = len(rows), sum(rows), 130000
    g = torch.Generator(device="cuda").manual_seed(d + f)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)  # noqa: E731
    xp, d_o = randn(R, d), randn(R, d)
    w1, w3, w2 = weights = [randn(e_cnt, d, f) * d ** -0.5, randn(e_cnt, d, f) * d ** -0.5, randn(e_cnt, f, d) * f ** -0.5]
    got, kinds = bf16_pass(rows, weights, xp, d_o, cap)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        for name in both:
            assert kinds[name] == (True, True), (name, kinds)
    off, other = [0] + list(np.cumsum(rows)), set()
    for e in range(e_cnt):
        if rows[e] == 0:
            continue
        part = slice(off[e], off[e + 1])
        x, dy, a1, a3, a2 = (t.float() for t in (xp[part], d_o[part], w1[e], w3[e], w2[e]))
        h1, h3 = x @ a1, x @ a3
        sig = torch.sigmoid(h1)
        dA = dy @ a2.T
        want = dict(h1=h1, h3=h3, o=(h1 * sig * h3) @ a2,
                    dxp=(dA * h3 * sig * (1 + h1 * (1 - sig))) @ a1.T + (dA * h1 * sig) @ a3.T)
        alone, kinds_alone = bf16_pass([rows[e]], [w[e:e + 1].contiguous() for w in weights], xp[part], d_o[part], cap)
        other |= {name for name in both if kinds_alone[name] != (True, True)}
        for name, ref in want.items():
            assert rel_err(host(got[name][part]), ref.cpu().numpy()) < TOL["bf16"], (name, e)
            assert torch.equal(got[name][part], alone[name]), (name, e)
    assert other == set(both)
