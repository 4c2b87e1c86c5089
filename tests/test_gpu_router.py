"""Parity of the router's linear map (logits = x W_r^T), its backward, and the layer closed from x, against the CPU
fp64 oracle, through the C ABI.

Bar: the logits and both router gradients are bf16 x bf16 products accumulated in fp32 (the upstream dlogits enters
as a bf16 head plus a bf16 remainder), so they are held to 2e-3 in the two-part criterion of test_gpu_parity.py
(per tensor relative to the largest reference value, per element relative to |ref| + quadrature magnitude); the
bf16 output dx and everything downstream of the expert path keep the 2e-2 bar.  The top-k choice is discrete: the
closed-layer test checks that the GPU's choice is a valid top-k of the reference logits within the logits' own error
and identical to the oracle's wherever the choice is forced, then evaluates the oracle for that choice.
"""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import moe_oracle as O
from test_gpu_parity import TOL, TOL_GATE, assert_close, dev, dev_bf16, f32w, ffn_on_device, host_f32, ws_for

pytestmark = pytest.mark.gpu

TOL_ROUTER = 2e-3


def router_case(T, d, E, seed):
    sh = W.MoEShape(T=T, d_model=d, d_ffn=64, E=E, k=1)
    xb = W.make_tokens(sh, seed)
    wrb = W.make_router_weight(sh, seed, std=0.05)
    dl = (np.random.default_rng([seed, 21]).standard_normal((T, E)) * 0.3).astype(np.float32)
    return sh, xb, wrb, dl


ROUTER_SHAPES = [
    # T, d, E: one tile, ragged token tail, E not a multiple of 4 / of 8, E over 128 (dx on the grouped GEMM kernel), many tiles
    (256, 512, 8), (777, 256, 60), (300, 128, 7), (1000, 192, 300), (4096, 1024, 128), (64, 64, 1), (2500, 2048, 16),
    # every expert-group count of the skinny dx kernel (32, 64, 128 padded experts) with ragged E, more columns than one
    # block's 1024, fewer tokens than one stage of 64
    (500, 320, 96), (130, 1280, 33), (40, 2112, 32),
    # the forward kernel for many experts and many tokens (both operands through LDS): 64- and 128-expert tiles, ragged
    # E (also not a multiple of 4), a ragged token tail, two expert tiles
    (8192, 256, 60), (8200, 128, 99), (8192, 192, 160),
    # the router of the two workloads bench.py times it on, at full size
    (4096, 4096, 8), (16384, 4096, 128),
]


@pytest.mark.parametrize("T,d,E", ROUTER_SHAPES)
def test_router_forward_and_backward(moe, T, d, E):
    sh, xb, wrb, dl = router_case(T, d, E, seed=T + E)
    s = moe.Shape.of(sh)
    ws = ws_for(moe, s)
    x, wr = dev_bf16(xb), dev_bf16(wrb)
    logits = torch.full((T, E), float("nan"), dtype=torch.float32, device="cuda")
    moe.moe_router_fwd(s, x, wr, logits, ws)
    xf, wf = W.bf16_bits_to_f32(xb), W.bf16_bits_to_f32(wrb)
    ref = O.router_logits(xf, wf)
    q_l, q_x, q_w = O.router_scales(xf, wf, dl)
    assert_close(logits.cpu().numpy(), ref, q_l, tol=TOL_ROUTER, what="logits")

    dxr = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    dwr = torch.full((E, d), float("nan"), dtype=torch.float32, device="cuda")
    moe.moe_router_bwd(s, x, wr, dev(dl), dxr, dwr, 0, ws)
    rdx, rdw = O.router_logits_bwd(xf, wf, dl)
    assert_close(host_f32(dxr), rdx, q_x, tol=TOL, what="dx_router")          # bf16 output
    assert_close(dwr.cpu().numpy(), rdw, q_w, tol=TOL_ROUTER, what="dw_router")
    # accumulate: a second call with half the upstream gradient adds half of the first result
    moe.moe_router_bwd(s, x, wr, dev(dl * np.float32(0.5)), dxr, dwr, 1, ws)
    assert_close(dwr.cpu().numpy(), 1.5 * rdw, 1.5 * q_w, tol=TOL_ROUTER, what="dw_router accumulated")
    assert_close(host_f32(dxr), 0.5 * rdx, 0.5 * q_x, tol=TOL, what="dx_router (never accumulated)")


# the one-launch backward and sizes just past it, and the edges of its pieces: tokens of 16 wavefronts times
# 16 in flight, 4 per dx wavefront, 128 and 512 columns; few tokens whose experts the forward spreads over blocks
@pytest.mark.parametrize("T,d,E", [(1, 64, 2), (255, 576, 8), (257, 128, 5), (1024, 64, 8), (1025, 64, 8), (512, 1088, 16),
                                   (513, 192, 13), (3, 640, 9), (16, 2048, 64), (17, 128, 100), (300, 64, 17)])
def test_router_few_tokens(moe, T, d, E):
    test_router_forward_and_backward(moe, T, d, E)


# dx of more than 128 experts: last row tiles of every class (64, 128, 192 and 256 rows), after whole ones and alone, over
# contractions of 3, 4 and 16 steps per pass, whole and ragged
@pytest.mark.parametrize("T,d,E", [(256 + 40, 320, 130), (512 + 100, 64, 200), (256 + 160, 576, 150), (40, 256, 1000), (100, 320, 256),
                                   (160, 128, 192), (256 + 193, 192, 1000), (129, 64, 129), (64, 64, 255)])
def test_router_many_experts_tile_heights(moe, T, d, E):
    test_router_forward_and_backward(moe, T, d, E)


# on which side of the one-launch backward's rule a size lies: up to 1024 tokens with 8 experts; with 16 up to 512, or 64 where
# the width is below 128 or above 8192
@pytest.mark.parametrize("T,d,E,one_launch", [(1024, 64, 8, True), (1025, 128, 8, False), (512, 128, 16, True), (513, 128, 9, False),
                                              (512, 64, 16, False), (65, 64, 9, False), (64, 64, 16, True), (64, 8256, 16, True),
                                              (65, 8256, 16, False), (1, 64, 17, False)])
def test_router_backward_launches(moe, T, d, E, one_launch):
    moe.profile_reset()
    moe.profile_enable(True)
    try:
        test_router_forward_and_backward(moe, T, d, E)
        labels = {label for label, _ in moe.profile_records()}
    finally:
        moe.profile_enable(False)
        moe.profile_reset()
    assert ("router_bwd" in labels, "router_prepare" in labels) == (one_launch, not one_launch)


def test_permute_bwd_add(moe):
    sh = W.MoEShape(T=300, d_model=256, d_ffn=64, E=8, k=3)
    inp = W.random_layer_inputs(sh, seed=3)
    s = moe.Shape.of(sh)
    idx, _, _ = O.route_topk(inp["logits"], sh.k, 0, True)
    _, _, ros, _ = O.permute_maps(idx, sh.E_total)
    rng = np.random.default_rng(8)
    dxp = W.f32_to_bf16_bits(rng.standard_normal((sh.N, sh.d_model)).astype(np.float32))
    add = W.f32_to_bf16_bits(rng.standard_normal((sh.T, sh.d_model)).astype(np.float32))
    dx = torch.empty(sh.T, sh.d_model, dtype=torch.bfloat16, device="cuda")
    moe.moe_permute_bwd_add(s, dev_bf16(dxp), dev(ros), dev_bf16(add), dx)
    ref = O.permute_bwd(W.bf16_bits_to_f32(dxp), ros, sh.K_slots) + W.bf16_bits_to_f32(add)
    # fp32 sum of K'+1 bf16 values, one bf16 rounding: half an ulp of the result plus the fp32 sum's own rounding
    assert np.all(np.abs(host_f32(dx) - ref) <= np.abs(ref) * 2.0 ** -8 + 1e-6)


@pytest.mark.parametrize("name", ["tiny", "finegrained", "imbalance"])
def test_closed_layer(moe, name):
    wl = W.WORKLOADS[name]
    wl = wl if name == "tiny" else W.scaled_down(wl)
    sh = wl.shape
    inp = W.make_layer_inputs(wl, seed=2)
    wrb = W.make_router_weight(sh, seed=2, std=0.05)
    s = moe.Shape.of(sh)
    buf = moe.MoeLayerBuffers(s)
    x, dout, wr = dev_bf16(inp["x"]), dev_bf16(inp["dout"]), dev_bf16(wrb)
    wg, wu, wd = dev_bf16(inp["w_gate"]), dev_bf16(inp["w_up"]), dev_bf16(inp["w_down"])
    moe.layer_forward(buf, x, wg, wu, wd, w_router=wr)
    moe.layer_backward(buf, dout, wg, wu, wd, x=x, w_router=wr)
    torch.cuda.synchronize()

    xf, wf, df = f32w(inp, "x"), W.bf16_bits_to_f32(wrb), f32w(inp, "dout")
    Wg, Wu, Wd = f32w(inp, "w_gate"), f32w(inp, "w_up"), f32w(inp, "w_down")
    lg64 = O.router_logits(xf, wf)
    q_l = O.router_scales(xf, wf, np.zeros_like(lg64))[0]
    assert_close(buf.logits.cpu().numpy(), lg64, q_l, tol=TOL_ROUTER, what="logits")
    # The top-k choice is piecewise constant in the logits, and the GPU takes it from its own fp32 logits.  Where
    # the k-th and (k+1)-th reference logits are closer than the logits' error, two choices are equally right; the
    # GPU's is checked to be a valid one (no unselected reference logit beats a selected one by more than the error
    # of the row's logits, listed by descending logit within that error), and everything continuous is then
    # evaluated by the oracle for THAT choice, for every token, with no condition on the checks that follow.
    got_lg = buf.logits.cpu().numpy().astype(np.float64)
    row_err = np.abs(got_lg - lg64).max(axis=1) + np.abs(lg64).max(axis=1) * 2.0 ** -23
    got_idx = buf.topk_idx.cpu().numpy()
    sel = got_idx[:, :sh.k].astype(np.int64)
    assert ((sel >= 0) & (sel < sh.E)).all()
    assert all(len(set(r)) == sh.k for r in sel.tolist())                      # distinct experts per token
    sel_lg = np.take_along_axis(lg64, sel, axis=1)
    unsel = lg64.copy()
    np.put_along_axis(unsel, sel, -np.inf, axis=1)
    assert (sel_lg.min(axis=1) >= unsel.max(axis=1) - 2 * row_err).all()       # a valid top-k of the reference logits
    assert (sel_lg[:, :-1] >= sel_lg[:, 1:] - 2 * row_err[:, None]).all()      # in descending order
    for j in range(sh.E_shared):
        assert (got_idx[:, sh.k + j] == sh.E + j).all()
    # most tokens are decided outright, and there the choice is the oracle's own
    ref_idx, _, _ = O.route_topk(lg64.astype(np.float32), sh.k, sh.E_shared, True)
    srt = np.sort(lg64, axis=1)[:, ::-1]
    margin = srt[:, sh.k - 1] - srt[:, sh.k] if sh.E > sh.k else np.full(sh.T, np.inf)
    decided = margin > 4 * row_err
    assert decided.mean() > 0.98
    assert all(set(got_idx[t, :sh.k]) == set(ref_idx[t, :sh.k]) for t in np.nonzero(decided)[0])
    cache = O.gate_of_selection(lg64, sel, sh.E_shared, True)
    assert np.array_equal(cache[0], got_idx)
    out_ref, _ = O.layer_forward(xf, cache[0], cache[1], Wg, Wu, Wd)

    g = O.closed_layer_backward(xf, wf, sh.k, Wg, Wu, Wd, df, cache, True)
    q = O.layer_scales_staged(xf, cache[0], cache[1], Wg, Wu, Wd, df, sh.E_total)
    _, q_xr, q_wr = O.router_scales(xf, wf, g["dlogits"])
    # a logit error e moves a gate weight by at most 2e of itself; the gate's own fp32 arithmetic adds 1e-5
    assert (np.abs(buf.topk_w.cpu().numpy() - cache[1]) <= (4 * row_err[:, None] + TOL_GATE) * cache[1]).all()
    assert_close(host_f32(buf.out), out_ref, q["out"], what="out")
    dl_scale = np.abs(g["dtopk_w"]).max()
    assert np.abs(buf.dlogits.cpu().numpy() - g["dlogits"]).max() <= TOL * dl_scale   # inherits dtopk_w's bf16 inputs
    assert_close(buf.dw_router.cpu().numpy(), g["dw_router"], q_wr + TOL * np.abs(g["dw_router"]).max(), tol=TOL, what="dw_router")
    assert_close(host_f32(buf.dx), g["dx_total"], np.sqrt(q["dx"] ** 2 + q_xr ** 2), what="dx (expert path + router)")
    assert_close(buf.dw_gate.cpu().numpy(), g["dw_gate"], q["dw_gate"], what="dw_gate")
    assert_close(buf.dw_up.cpu().numpy(), g["dw_up"], q["dw_up"], what="dw_up")
    assert_close(buf.dw_down.cpu().numpy(), g["dw_down"], q["dw_down"], what="dw_down")


# one launch: a group of 8, 16 and 32 lanes per token, whole and partial blocks of 16 tokens; two: experts spread over blocks, more than 32
# of them, blocks of 32 tokens
@pytest.mark.parametrize("T,d,E,k,Es,renorm,one_launch", [(1, 64, 1, 1, 0, 1, True), (37, 512, 8, 2, 0, 1, True), (48, 1088, 9, 3, 1, 0, True),
                                                          (1003, 192, 16, 16, 2, 1, True), (4097, 64, 17, 4, 0, 0, True), (4096, 64, 32, 8, 1, 1, True),
                                                          (4064, 64, 32, 2, 0, 1, False), (4096, 64, 33, 2, 0, 1, False), (8191, 64, 5, 2, 0, 1, True),
                                                          (8192, 64, 5, 2, 0, 1, False)])
def test_router_and_gating_in_one(moe, T, d, E, k, Es, renorm, one_launch):
    """What the two calls give, bit for bit."""
    s = moe.Shape(T, d, 64, E, k, Es, renorm)
    g = torch.Generator(device="cuda").manual_seed(T + E)
    x, w = (torch.randn(n, d, device="cuda", generator=g).to(torch.bfloat16) for n in (T, E))
    ws = torch.empty(max(moe.workspace_bytes(s), 256), dtype=torch.uint8, device="cuda")
    two, one = ([torch.full(sz, float("nan"), device="cuda") for sz in ((T, E), (T, s.K_slots), (T, E))] for _ in range(2))
    idx, idx1 = (torch.full((T, s.K_slots), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    moe.moe_router_fwd(s, x, w, two[0], ws)
    moe.moe_route_topk(s, two[0], idx, two[1], two[2])
    moe.profile_reset()
    moe.profile_enable(True)
    moe.moe_router_route_fwd(s, x, w, one[0], idx1, one[1], one[2], ws)
    torch.cuda.synchronize()
    labels = [label for label, _ in moe.profile_records()]
    moe.profile_enable(False)
    moe.profile_reset()
    assert labels == (["router_route_fwd"] if one_launch else ["router_fwd", "route_topk"])
    assert torch.equal(idx, idx1) and all(torch.equal(a, b) for a, b in zip(two, one))


# the router's blocks before dX on 64-row tiles and on those of 128 columns, and with dX in a launch of its own, for up to 8, 16 and several
# times 16 experts; too many tokens for the weight gradients beside them, too many experts
@pytest.mark.parametrize("d,f,counts,joined", [
    (512, 1024, [64] * 8, True), (64, 128, [5] * 15 + [0], True), (1088, 1984, [100] * 13, True), (2560, 1600, [500, 0, 700, 1], True),
    (4096, 8192, [2048, 2048], True), (1024, 1024, [4] * 17, True), (192, 320, [0, 7] * 50, True),
    (64, 64, [512] * 8, False), (128, 128, [2] * 129, False),
])
def test_router_backward_beside_the_weight_gradients(moe, d, f, counts, joined):
    """What the two calls give: the experts' results bit for bit, the router's against fp64 (dx is one rounding to bf16 of sums in fp32 or of
    operands of 16 bits, 2^-9 of each element; dW_r sums of T products in fp32 or of 16 bits, 2^-16 of the norm)."""
    s, x, dy, off, w, ws, _, sg, su = ffn_on_device(moe, d, f, counts)
    T, E = s.T, s.E
    g = torch.Generator(device="cuda").manual_seed(1)
    wr = (torch.randn(E, d, device="cuda", generator=g) * 0.05).to(torch.bfloat16)
    dl = torch.randn(T, E, device="cuda", generator=g) * 0.3
    want = torch.full_like(x, float("nan")), [torch.full(t.shape, float("nan"), device="cuda") for t in w]
    moe.moe_grouped_ffn_bwd(s, dy, x, off, *w, sg, su, want[0], *want[1], False, ws)
    start = torch.randn(E, d, device="cuda", generator=g)
    over = None
    for accumulate in (False, True):
        dx, dxr = torch.full_like(x, float("nan")), torch.full_like(x, float("nan"))
        dw = [torch.zeros(t.shape, device="cuda") if accumulate else torch.full(t.shape, float("nan"), device="cuda") for t in w]
        dwr = start.clone() if accumulate else torch.full((E, d), float("nan"), device="cuda")
        ws.fill_(255)
        moe.profile_reset()
        moe.profile_enable(True)
        moe.moe_grouped_ffn_router_bwd(s, dy, x, off, *w, sg, su, dx, *dw, x, wr, dl, dxr, dwr, accumulate, ws)
        torch.cuda.synchronize()
        labels = [label for label, _ in moe.profile_records()]
        moe.profile_enable(False)
        moe.profile_reset()
        assert any(label.startswith("router") for label in labels) == (not joined)
        assert torch.equal(dx.view(torch.int16), want[0].view(torch.int16)) and all(torch.equal(a, b) for a, b in zip(dw, want[1]))
        if accumulate:
            assert torch.equal(dwr, start + over)
        else:
            over = dwr.clone()
            ref = dl.double().T @ x.double()
            assert float((dwr.double() - ref).norm()) <= 2.0 ** -16 * float(ref.norm())
        ref = dl.double() @ wr.double()
        assert float((dxr.double() - ref).norm()) <= 2.0 ** -8 * float(ref.norm()) and bool(torch.isfinite(dxr.float()).all())


# tokens below, at and above the 16 partial sums and the 16 x 16 requested together, 1 .. 16 experts
@pytest.mark.parametrize("d,f,counts", [(512, 1024, [3, 0, 4]), (512, 2048, [127, 129] * 4), (128, 1024, [5] * 15 + [0]), (1088, 1984, [39] * 13),
                                        (2560, 1600, [16]), (192, 4096, [17] * 9)])
def test_router_backward_has_the_same_bits_in_either_launch(moe, d, f, counts):
    """dW_r of up to 16 experts is the same 16 sums over the tokens in the launch of its own and in that of the weight gradients."""
    s, x, dy, off, w, ws, _, sg, su = ffn_on_device(moe, d, f, counts)
    T, E = s.T, s.E
    g = torch.Generator(device="cuda").manual_seed(2)
    wr = (torch.randn(E, d, device="cuda", generator=g) * 0.05).to(torch.bfloat16)
    dl = torch.randn(T, E, device="cuda", generator=g) * 0.3
    start = torch.randn(E, d, device="cuda", generator=g)
    dx, dw = torch.empty_like(x), [torch.zeros(t.shape, device="cuda") for t in w]
    for accumulate in (False, True):
        got = []
        for joined in (False, True):
            dxr, dwr = torch.full_like(x, float("nan")), start.clone() if accumulate else torch.full_like(start, float("nan"))
            moe.profile_reset()
            moe.profile_enable(True)
            if joined:
                moe.moe_grouped_ffn_router_bwd(s, dy, x, off, *w, sg, su, dx, *dw, x, wr, dl, dxr, dwr, accumulate, ws)
            else:
                moe.moe_router_bwd(s, x, wr, dl, dxr, dwr, accumulate, ws)
            torch.cuda.synchronize()
            labels = [label for label, _ in moe.profile_records()]
            moe.profile_enable(False)
            moe.profile_reset()
            assert ("router_bwd" in labels) == (not joined)
            got.append((dxr.view(torch.int16), dwr.view(torch.int32)))
        assert all(torch.equal(a, b) for a, b in zip(*got))
