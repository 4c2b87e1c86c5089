"""Parity of the HIP path against the CPU fp64 oracle, element by element, through the C ABI.

Bar: routing indices, counts, offsets, both maps and the permuted rows are bit-exact.  Floating-point outputs
and gradients stay within max relative error 2e-2 (bf16 operands, fp32 accumulation, against fp64), read as
BOTH  max|got-ref| / max|ref| <= 2e-2  per tensor and, for every element,  |got-ref| <= 2e-2*(|ref| + q)  where
q is the quadrature magnitude of the terms of the contraction that forms the element (so an element whose
terms cancel is held to the size of its terms, and a dropped tile, row or k-tail cannot hide behind a norm).
The fp32 gate paths (topk_w, probs, dlogits) are held to 1e-5.
"""
import warnings

import numpy as np
import pytest
import torch

import workloads as W
from oracle import moe_oracle as O

pytestmark = pytest.mark.gpu

TOL = 2e-2
TOL_GATE = 1e-5


# ---------------------------------------------------------------------------------------------------------
# helpers
# ---------------------------------------------------------------------------------------------------------

def dev_bf16(bits: np.ndarray) -> torch.Tensor:
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).cuda().view(torch.bfloat16)


def host_bits(t: torch.Tensor) -> np.ndarray:
    return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


def host_f32(t: torch.Tensor) -> np.ndarray:
    if t.dtype == torch.bfloat16:
        return W.bf16_bits_to_f32(host_bits(t))
    return t.cpu().numpy()


def dev(a: np.ndarray) -> torch.Tensor:
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def assert_close(got, ref, scale, tol=TOL, what=""):
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    assert got.shape == ref.shape, (what, got.shape, ref.shape)
    assert np.all(np.isfinite(got)), what
    r = O.rel_to_max_error(got, ref)
    x = O.elementwise_excess(got, ref, scale, tol)
    # the other element-wise reading of the bound, |got-ref| <= tol*|ref| + tol*rms(ref): reported, not enforced (an
    # element of a heavy-tailed tensor whose terms are much larger than the tensor's rms may exceed it legitimately)
    if ref.size:
        rms = float(np.sqrt(np.mean(ref * ref)))
        x_rms = float((np.abs(got - ref) - tol * np.abs(ref) - tol * rms).max())
        if x_rms > 0.0:
            warnings.warn(f"{what}: rms-form element-wise bound exceeded by {x_rms:.3e} (rms(ref) = {rms:.3e})")
    assert r <= tol, f"{what}: max-relative error {r:.3e} > {tol}"
    assert x <= 0.0, f"{what}: element-wise bound exceeded by {x:.3e}"


def f32w(inp, key):
    return W.bf16_bits_to_f32(inp[key])


def ws_for(moe, shape):
    return torch.empty(max(moe.workspace_bytes(shape), 256), dtype=torch.uint8, device="cuda")


# ---------------------------------------------------------------------------------------------------------
# routing
# ---------------------------------------------------------------------------------------------------------

ROUTE_CASES = [
    # T, E, k, E_shared, renorm, kind
    (256, 8, 2, 0, 1, "normal"),
    (100, 8, 8, 0, 0, "normal"),
    (333, 16, 1, 0, 1, "ties"),
    (257, 32, 4, 1, 1, "normal"),
    (1000, 64, 6, 2, 1, "normal"),
    (1000, 64, 6, 2, 0, "ties"),
    (513, 128, 4, 0, 1, "dead"),
    (77, 160, 8, 0, 1, "normal"),
    (50, 384, 16, 3, 0, "ties"),
    (40, 1000, 70, 0, 1, "normal"),
    (1, 8, 2, 0, 1, "normal"),
    # a wavefront per token and two or four logits per lane: equal logits on different lanes and in different slots of a lane, also
    # where fewer than k experts are alive and equal -1e30 and one -inf are chosen among
    (200, 128, 8, 0, 1, "ties"),
    (200, 256, 8, 1, 0, "ties"),
    (60, 64, 60, 0, 0, "dead"),
    (60, 128, 120, 0, 1, "dead"),
    (60, 250, 240, 2, 0, "dead"),
]


def make_logits(T, E, kind, seed):
    rng = np.random.default_rng(seed)
    lg = rng.standard_normal((T, E)).astype(np.float32) * 2
    if kind == "ties":
        lg = np.round(lg * 2) / 2
    if kind == "dead":
        lg[:, rng.choice(E, E // 5, replace=False)] = -1e30
        lg[:, 3] = -np.inf
    return lg.astype(np.float32)


@pytest.mark.parametrize("T,E,k,Es,renorm,kind", ROUTE_CASES)
def test_route_topk_and_bwd(moe, T, E, k, Es, renorm, kind):
    s = moe.Shape(T, 64, 64, E, k, Es, renorm)
    lg = make_logits(T, E, kind, seed=T + E)
    idx_ref, w_ref, p_ref = O.route_topk(lg, k, Es, bool(renorm))
    d_lg = dev(lg)
    idx = torch.full((T, k + Es), -7, dtype=torch.int32, device="cuda")
    w = torch.zeros((T, k + Es), dtype=torch.float32, device="cuda")
    probs = torch.zeros((T, E), dtype=torch.float32, device="cuda")
    moe.moe_route_topk(s, d_lg, idx, w, probs)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), idx_ref)                      # bit-exact indices
    np.testing.assert_allclose(w.cpu().numpy(), w_ref, rtol=TOL_GATE, atol=1e-30)
    np.testing.assert_allclose(probs.cpu().numpy(), p_ref, rtol=TOL_GATE, atol=1e-30)
    # probs_save may be omitted
    idx2 = torch.zeros_like(idx)
    w2 = torch.zeros_like(w)
    moe.moe_route_topk(s, d_lg, idx2, w2, None)
    assert torch.equal(idx2, idx) and torch.equal(w2, w)
    # backward
    rng = np.random.default_rng(5)
    dw = rng.standard_normal((T, k + Es)).astype(np.float32)
    dl_ref = O.route_topk_bwd(dw, idx_ref, w.cpu().numpy(), probs.cpu().numpy(), k, bool(renorm))
    dl = torch.full((T, E), 99.0, dtype=torch.float32, device="cuda")
    moe.moe_route_topk_bwd(s, dev(dw), idx, w, probs, dl)
    torch.cuda.synchronize()
    # dlogits is a difference of products of w (<= 1) and dw, so fp32 rounding scales with max|dw| (k = 1 with
    # renorm has the exact result 0)
    scale = np.abs(dw).max()
    assert np.abs(dl.cpu().numpy() - dl_ref).max() <= TOL_GATE * scale


# ---------------------------------------------------------------------------------------------------------
# permutation and the streaming kernels
# ---------------------------------------------------------------------------------------------------------

PERM_CASES = [
    # T, d, E, k, E_shared, kind
    (256, 512, 8, 2, 0, "uniform"),
    (1500, 128, 5, 3, 0, "skewed"),          # N = 4500: several 1024-slot blocks and a ragged tail
    (1111, 192, 64, 6, 2, "uniform"),
    (4096, 64, 32, 1, 0, "skewed"),          # k = 1: an expert-parallel shard
    (3000, 64, 128, 4, 0, "dead"),
    (700, 64, 1000, 5, 24, "uniform"),       # E' = 1024, the ABI limit
    (1, 64, 8, 2, 0, "uniform"),
    (600, 64, 4, 4, 0, "uniform"),           # k = E
]


def make_topk_idx(T, E, k, Es, kind, seed):
    rng = np.random.default_rng(seed)
    if kind == "uniform":
        p = np.ones(E)
    elif kind == "skewed":
        p = 1.0 / np.arange(1, E + 1) ** 1.2
    else:
        p = np.ones(E)
        p[rng.choice(E, E // 5, replace=False)] = 0.0
        p[: max(E // 10, 1)] *= 30
    p = p / p.sum()
    idx = np.empty((T, k + Es), dtype=np.int32)
    for t in range(T):
        idx[t, :k] = rng.choice(E, size=k, replace=False, p=p)
    for j in range(Es):
        idx[:, k + j] = E + j
    return idx


@pytest.mark.parametrize("T,d,E,k,Es,kind", PERM_CASES)
def test_permute_maps_rows_and_streams(moe, T, d, E, k, Es, kind):
    s = moe.Shape(T, d, 64, E, k, Es, 1)
    Et, Kp, N = E + Es, k + Es, T * (k + Es)
    idx = make_topk_idx(T, E, k, Es, kind, seed=T)
    xb = W.make_tokens(W.MoEShape(T, d, 64, E, k, Es), seed=T)
    counts_ref, offsets_ref, ros_ref, sor_ref = O.permute_maps(idx, Et)
    ws = ws_for(moe, s)
    d_idx, d_x = dev(idx), dev_bf16(xb)
    outs = []
    for rep in range(2):            # twice: the result must not depend on scheduling
        counts = torch.full((Et,), -1, dtype=torch.int32, device="cuda")
        offsets = torch.full((Et + 1,), -1, dtype=torch.int32, device="cuda")
        ros = torch.full((N,), -1, dtype=torch.int32, device="cuda")
        sor = torch.full((N,), -1, dtype=torch.int32, device="cuda")
        xp = torch.zeros((N, d), dtype=torch.bfloat16, device="cuda")
        moe.moe_permute(s, d_x, d_idx, xp, counts, offsets, ros, sor, ws)
        torch.cuda.synchronize()
        outs.append((counts, offsets, ros, sor, xp))
    counts, offsets, ros, sor, xp = outs[0]
    assert np.array_equal(counts.cpu().numpy(), counts_ref)
    assert np.array_equal(offsets.cpu().numpy(), offsets_ref)
    assert np.array_equal(ros.cpu().numpy(), ros_ref)
    assert np.array_equal(sor.cpu().numpy(), sor_ref)
    assert np.array_equal(host_bits(xp), O.permute_rows(xb, sor_ref, Kp))
    for a, b in zip(outs[0], outs[1]):
        assert torch.equal(a, b)
    # maps only (x, x_perm both NULL)
    ros2 = torch.zeros_like(ros)
    sor2 = torch.zeros_like(sor)
    moe.moe_permute(s, None, d_idx, None, counts, offsets, ros2, sor2, ws)
    assert torch.equal(ros2, ros) and torch.equal(sor2, sor)

    # combine, combine_bwd, permute_bwd on random bf16 rows
    rng = np.random.default_rng(T + 1)
    yb = W.f32_to_bf16_bits(rng.standard_normal((N, d)).astype(np.float32))
    gb = W.f32_to_bf16_bits(rng.standard_normal((T, d)).astype(np.float32))
    wt = rng.random((T, Kp)).astype(np.float32)
    y64, g64 = W.bf16_bits_to_f32(yb), W.bf16_bits_to_f32(gb)
    d_y, d_g, d_w = dev_bf16(yb), dev_bf16(gb), dev(wt)
    out = torch.zeros((T, d), dtype=torch.bfloat16, device="cuda")
    moe.moe_unpermute_combine(s, d_y, ros, d_w, out)
    assert_close(host_f32(out), O.unpermute_combine(y64, ros_ref, wt),
                 O.unpermute_combine_scale(np.abs(y64), ros_ref, wt), what="combine")
    dy = torch.zeros((N, d), dtype=torch.bfloat16, device="cuda")
    dtw = torch.zeros((T, Kp), dtype=torch.float32, device="cuda")
    moe.moe_unpermute_combine_bwd(s, d_g, d_y, ros, d_w, dy, dtw)
    dy_ref, dtw_ref = O.unpermute_combine_bwd(g64, y64, ros_ref, wt)
    assert_close(host_f32(dy), dy_ref, 0.0, what="combine_bwd dy")
    q_dtw = np.sqrt(((g64.astype(np.float64)[:, None, :] * y64[ros_ref.reshape(T, Kp)]) ** 2).sum(axis=2))
    assert_close(dtw.cpu().numpy(), dtw_ref, q_dtw, tol=1e-4, what="combine_bwd dtopk_w")
    dx = torch.zeros((T, d), dtype=torch.bfloat16, device="cuda")
    moe.moe_permute_bwd(s, d_y, ros, dx)
    assert_close(host_f32(dx), O.permute_bwd(y64, ros_ref, Kp),
                 O.unpermute_combine_scale(np.abs(y64), ros_ref, np.ones((T, Kp))), what="permute_bwd")


# few slots: one, a sub-group of 64 and its neighbours, several sub-groups and slots per token (ranked by the scatter), and sizes past it
@pytest.mark.parametrize("T,E,k,Es", [(1, 1, 1, 0), (64, 3, 1, 0), (65, 7, 1, 0), (341, 9, 3, 0), (1025, 5, 1, 1), (4096, 256, 1, 0),
                                      (4096, 257, 1, 0), (4097, 4, 1, 0), (100, 1000, 2, 1)])
def test_permute_few_slots(moe, T, E, k, Es):
    test_permute_maps_rows_and_streams(moe, T, 64, E, k, Es, "skewed")


# the counting sort in two launches, where the scatter does not rank the slots itself (more than 128 experts, 8 slots per token or
# N K' = 16384): a slot, one sub-group of 64 and its neighbours, tokens whose slots cross sub-groups and blocks of 1024 slots, its limits
@pytest.mark.parametrize("T,E,k,Es", [(1, 129, 1, 0), (64, 129, 1, 0), (65, 130, 1, 0), (7, 20, 8, 1), (1023, 129, 1, 0), (1025, 129, 1, 0),
                                      (114, 9, 9, 0), (1024, 200, 2, 1), (455, 11, 9, 0), (512, 12, 8, 0)])
def test_permute_in_two_launches(moe, T, E, k, Es):
    moe.profile_reset()
    moe.profile_enable(True)
    try:
        test_permute_maps_rows_and_streams(moe, T, 64, E, k, Es, "skewed")
        labels = {label for label, _ in moe.profile_records()}
    finally:
        moe.profile_enable(False)
        moe.profile_reset()
    assert labels >= {"perm_rank_scan", "perm_scatter_gather"} and not labels & {"perm_rank", "perm_sort_scatter_gather"}


# on which side of the one-launch sort's rule a size lies: up to 3072 slots (4096 with at most 12 experts) and 64 x 256 table entries
@pytest.mark.parametrize("N,E,one_launch", [(1, 1000, True), (3072, 341, True), (3072, 342, False), (3073, 12, True), (3073, 13, False),
                                            (4096, 12, True), (4097, 12, False), (4096, 256, False), (1024, 1000, True)])
def test_permute_launches(moe, N, E, one_launch):
    moe.profile_reset()
    moe.profile_enable(True)
    try:
        test_permute_maps_rows_and_streams(moe, N, 64, E, 1, 0, "skewed")
        labels = {label for label, _ in moe.profile_records()}
    finally:
        moe.profile_enable(False)
        moe.profile_reset()
    assert ("perm_rank_scan" in labels, "perm_scan" in labels) == (one_launch, not one_launch)


# the sort inside the scatter: one slot, a group of 64 and 8 of them (and their neighbours), and both sides of its limits (4096 slots,
# 128 experts, 8 slots per token, N K' of 16384, wavefronts x N of 2^23 beyond 1536 slots)
@pytest.mark.parametrize("T,d,E,k,Es,one_launch", [(1, 64, 1, 1, 0, True), (64, 64, 128, 1, 0, True), (65, 64, 126, 1, 2, True), (171, 1024, 5, 3, 0, True),
                                                   (256, 2048, 127, 8, 0, True), (257, 64, 127, 8, 0, False), (1024, 64, 9, 4, 0, True),
                                                   (2896, 64, 3, 1, 0, True), (2897, 64, 3, 1, 0, False), (1536, 2048, 3, 1, 0, True),
                                                   (100, 64, 129, 1, 0, False), (100, 64, 64, 7, 2, False)])
def test_permute_ranked_by_the_scatter(moe, T, d, E, k, Es, one_launch):
    moe.profile_reset()
    moe.profile_enable(True)
    try:
        test_permute_maps_rows_and_streams(moe, T, d, E, k, Es, "skewed")
        labels = {label for label, _ in moe.profile_records()}
    finally:
        moe.profile_enable(False)
        moe.profile_reset()
    assert ("perm_sort_scatter_gather" in labels, "perm_scatter_gather" in labels) == (one_launch, not one_launch)


# the keys ranked in quarters by the wavefronts of a block (more than 512 slots): quarters of 128 + 1 and of whole groups of 64, blocks of 1, 2
# and 4 tokens of which the last is not full, one to eight slots per token, and the most slots where a row has parts
@pytest.mark.parametrize("T,d,E,k,Es,ranked", [(513, 2048, 5, 1, 0, True), (257, 1024, 7, 2, 0, True), (171, 64, 9, 3, 0, True), (256, 2048, 3, 2, 1, True),
                                               (4096, 2048, 128, 1, 0, True), (4096, 1024, 2, 1, 0, True), (512, 2048, 12, 8, 0, True),
                                               (585, 1024, 100, 7, 0, True), (1023, 512, 16, 4, 0, True), (683, 1088, 9, 5, 1, False)])
def test_permute_ranked_in_quarters(moe, T, d, E, k, Es, ranked):
    moe.profile_reset()
    moe.profile_enable(True)
    try:
        test_permute_maps_rows_and_streams(moe, T, d, E, k, Es, "skewed")
        labels = {label for label, _ in moe.profile_records()}
    finally:
        moe.profile_enable(False)
        moe.profile_reset()
    assert ("perm_sort_scatter_gather" in labels) == ranked   # (the maps alone, without rows, are a problem of one part)


def test_permute_is_deterministic_over_100_runs(moe):
    """The order of equal keys never depends on scheduling: 100 runs of one larger shape (64 rank blocks, 128
    experts of which a fifth are empty and a tenth are hot), every output bit for bit the first run's and the oracle's."""
    T, d, E, k = 16384, 256, 128, 4
    s = moe.Shape(T, d, 64, E, k, 0, 1)
    N = T * k
    rng = np.random.default_rng(77)
    p = np.ones(E)
    p[rng.choice(E, E // 5, replace=False)] = 0.0
    p[: E // 10] *= 30
    # top-k without replacement by the Gumbel trick (input recipe only)
    keys = np.log(np.maximum(p, 1e-300))[None, :] + rng.gumbel(size=(T, E))
    idx = np.argsort(-keys, axis=1)[:, :k].astype(np.int32)
    xb = W.make_tokens(W.MoEShape(T, d, 64, E, k, 0), seed=3)
    counts_ref, offsets_ref, ros_ref, sor_ref = O.permute_maps(idx, E)
    ws = ws_for(moe, s)
    d_idx, d_x = dev(idx), dev_bf16(xb)
    first = None
    for rep in range(100):
        counts = torch.full((E,), -1, dtype=torch.int32, device="cuda")
        offsets = torch.full((E + 1,), -1, dtype=torch.int32, device="cuda")
        ros = torch.full((N,), -1, dtype=torch.int32, device="cuda")
        sor = torch.full((N,), -1, dtype=torch.int32, device="cuda")
        xp = torch.zeros((N, d), dtype=torch.bfloat16, device="cuda")
        moe.moe_permute(s, d_x, d_idx, xp, counts, offsets, ros, sor, ws)
        cur = (counts, offsets, ros, sor, xp)
        if first is None:
            first = cur
            assert np.array_equal(counts.cpu().numpy(), counts_ref) and np.array_equal(offsets.cpu().numpy(), offsets_ref)
            assert np.array_equal(ros.cpu().numpy(), ros_ref) and np.array_equal(sor.cpu().numpy(), sor_ref)
            assert np.array_equal(host_bits(xp), O.permute_rows(xb, sor_ref, k))
        else:
            for a, b in zip(first, cur):
                assert torch.equal(a, b), rep


def test_permute_empty_batch(moe):
    s = moe.Shape(0, 64, 64, 8, 2, 0, 1)
    ws = ws_for(moe, s)
    counts = torch.full((8,), -1, dtype=torch.int32, device="cuda")
    offsets = torch.full((9,), -1, dtype=torch.int32, device="cuda")
    e_i = torch.zeros((16,), dtype=torch.int32, device="cuda")
    e_b = torch.zeros((16,), dtype=torch.bfloat16, device="cuda")
    moe.moe_permute(s, e_b, e_i, e_b, counts, offsets, e_i, e_i, ws)
    torch.cuda.synchronize()
    assert counts.cpu().tolist() == [0] * 8 and offsets.cpu().tolist() == [0] * 9


# ---------------------------------------------------------------------------------------------------------
# grouped FFN, stage by stage
# ---------------------------------------------------------------------------------------------------------

FFN_CASES = [
    # T, d, f, E, k, E_shared, dead experts
    (300, 192, 320, 5, 2, 0, 1),       # d, f multiples of 64 but not of 128: column masks; one empty expert
    (256, 512, 1024, 8, 2, 0, 0),      # the tiny workload's shape
    (700, 128, 256, 3, 1, 1, 0),       # ~230 rows per expert + a 700-row shared expert: several row tiles, ragged
    (90, 256, 128, 16, 2, 0, 5),       # experts with a handful of rows
    (600, 256, 2048, 2, 1, 0, 0),      # few tiles and a long K in Y = H W_down and dX (32 and 64 k-steps)
    (513, 64, 64, 1, 1, 0, 0),         # one expert, the smallest legal widths, a one-row third tile
    (40, 128, 192, 24, 1, 0, 20),      # most experts empty: zero-filled weight gradients, experts ordered by row count
]


def staged_inputs(T, d, f, E, k, Es, dead, seed=0):
    shape = W.MoEShape(T, d, f, E, k, Es)
    inp = W.random_layer_inputs(shape, seed=seed, dead_experts=dead)
    idx, w, probs = O.route_topk(inp["logits"], k, Es, True)
    counts, offsets, ros, sor = O.permute_maps(idx, E + Es)
    xp_bits = O.permute_rows(inp["x"], sor, k + Es)
    return shape, inp, idx, w, counts, offsets, ros, sor, xp_bits


@pytest.mark.parametrize("T,d,f,E,k,Es,dead", FFN_CASES)
def test_grouped_ffn_fwd_bwd(moe, T, d, f, E, k, Es, dead):
    shape, inp, idx, w, counts, offsets, ros, sor, xp_bits = staged_inputs(T, d, f, E, k, Es, dead)
    if dead:
        assert counts.min() == 0
    s = moe.Shape.of(shape)
    N, Et = s.N, s.E_total
    ws = ws_for(moe, s)
    d_xp, d_off = dev_bf16(xp_bits), dev(offsets)
    d_wg, d_wu, d_wd = dev_bf16(inp["w_gate"]), dev_bf16(inp["w_up"]), dev_bf16(inp["w_down"])
    y = torch.zeros((N, d), dtype=torch.bfloat16, device="cuda")
    sg = torch.zeros((N, f), dtype=torch.bfloat16, device="cuda")
    su = torch.zeros((N, f), dtype=torch.bfloat16, device="cuda")
    moe.moe_grouped_ffn_fwd(s, d_xp, d_off, d_wg, d_wu, d_wd, y, sg, su, ws)
    torch.cuda.synchronize()
    wg, wu, wd = f32w(inp, "w_gate"), f32w(inp, "w_up"), f32w(inp, "w_down")
    xp = W.bf16_bits_to_f32(xp_bits)
    Y, G, U = O.grouped_ffn_fwd(xp, offsets, wg, wu, wd)
    qY, qG, qU = O.grouped_ffn_fwd_scales(xp, offsets, wg, wu, wd)
    assert_close(host_f32(sg), G, qG, what="save_g")
    assert_close(host_f32(su), U, qU, what="save_u")
    assert_close(host_f32(y), Y, qY, what="y_perm")

    # backward with an upstream gradient of the combine's scale
    rng = np.random.default_rng(9)
    dy_bits = W.f32_to_bf16_bits((rng.standard_normal((N, d)) * rng.random((N, 1))).astype(np.float32))
    dyp = W.bf16_bits_to_f32(dy_bits)
    dX, dWg, dWu, dWd = O.grouped_ffn_bwd(dyp, xp, offsets, wg, wu, wd)
    dxp = torch.zeros((N, d), dtype=torch.bfloat16, device="cuda")
    gwg = torch.full((Et, d, f), 7.0, dtype=torch.float32, device="cuda")
    gwu = torch.full((Et, d, f), 7.0, dtype=torch.float32, device="cuda")
    gwd = torch.full((Et, f, d), 7.0, dtype=torch.float32, device="cuda")
    moe.moe_grouped_ffn_bwd(s, dev_bf16(dy_bits), d_xp, d_off, d_wg, d_wu, d_wd, sg, su, dxp, gwg, gwu, gwd, 0, ws)
    torch.cuda.synchronize()
    qX, qWg, qWu, qWd = O.grouped_ffn_bwd_scales(dyp, xp, offsets, wg, wu, wd)
    assert_close(host_f32(dxp), dX, qX, what="dx_perm")
    assert_close(gwg.cpu().numpy(), dWg, qWg, what="dw_gate")
    assert_close(gwu.cpu().numpy(), dWu, qWu, what="dw_up")
    assert_close(gwd.cpu().numpy(), dWd, qWd, what="dw_down")
    for e in np.nonzero(counts == 0)[0]:      # empty experts: exact zeros when overwriting
        assert not gwg[e].any() and not gwu[e].any() and not gwd[e].any()
    # accumulate = 1 adds to what is there (and leaves empty experts untouched)
    base = 0.25
    gwg.fill_(base); gwu.fill_(base); gwd.fill_(base)
    moe.moe_grouped_ffn_bwd(s, dev_bf16(dy_bits), d_xp, d_off, d_wg, d_wu, d_wd, sg, su, dxp, gwg, gwu, gwd, 1, ws)
    torch.cuda.synchronize()
    assert_close(gwg.cpu().numpy() - base, dWg, qWg + 1e-5, what="dw_gate accumulate")
    assert_close(gwd.cpu().numpy() - base, dWd, qWd + 1e-5, what="dw_down accumulate")
    for e in np.nonzero(counts == 0)[0]:
        assert torch.all(gwu[e] == base)


ALL_GEMMS = ("gate_up", "down", "dh", "dx")
HEIGHT_COUNTS = [1, 31, 33, 64, 65, 128, 129, 256, 257, 300, 320, 321, 0, 577, 512 + 65]
FEW_COUNTS = [33, 300, 65, 0, 130]
MANY_TILE_COUNTS = [1300, 70, 0, 1400, 1024 + 30]   # 5 row tiles with a tall last one, 6 with a short last one, 4 with a tall one


@pytest.mark.parametrize("d,f,counts", [(128, 256, HEIGHT_COUNTS), (256, 1088, HEIGHT_COUNTS), (3072, 256, HEIGHT_COUNTS),
                                        (128, 3136, HEIGHT_COUNTS), (3072, 1536, FEW_COUNTS),
                                        (256, 2304, MANY_TILE_COUNTS)])
def test_grouped_ffn_every_tile_height(moe, d, f, counts):
    """Experts whose row counts fall into the height classes of a row tile: 1..64 rows (two 16-row blocks per wavefront), 65..128
    (four), 129..192 (six), 193..256 (eight), 257..288 and 289..320 (nine and ten: a full tile that carries up to 64 more
    rows), 321 (a full tile plus a short one), an empty expert, and a multi-tile expert whose remainder rides on its last tile.
    (f = 1088 = 4 * 256 + 64 also puts a 64-wide last column tile on every class.)  These shapes are small enough for most of
    their GEMMs to run on the 64-row tiles; test_grouped_ffn_on_256_row_tiles has the same counts on the others, and
    test_row_tile_classes both sides of every class boundary.

    The workspace holds NaN and -1 before either call: neither reads what it has not written (the schedule, the order of the
    experts, the zero page)."""
    counts = np.array(counts, dtype=np.int64)
    E, N = counts.size, int(counts.sum())
    offsets = np.zeros(E + 1, dtype=np.int32)
    offsets[1:] = np.cumsum(counts)
    shape = W.MoEShape(N, d, f, E, 1)        # (T = N rows with one slot each: only the sizes matter here)
    s = moe.Shape.of(shape)
    rng = np.random.default_rng(d + f)
    xp_bits = W.f32_to_bf16_bits(rng.standard_normal((N, d)).astype(np.float32))
    dy_bits = W.f32_to_bf16_bits((rng.standard_normal((N, d)) * rng.random((N, 1))).astype(np.float32))
    wgb, wub, wdb = W.make_expert_weights(shape, seed=1, std=0.05)
    ws = ws_for(moe, s)
    d_xp, d_off = dev_bf16(xp_bits), dev(offsets)
    d_wg, d_wu, d_wd = dev_bf16(wgb), dev_bf16(wub), dev_bf16(wdb)
    y = torch.full((N, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    sg = torch.full((N, f), float("nan"), dtype=torch.bfloat16, device="cuda")
    su = torch.full((N, f), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws.fill_(255)
    moe.moe_grouped_ffn_fwd(s, d_xp, d_off, d_wg, d_wu, d_wd, y, sg, su, ws)
    xp, dyp = W.bf16_bits_to_f32(xp_bits), W.bf16_bits_to_f32(dy_bits)
    wg, wu, wd = W.bf16_bits_to_f32(wgb), W.bf16_bits_to_f32(wub), W.bf16_bits_to_f32(wdb)
    Y, G, U = O.grouped_ffn_fwd(xp, offsets, wg, wu, wd)
    qY, qG, qU = O.grouped_ffn_fwd_scales(xp, offsets, wg, wu, wd)
    assert_close(host_f32(sg), G, qG, what="save_g")
    assert_close(host_f32(su), U, qU, what="save_u")
    assert_close(host_f32(y), Y, qY, what="y_perm")
    dxp = torch.full((N, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    gwg = torch.full((E, d, f), 7.0, dtype=torch.float32, device="cuda")
    gwu = torch.full((E, d, f), 7.0, dtype=torch.float32, device="cuda")
    gwd = torch.full((E, f, d), 7.0, dtype=torch.float32, device="cuda")
    ws.fill_(255)
    moe.moe_grouped_ffn_bwd(s, dev_bf16(dy_bits), d_xp, d_off, d_wg, d_wu, d_wd, sg, su, dxp, gwg, gwu, gwd, 0, ws)
    dX, dWg, dWu, dWd = O.grouped_ffn_bwd(dyp, xp, offsets, wg, wu, wd)
    qX, qWg, qWu, qWd = O.grouped_ffn_bwd_scales(dyp, xp, offsets, wg, wu, wd)
    assert_close(host_f32(dxp), dX, qX, what="dx_perm")
    assert_close(gwg.cpu().numpy(), dWg, qWg, what="dw_gate")
    assert_close(gwu.cpu().numpy(), dWu, qWu, what="dw_up")
    assert_close(gwd.cpu().numpy(), dWd, qWd, what="dw_down")
    empty = int(np.nonzero(counts == 0)[0][0])
    assert not gwg[empty].any() and not gwd[empty].any()    # the empty expert


# (the pair's bands of 4 or 8 of the 128-row tiles along d: whole ones, last ones of 1, 5 and 2 tiles)
@pytest.mark.parametrize("d,f,counts", [(640, 192, [300, 200, 0]), (1536, 64, [300, 200, 0]), (1600, 64, [300, 200, 0]),
                                        (1280, 64, [1700, 1601, 0])])
def test_weight_gradient_bands(moe, d, f, counts):
    test_grouped_ffn_every_tile_height(moe, d, f, counts)


@pytest.mark.parametrize("d,f", [(64, 64), (192, 320), (448, 128)])
def test_weight_gradient_edges(moe, d, f):
    """Row counts around the weight gradients' 32-row steps and their ring of three (0, 1, 2, 3, 4 steps, whole and
    ragged), widths that leave half of a 128-row or 128-column piece of a tile empty."""
    test_grouped_ffn_every_tile_height(moe, d, f, [1, 31, 32, 33, 64, 65, 0, 96, 97, 128, 129])


@pytest.mark.parametrize("d,f", [(320, 576), (1152, 192)])
def test_weight_gradient_begins(moe, d, f):
    """The tiles of a chunk begin at different steps of the contraction and go round, with the addresses of the next step's loads
    carried along: row counts on either side of the step counts where the rule changes (4, 8, 24 steps of 32), whole and ragged, so
    that the short last step comes first, last and in between."""
    test_grouped_ffn_every_tile_height(moe, d, f, [96, 97, 128, 161, 0, 224, 225, 256, 257, 300, 768, 769, 801])


def assert_runs_on(moe, d, f, counts, small, mid):
    """Exactly these GEMMs run on 64-row tiles and on tiles of 128 columns; all others on 256-row tiles."""
    s = moe.Shape(sum(counts), d, f, len(counts), 1)
    assert (moe.grouped_ffn_small_tiles(s), moe.grouped_ffn_mid_tiles(s)) == (small, mid)


# (d, f, counts, GEMMs on 64-row tiles, those on tiles of 128 columns)
@pytest.mark.parametrize("d,f,counts,small,mid", [
    (64, 64, [1, 32, 33, 0], ALL_GEMMS, ()),                     # one k-step: three of four, seven of eight wavefronts have none
    (192, 576, [64, 65, 31, 0, 128], ("down", "dh", "dx"), ("gate_up",)),   # 3 and 9 k-steps: unequal shares; tiles of one and two 32-row blocks
    (1088, 128, [200, 0, 7], ALL_GEMMS, ()),                     # 17 k-steps of dH and gate | up, 2 of down, 4 of dX
    (64, 64, [4500, 0, 257, 7], ("down", "dh", "dx"), ("gate_up",)),
    # an expert of more tiles (71) than a wavefront has lanes, one of 5: the schedule's writers
    (64, 64, [4500, 0, 257, 7] + 126 * [1], ALL_GEMMS, ()),
    # tiles found without a schedule: experts on either side of a wavefront's 64 lanes, 128 of them, the first and last ones empty
    # or not; and one and two experts too many for that
    (64, 128, [0, 65] + 61 * [3] + [130, 70, 0, 5], ("down", "dh", "dx"), ("gate_up",)),
    (64, 64, [0] + 62 * [1] + [0, 0] + 62 * [2] + [129], ("down", "dh"), ("gate_up", "dx")),
    (64, 64, 64 * [0] + [3] + 63 * [0], ALL_GEMMS, ()),
    (64, 64, 128 * [2] + [0], ALL_GEMMS, ()),
    (64, 64, 129 * [2] + [0], ALL_GEMMS, ()),
    # few row tiles of many columns, next to a dX of 212 .. 520 k-steps
    (128, 64 * 106, [1, 40, 63, 0, 64, 65, 100], ("down",), ("gate_up", "dh")),
    (128, 64 * 160, [1, 40, 63, 0, 64, 65, 100], (), ("gate_up", "dh")),
    (64, 64 * 260, [1, 40, 63, 0, 64, 65, 100], (), ("gate_up", "dh")),
])
def test_small_problem_tiles(moe, d, f, counts, small, mid):
    """The kernels for small problems, alone, together and next to the large one's in a call (two schedules), and both sides of the rules that
    choose them for each GEMM.  Only a call without a GEMM on 256-row tiles, with at most 128 experts, launches no schedule."""
    assert_runs_on(moe, d, f, counts, small, mid)
    moe.profile_reset()
    moe.profile_enable(True)
    try:
        test_grouped_ffn_every_tile_height(moe, d, f, counts)
        labels = [label for label, _ in moe.profile_records()]
    finally:
        moe.profile_enable(False)
        moe.profile_reset()
    calls = ("gate_up", "down"), ("dh", "dx")
    assert labels.count("ffn_schedule") == sum(len(counts) > 128 or not set(call) <= set(small + mid) for call in calls)


@pytest.mark.parametrize("d,f,counts,small,mid", [
    # every height class in all four GEMMs; column tiles of 64 (f) and 128 (d) at the end (more than 128 experts: none on tiles of 128 columns)
    (384, 320, 9 * HEIGHT_COUNTS, (), ()),
    # gate | up of experts of more than four row tiles, which the kernel walks column tile by column tile with a tall tile first, next to
    # one of four, walked in bands of 8 column tiles: 18 column tiles, i.e. two full bands and one of two
    (1408, 2304, MANY_TILE_COUNTS, (), ("down", "dh", "dx")),
    # few tiles and 48 k-steps or more: cut along k.  dH of 128 steps in up to 8 parts, a tall tile, a short one and one of 65
    # rows among them, whose last part to arrive applies the d(SwiGLU) epilogue to the sums ...
    (8192, 128, [300, 33, 0, 0, 65], ("gate_up",), ("down", "dx")),
    # ... down and dX, of 128 and 256 steps ...
    (128, 8192, [300, 33, 0, 0, 0, 0, 65], (), ("gate_up", "dh")),
    # ... and dH of 64 steps.  (dH and dX in one backward call, on the same arrival counters: test_dh_and_dx_cut_along_k)
    (4096, 2048, [12, 0, 31], ("gate_up", "down"), ("dx",)),
])
def test_grouped_ffn_on_256_row_tiles(moe, d, f, counts, small, mid):
    """The kernel of large problems at whole-tensor precision."""
    assert_runs_on(moe, d, f, counts, small, mid)
    test_grouped_ffn_every_tile_height(moe, d, f, counts)


# rows on either side of every class boundary (64, 128, 192, 256, 288, 320), inside the classes, and experts of two and three tiles
# whose last ones are of the classes of 320 and 192 rows
CLASS_COUNTS = [64, 65, 128, 129, 161, 192, 193, 256, 257, 272, 288, 289, 320, 0, 512 + 33, 512 + 160, 321, 100, 224]


@pytest.mark.parametrize("d,f,counts,small,mid", [
    # (more than 128 experts: none on tiles of 128 columns)
    (64, 256, 7 * CLASS_COUNTS, ("down", "dx"), ()),          # gate | up and dH of 1 step: fewer than the stages of any class
    (192, 256, 7 * CLASS_COUNTS, (), ()),                     # of 3 steps, down of 4, dX of 8
    (256, 64, 7 * CLASS_COUNTS, ("gate_up", "dh"), ()),       # down of 1 step, dX of 2
    (1088, 1600, 4 * CLASS_COUNTS, (), ("dh", "dx")),         # gate | up and down: 17 and 25 steps
    # the same rows on tiles of 128 columns
    (64, 4096, CLASS_COUNTS, ("down", "dx"), ("gate_up", "dh")),
    (192, 4096, CLASS_COUNTS, ("down", "dx"), ("gate_up", "dh")),
    (4096, 128, CLASS_COUNTS, ("gate_up", "dh"), ("down", "dx")),
])
def test_row_tile_classes(moe, d, f, counts, small, mid):
    test_grouped_ffn_on_256_row_tiles(moe, d, f, counts, small, mid)


# left-over tiles in pieces of whole 64 rows: gate | up in 2; (gate | up, down, dH, dX) in 5, 4, 5 and 4, more
# than some of the tiles have rows for; tall tiles, all four in 2 (more than 128 experts: none on tiles of 128 columns)
@pytest.mark.parametrize("d,f,counts,mid", [(1088, 1600, 3 * CLASS_COUNTS, ("down", "dh", "dx")), (448, 1216, 7 * CLASS_COUNTS, ()),
                                            (256, 256, 122 * [320] + [289, 0, 257, 200, 0, 0, 0], ())])
def test_row_tiles_cut_along_rows(moe, d, f, counts, mid):
    test_grouped_ffn_on_256_row_tiles(moe, d, f, counts, (), mid)


def ffn_on_device(moe, d, f, counts, seed=0):
    """Inputs and one saving forward of the grouped FFN over experts of `counts` rows, all on the device."""
    E, N = len(counts), sum(counts)
    s = moe.Shape(N, d, f, E, 1)
    g = torch.Generator(device="cuda").manual_seed(seed)
    normal = lambda *sz, std=1.0: (torch.randn(*sz, device="cuda", generator=g) * std).to(torch.bfloat16)  # noqa: E731
    e = lambda *sz: torch.full(sz, float("nan"), dtype=torch.bfloat16, device="cuda")  # noqa: E731
    off = dev(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32))
    x, dy = normal(N, d), normal(N, d)
    w = [normal(E, d, f, std=0.05), normal(E, d, f, std=0.05), normal(E, f, d, std=0.05)]
    ws, y, sg, su = ws_for(moe, s), e(N, d), e(N, f), e(N, f)
    moe.moe_grouped_ffn_fwd(s, x, off, *w, y, sg, su, ws)
    return s, x, dy, off, w, ws, y, sg, su


EDGE_COUNTS = [1, 31, 32, 33, 64, 65, 0, 96, 97, 128, 129]


@pytest.mark.parametrize("d,f,counts", [(64, 64, EDGE_COUNTS), (192, 320, EDGE_COUNTS), (448, 128, EDGE_COUNTS), (640, 1088, [300, 0, 577]),
                                        (2304, 2304, [30, 0, 7, 64])])
def test_weight_gradients_accumulate(moe, d, f, counts):
    """accumulate = 1: every element of the three gradients is the fp32 sum of its start value and what the overwriting call
    writes there, bit for bit, saved and recomputing call alike; an expert without rows keeps its start values."""
    s, x, dy, off, w, ws, y, sg, su = ffn_on_device(moe, d, f, counts)
    dx = torch.empty_like(x)
    over = [torch.full(t.shape, float("nan"), device="cuda") for t in w]
    moe.moe_grouped_ffn_bwd(s, dy, x, off, *w, sg, su, dx, *over, 0, ws)
    start = [torch.randn(t.shape, device="cuda") for t in w]
    for recompute in (False, True):
        got, dx2 = [t.clone() for t in start], torch.empty_like(dx)
        if recompute:
            moe.moe_grouped_ffn_bwd_recompute(s, dy, x, off, *w, dx2, *got, 1, ws)
        else:
            moe.moe_grouped_ffn_bwd(s, dy, x, off, *w, sg, su, dx2, *got, 1, ws)
        assert torch.equal(dx2.view(torch.int16), dx.view(torch.int16))
        for name, a, b, c in zip(("dw_gate", "dw_up", "dw_down"), got, start, over):
            assert bool(torch.isfinite(c).all()) and torch.equal(a, b + c), (name, recompute)


@pytest.mark.parametrize("d,f,counts,small,mid", [
    (2560, 1600, CLASS_COUNTS + 8 * [2000], (), ()),              # all on 256-row tiles
    (640, 1088, HEIGHT_COUNTS + [1500, 2000, 1800], (), ALL_GEMMS),   # all on tiles of 128 columns
    (256, 192, [248] * 64 + [2048, 2048], (), ALL_GEMMS),
    (256, 192, [248] * 64 + [2048, 2048] + 63 * [0], ("dh",), ()),   # 256-row forward, dH on 64-row tiles, dX on 256-row tiles
    (4096, 1088, [3, 0, 31, 9, 1, 0, 12, 30, 2, 2, 0, 5, 1, 1, 1, 2, 4], (), ("down", "dx")),   # few rows; dH cut along k
    (8192, 128, [300, 33, 0, 0, 65], ("gate_up",), ("down", "dx")),  # dH, cut along k, on 256-row tiles
    (4096, 6400, [9, 20], ("gate_up", "down"), ()),               # dH and dX cut along k
    (512, 1024, [64] * 8, ("down", "dh", "dx"), ("gate_up",)),
    (512, 192, [16] * 8, ALL_GEMMS, ()),
])
def test_recomputing_backward_on_either_kernel(moe, d, f, counts, small, mid):
    """The recomputing backward gives the saving pair's bits whichever kernels its GEMMs run on (G and U, recomputed into the
    memory of dG and dU, are read and overwritten in place)."""
    assert_runs_on(moe, d, f, counts, small, mid)
    s, x, dy, off, w, ws, y, sg, su = ffn_on_device(moe, d, f, counts)
    y2 = torch.full_like(y, float("nan"))
    moe.moe_grouped_ffn_fwd(s, x, off, *w, y2, None, None, ws)
    outs = [y.view(torch.int16)], [y2.view(torch.int16)]
    for recompute, out in enumerate(outs):
        dx, dws = torch.full_like(x, float("nan")), [torch.full(t.shape, float("nan"), device="cuda") for t in w]
        if recompute:
            moe.moe_grouped_ffn_bwd_recompute(s, dy, x, off, *w, dx, *dws, 0, ws)
        else:
            moe.moe_grouped_ffn_bwd(s, dy, x, off, *w, sg, su, dx, *dws, 0, ws)
        assert bool(torch.isfinite(dx).all()) and all(bool(torch.isfinite(t).all()) for t in dws)
        out += [dx.view(torch.int16)] + [t.view(torch.int32) for t in dws]
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("d,f,counts,schedules", [
    (832, 1856, [372, 0, 744] + 5 * [372], 1),       # gate | up on 256-row tiles, dH and dX on those of 128 columns
    (64, 3072, 15 * [300, 384], 1),                  # ... dX on 64-row tiles
    (4160, 1600, [13], 1),                           # dH on 256-row tiles, gate | up and dX on 64-row tiles
    (320, 64, 9 * [178, 100], 0),                    # none on 256-row tiles
])
def test_one_schedule_of_a_recomputing_backward(moe, d, f, counts, schedules):
    """All GEMMs of a recomputing backward share a schedule, and give the saving pair's bits."""
    s, x, dy, off, w, ws, y, sg, su = ffn_on_device(moe, d, f, counts)
    outs = []
    for recompute in (False, True):
        ws.zero_()
        dx, dws = torch.full_like(x, float("nan")), [torch.full(t.shape, float("nan"), device="cuda") for t in w]
        moe.profile_reset()
        moe.profile_enable(True)
        try:
            if recompute:
                moe.moe_grouped_ffn_bwd_recompute(s, dy, x, off, *w, dx, *dws, 0, ws)
            else:
                moe.moe_grouped_ffn_bwd(s, dy, x, off, *w, sg, su, dx, *dws, 0, ws)
            labels = [label for label, _ in moe.profile_records()]
        finally:
            moe.profile_enable(False)
            moe.profile_reset()
        outs.append([dx.view(torch.int16)] + [t.view(torch.int32) for t in dws])
    assert labels.count("ffn_schedule") == schedules
    for a, b in zip(*outs):
        assert torch.equal(a, b)


# ---------------------------------------------------------------------------------------------------------
# the whole layer, forward + backward, against the per-token definition
# ---------------------------------------------------------------------------------------------------------

def run_layer(moe, inp, renorm=1):
    sh = inp["shape"]
    s = moe.Shape(sh.T, sh.d_model, sh.d_ffn, sh.E, sh.k, sh.E_shared, renorm)
    buf = moe.MoeLayerBuffers(s)
    x, dout = dev_bf16(inp["x"]), dev_bf16(inp["dout"])
    wg, wu, wd = dev_bf16(inp["w_gate"]), dev_bf16(inp["w_up"]), dev_bf16(inp["w_down"])
    if "logits" in inp:
        logits = dev(inp["logits"])
    else:
        logits = None
        buf.topk_idx.copy_(dev(inp["topk_idx"]))
        buf.topk_w.copy_(dev(inp["topk_w"]))
    moe.layer_forward(buf, x, wg, wu, wd, logits)
    moe.layer_backward(buf, dout, wg, wu, wd, accumulate=False, with_router=logits is not None)
    torch.cuda.synchronize()
    return s, buf


def check_layer_against_definition(moe, inp, renorm=1):
    sh = inp["shape"]
    s, buf = run_layer(moe, inp, renorm)
    if "logits" in inp:
        idx, w, probs = O.route_topk(inp["logits"], sh.k, sh.E_shared, bool(renorm))
        assert np.array_equal(buf.topk_idx.cpu().numpy(), idx)
        np.testing.assert_allclose(buf.topk_w.cpu().numpy(), w, rtol=TOL_GATE)
    else:
        idx, w, probs = inp["topk_idx"], inp["topk_w"].astype(np.float64), None
    counts, offsets, ros, sor = O.permute_maps(idx, sh.E_total)
    assert np.array_equal(buf.counts.cpu().numpy(), counts)
    assert np.array_equal(buf.offsets.cpu().numpy(), offsets)
    assert np.array_equal(buf.row_of_slot.cpu().numpy(), ros)
    assert np.array_equal(buf.slot_of_row.cpu().numpy(), sor)
    assert np.array_equal(host_bits(buf.x_perm), O.permute_rows(inp["x"], sor, sh.K_slots))
    x, dout = f32w(inp, "x"), f32w(inp, "dout")
    wg, wu, wd = f32w(inp, "w_gate"), f32w(inp, "w_up"), f32w(inp, "w_down")
    out, _ = O.layer_forward(x, idx, w, wg, wu, wd)
    q = O.layer_scales(x, idx, w, wg, wu, wd, dout, sh.E_total)
    assert_close(host_f32(buf.out), out, q["out"], what="out")
    g = O.layer_backward(x, idx, w, wg, wu, wd, dout)
    assert_close(host_f32(buf.dx), g["dx"], q["dx"], what="dx")
    assert_close(buf.dtopk_w.cpu().numpy(), g["dtopk_w"], q["dtopk_w"], what="dtopk_w")
    assert_close(buf.dw_gate.cpu().numpy(), g["dw_gate"], q["dw_gate"], what="dw_gate")
    assert_close(buf.dw_up.cpu().numpy(), g["dw_up"], q["dw_up"], what="dw_up")
    assert_close(buf.dw_down.cpu().numpy(), g["dw_down"], q["dw_down"], what="dw_down")
    if probs is not None:
        dl = O.route_topk_bwd(g["dtopk_w"], idx, w, probs, sh.k, bool(renorm))
        # dlogits is linear in dtopk_w with coefficients <= 1: held to the largest dtopk_w scale of its token
        q_dl = np.broadcast_to(q["dtopk_w"].max(axis=1, keepdims=True), dl.shape)
        assert_close(buf.dlogits.cpu().numpy(), dl, q_dl, what="dlogits")
    return counts


@pytest.mark.parametrize("renorm", [1, 0])
def test_layer_tiny_workload(moe, renorm):
    inp = W.make_layer_inputs(W.WORKLOADS["tiny"], seed=0)
    check_layer_against_definition(moe, inp, renorm)


@pytest.mark.parametrize("name", ["mixtral", "finegrained", "shard", "imbalance"])
def test_layer_scaled_down_workloads(moe, name):
    """Same E, k, shared experts and routing recipe as the full workload; d, f / 8 and T / 4 so that the full
    fp64 oracle finishes in seconds."""
    w = W.scaled_down(W.WORKLOADS[name])
    inp = W.make_layer_inputs(w, seed=0)
    counts = check_layer_against_definition(moe, inp)
    if name == "imbalance":
        assert (counts == 0).sum() >= 20 and counts.max() > 4 * counts[counts > 0].mean()
    if name == "shard":
        assert counts.min() < 16


def test_dense_reduction_on_gpu(moe):
    """E = 1, k = 1: the layer is a dense SwiGLU FFN with gate weight 1."""
    sh = W.MoEShape(200, 128, 192, 1, 1)
    inp = W.random_layer_inputs(sh, seed=3)
    check_layer_against_definition(moe, inp)


def test_recomputing_backward_is_bit_identical(moe):
    """Checkpointed forward (G, U not kept) + recomputing backward: bit for bit the saving pair's outputs (same
    kernels on the same inputs), and within the bound of the oracle's grouped FFN like the saving pair."""
    wl = W.scaled_down(W.WORKLOADS["finegrained"])
    sh = wl.shape
    inp = W.make_layer_inputs(wl, seed=5)
    s = moe.Shape.of(sh)
    idx, w, _ = O.route_topk(inp["logits"], sh.k, sh.E_shared, True)
    counts, offsets, ros, sor = O.permute_maps(idx, sh.E_total)
    x_perm = dev_bf16(O.permute_rows(inp["x"], sor, sh.K_slots))
    dy = dev_bf16(W.f32_to_bf16_bits(np.random.default_rng(9).standard_normal((sh.N, sh.d_model)).astype(np.float32)))
    wg, wu, wd = dev_bf16(inp["w_gate"]), dev_bf16(inp["w_up"]), dev_bf16(inp["w_down"])
    off = dev(offsets.astype(np.int32))
    ws = ws_for(moe, s)
    e = lambda *sz, dtype=torch.bfloat16: torch.empty(*sz, dtype=dtype, device="cuda")  # noqa: E731
    y1, y2, sg, su = e(sh.N, sh.d_model), e(sh.N, sh.d_model), e(sh.N, sh.d_ffn), e(sh.N, sh.d_ffn)
    moe.moe_grouped_ffn_fwd(s, x_perm, off, wg, wu, wd, y1, sg, su, ws)
    moe.moe_grouped_ffn_fwd(s, x_perm, off, wg, wu, wd, y2, None, None, ws)
    assert torch.equal(y1.view(torch.int16), y2.view(torch.int16))
    outs = []
    for mode in ("saved", "recompute"):
        dx = e(sh.N, sh.d_model)
        dws = [e(sh.E_total, sh.d_model, sh.d_ffn, dtype=torch.float32), e(sh.E_total, sh.d_model, sh.d_ffn, dtype=torch.float32),
               e(sh.E_total, sh.d_ffn, sh.d_model, dtype=torch.float32)]
        if mode == "saved":
            moe.moe_grouped_ffn_bwd(s, dy, x_perm, off, wg, wu, wd, sg, su, dx, dws[0], dws[1], dws[2], 0, ws)
        else:
            moe.moe_grouped_ffn_bwd_recompute(s, dy, x_perm, off, wg, wu, wd, dx, dws[0], dws[1], dws[2], 0, ws)
        outs.append([dx.view(torch.int16)] + [t.view(torch.int32) for t in dws])
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    # ... and the recomputing call is held to the oracle directly
    wgf, wuf, wdf = f32w(inp, "w_gate"), f32w(inp, "w_up"), f32w(inp, "w_down")
    xpf, dyf = host_f32(x_perm), host_f32(dy)
    dX, dWg, dWu, dWd = O.grouped_ffn_bwd(dyf, xpf, offsets, wgf, wuf, wdf)
    qX, qWg, qWu, qWd = O.grouped_ffn_bwd_scales(dyf, xpf, offsets, wgf, wuf, wdf)
    assert_close(host_f32(dx), dX, qX, what="recompute dx_perm")
    assert_close(dws[0].cpu().numpy(), dWg, qWg, what="recompute dw_gate")
    assert_close(dws[1].cpu().numpy(), dWu, qWu, what="recompute dw_up")
    assert_close(dws[2].cpu().numpy(), dWd, qWd, what="recompute dw_down")
    Y, _, _ = O.grouped_ffn_fwd(xpf, offsets, wgf, wuf, wdf)
    assert_close(host_f32(y2), Y, O.grouped_ffn_fwd_scales(xpf, offsets, wgf, wuf, wdf)[0], what="checkpointed forward y_perm")


def test_weight_gradient_launches(moe):
    """Both weight-gradient problems in one launch, and in two beyond its limit (here between 600 and 612 experts): an expert's
    gradients are the same bits either way."""
    d = f = 768
    E, E1 = 612, 600
    s, x, dy, off, w, ws, _, sg, su = ffn_on_device(moe, d, f, [5] * E)
    got = []
    for e in (E, E1):
        sh = moe.Shape(5 * e, d, f, e, 1)
        dw = [torch.full(sz, float("nan"), device="cuda") for sz in ((e, d, f), (e, d, f), (e, f, d))]
        moe.profile_reset()
        moe.profile_enable(True)
        moe.moe_grouped_ffn_bwd(sh, dy[:5 * e], x[:5 * e], off[:e + 1], *(v[:e] for v in w), sg[:5 * e], su[:5 * e], torch.empty_like(x[:5 * e]), *dw,
                                False, ws)
        torch.cuda.synchronize()
        moe.profile_enable(False)
        labels = {label for label, _ in moe.profile_records()}
        moe.profile_reset()
        assert ("ffn_bwd_dw" in labels, "ffn_bwd_dw_down" in labels) == (e == E1, e == E)
        got.append(dw)
    assert moe.grouped_ffn_small_tiles(s) == moe.grouped_ffn_small_tiles(moe.Shape(5 * E1, d, f, E1, 1))
    for a, b in zip(*got):
        assert torch.equal(a[:E1], b)   # (not equal where one was left unwritten)


# one wavefront's experts and beyond, 1, 2 and 4 wavefronts per token, as many slots as are held in registers and one more
@pytest.mark.parametrize("T,d,E,k,Es,renorm", [(1, 64, 1, 1, 0, 1), (37, 512, 8, 2, 0, 1), (37, 512, 9, 3, 1, 0), (50, 1088, 64, 6, 2, 0), (50, 2112, 65, 8, 0, 1),
                                               (33, 2048, 200, 7, 1, 0), (20, 64, 1000, 8, 1, 1)])
def test_combine_and_route_backward_in_one(moe, T, d, E, k, Es, renorm):
    """dlogits made with dtopk_w: what the two calls give, which are compared with the oracle above (the same sums in the same order)."""
    s = moe.Shape(T, d, 64, E, k, Es, renorm)
    g = torch.Generator(device="cuda").manual_seed(T + E)
    idx = torch.empty(T, s.K_slots, dtype=torch.int32, device="cuda")
    w, dw, dw1 = (torch.empty(T, s.K_slots, device="cuda") for _ in range(3))
    probs, dl, dl1 = (torch.full((T, E), float("nan"), device="cuda") for _ in range(3))
    moe.moe_route_topk(s, torch.randn(T, E, device="cuda", generator=g), idx, w, probs)
    rows = torch.randperm(s.N, device="cuda", generator=g).to(torch.int32)
    dout, y = (torch.randn(n, d, device="cuda", generator=g).to(torch.bfloat16) for n in (T, s.N))
    dy, dy1 = torch.zeros_like(y), torch.zeros_like(y)
    moe.moe_unpermute_combine_bwd(s, dout, y, rows, w, dy, dw)
    moe.moe_route_topk_bwd(s, dw, idx, w, probs, dl)
    moe.moe_unpermute_combine_route_bwd(s, dout, y, rows, idx, w, probs, dy1, dw1, dl1)
    assert torch.equal(dy, dy1) and torch.equal(dw, dw1)
    # (the sums are alike, but for which of their products the compiler fuses with an addition: 2^-23 of each of the terms, of which a
    # logit's derivative has at most k + 1)
    bound = 2.0 ** -23 * 2 * (k + 1) * (w * dw).abs().sum(1, keepdim=True)
    assert bool(((dl - dl1).abs() <= bound).all())


@pytest.mark.parametrize("E", [151, 152])
def test_dx_beside_the_weight_gradients(moe, E):
    """dX on 64-row tiles shares the weight gradients' launch up to 256 of their chunks (here 151 experts of 54 tiles) and has one of its
    own beyond: against fp32 on the saved activations."""
    d = f = 768
    s, x, dy, off, w, ws, _, sg, su = ffn_on_device(moe, d, f, [70, 0, 1] + [5] * (E - 3))
    dx = torch.full((s.N, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    dw = [torch.full(t.shape, float("nan"), device="cuda") for t in w]
    moe.profile_reset()
    moe.profile_enable(True)
    moe.moe_grouped_ffn_bwd(s, dy, x, off, *w, sg, su, dx, *dw, False, ws)
    torch.cuda.synchronize()
    labels = [label for label, _ in moe.profile_records()]
    moe.profile_enable(False)
    moe.profile_reset()
    assert ("ffn_bwd_dx_dw" in labels, "ffn_bwd_dx" in labels) == (E == 151, E == 152)
    bounds = off.tolist()
    for e in (0, 1, 2, 3, E - 1):
        r = slice(bounds[e], bounds[e + 1])
        g, u = sg[r].float(), su[r].float()
        dh = dy[r].float() @ w[2][e].float().T
        sig = torch.sigmoid(g)
        # dG, dU and H are rounded to bf16 between the GEMMs: an error of 2^-9 of each, in quadrature over the contraction, so 2^-8
        # of the norm of a result bounds it with room
        h, du, dg = (z.to(torch.bfloat16).float() for z in (g * sig * u, dh * g * sig, dh * u * sig * (1 + g * (1 - sig))))
        want = (dg @ w[0][e].float().T + du @ w[1][e].float().T, x[r].float().T @ dg, x[r].float().T @ du, h.T @ dy[r].float())
        for got, ref in zip((dx[r].float(), dw[0][e], dw[1][e], dw[2][e]), want):
            assert bool(torch.isfinite(got).all()) and float((got - ref).norm()) <= 2.0 ** -8 * float(ref.norm())


# k-steps of dX: 64 always, 66 beside 4 chunks not; 128 beside 16 chunks and not beside 12; 240 beside 31, 242 never
@pytest.mark.parametrize("d,f,joined", [(64, 2048, True), (64, 2112, False), (640, 4096, True), (512, 4096, False), (640, 7680, True),
                                        (640, 7744, False)])
def test_long_dx_has_a_launch_of_its_own(moe, d, f, joined):
    moe.profile_reset()
    moe.profile_enable(True)
    try:
        test_grouped_ffn_every_tile_height(moe, d, f, [256, 0])
        labels = [label for label, _ in moe.profile_records()]
    finally:
        moe.profile_enable(False)
        moe.profile_reset()
    assert ("ffn_bwd_dx_dw" in labels, "ffn_bwd_dx" in labels) == (joined, not joined)


def test_grouped_ffn_with_no_rows(moe):
    """T = 0: nothing to compute, but overwritten weight gradients must be exact zeros and accumulated ones untouched."""
    shape = W.MoEShape(0, 128, 64, 4, 2)
    s = moe.Shape.of(shape)
    ws = ws_for(moe, s)
    off = torch.zeros(5, dtype=torch.int32, device="cuda")
    z = torch.zeros((16,), dtype=torch.bfloat16, device="cuda")
    wts = [torch.randn(4, 128, 64, device="cuda").to(torch.bfloat16), torch.randn(4, 128, 64, device="cuda").to(torch.bfloat16),
           torch.randn(4, 64, 128, device="cuda").to(torch.bfloat16)]
    dws = [torch.full((4, 128, 64), 3.0, device="cuda"), torch.full((4, 128, 64), 3.0, device="cuda"), torch.full((4, 64, 128), 3.0, device="cuda")]
    moe.moe_grouped_ffn_fwd(s, z, off, wts[0], wts[1], wts[2], z, z, z, ws)
    moe.moe_grouped_ffn_bwd(s, z, z, off, wts[0], wts[1], wts[2], z, z, z, dws[0], dws[1], dws[2], 1, ws)
    assert all(bool((t == 3.0).all()) for t in dws)
    moe.moe_grouped_ffn_bwd(s, z, z, off, wts[0], wts[1], wts[2], z, z, z, dws[0], dws[1], dws[2], 0, ws)
    assert all(not bool(t.any()) for t in dws)


MID_COUNTS = [1, 31, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 0, 256, 257, 385, 500]


# Tiles of 128 columns and up to 128 or 192 rows: rows on both sides of every class of 32 and of a second and third tile, a last column tile of
# 64 (d = 1088), contractions of 1, 2, 3 and more k-steps, experts of more than 12 row tiles (walked in bands), 128 experts with
# empty first and last ones (found from the offsets; the order of the experts is written by dH), dX in a launch of its own (4096 rows per expert)
@pytest.mark.parametrize("d,f,counts,mid", [
    (1088, 1728, MID_COUNTS, ALL_GEMMS),                          # up to 128 rows
    (1088, 1152, MID_COUNTS, ALL_GEMMS),                          # up to 192
    (64, 1088, 2 * MID_COUNTS, ("gate_up", "dh")),                # one k-step of gate | up and dH
    (1088, 64, 2 * MID_COUNTS, ("down", "dx")),                   # one of down, two of dX
    (192, 704, [2600, 0, 77, 1700], ("gate_up", "dh")),           # 3 k-steps; 21 row tiles of one expert
    (576, 192, [0, 0, 130] + 61 * [33, 2] + [1, 64, 0], ALL_GEMMS),
    (320, 320, [8200, 0], ALL_GEMMS),
    # experts of 18 to 36 row tiles: up to five bands of rows, of equal and of unequal height
    (640, 832, [4500, 0, 3400, 3392, 2817], ALL_GEMMS),
])
def test_mid_row_tiles(moe, d, f, counts, mid):
    s = moe.Shape(sum(counts), d, f, len(counts), 1)
    assert moe.grouped_ffn_mid_tiles(s) == mid
    moe.profile_reset()
    moe.profile_enable(True)
    try:
        test_grouped_ffn_every_tile_height(moe, d, f, counts)
        labels = [label for label, _ in moe.profile_records()]
    finally:
        moe.profile_enable(False)
        moe.profile_reset()
    assert ("ffn_schedule" in labels) == (not set(mid) | set(moe.grouped_ffn_small_tiles(s)) >= set(ALL_GEMMS))
    if "dx" in mid:
        assert ("ffn_bwd_dx" in labels) == (s.N >= 4096 * len(counts))


# The 256-row tiles where the smaller ones do not take over: every height class in all four GEMMs, left-over tiles (gate | up, down, dH, dX) in
# 2, 2, 2 and 2 pieces, whole and in 3, 5 and 3
@pytest.mark.parametrize("n_large", [8, 11])
def test_large_problem_on_256_row_tiles(moe, n_large):
    compare_ffn_on_device(moe, 2560, 1600, CLASS_COUNTS + n_large * [2000], (), ())


# experts of 18, 14, 13 (the last tile a tall one) and 11 row tiles: three and two bands of rows, of equal and of unequal height, and none; of 5
# tiles with a tall last one, 6 with a short one and 4, walked in bands of 8 of 9 column tiles (dX and down; 18 of gate | up)
def test_bands_of_256_row_tiles(moe):
    compare_ffn_on_device(moe, 2304, 2304, [4500, 0, 3400, 3392, 2817] + MANY_TILE_COUNTS, (), ())


# dH of 64 steps and dX of 200 in one backward, left-over tiles of both in 4 and 8 parts along k, on the same arrival counters
def test_dh_and_dx_cut_along_k(moe):
    compare_ffn_on_device(moe, 4096, 6400, [9, 20], ("gate_up", "down"), ())


def compare_ffn_on_device(moe, d, f, counts, small, mid):
    """Against fp32 on the device, expert by expert."""
    assert_runs_on(moe, d, f, counts, small, mid)
    s, x, dy, off, w, ws, y, sg, su = ffn_on_device(moe, d, f, counts)
    dx = torch.full((s.N, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    dw = [torch.full(t.shape, float("nan"), device="cuda") for t in w]
    moe.moe_grouped_ffn_bwd(s, dy, x, off, *w, sg, su, dx, *dw, False, ws)
    bounds = off.tolist()
    for e, n in enumerate(counts):
        r = slice(bounds[e], bounds[e + 1])
        if n == 0:
            assert not any(bool(t[e].any()) for t in dw)
            continue
        xe, dye, we = x[r].float(), dy[r].float(), [t[e].float() for t in w]
        # (a result rounded to bf16, of operands of which some were: 2^-9 each, so 2^-8 of the norm bounds them with room)
        g, u = sg[r].float(), su[r].float()
        sig = torch.sigmoid(g)
        dh = dye @ we[2].T
        h, du, dg = (z.to(torch.bfloat16).float() for z in (g * sig * u, dh * g * sig, dh * u * sig * (1 + g * (1 - sig))))
        want = (xe @ we[0], xe @ we[1], h @ we[2], dg @ we[0].T + du @ we[1].T, xe.T @ dg, xe.T @ du, h.T @ dye)
        for got, ref in zip((g, u, y[r].float(), dx[r].float(), dw[0][e], dw[1][e], dw[2][e]), want):
            assert bool(torch.isfinite(got).all()) and float((got - ref).norm()) <= 2.0 ** -8 * float(ref.norm()), (e, n)
            rows = (got - ref).norm(dim=1) / ref.norm(dim=1)   # (no row is lost in the norm of the whole)
            assert float(rows.max()) <= 2.0 ** -6, (e, n, float(rows.max()))
