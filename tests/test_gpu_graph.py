"""A whole layer step (forward + backward, ragged counts read on the device) captured into a HIP graph: every replay,
with new inputs written into the graph's static tensors and eager work and synchronisations in between, must give
bit for bit what the eager call order gives on the same inputs (same kernels, same launch shapes, fixed reduction
orders), and the eager result itself is held to the oracle by the parity tests."""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_parity import dev, dev_bf16, ffn_on_device

pytestmark = pytest.mark.gpu

CASES = [
    ("tiny", W.WORKLOADS["tiny"]),
    ("imbalance_scaled", W.scaled_down(W.WORKLOADS["imbalance"])),      # empty experts, ragged tiles; all on tiles of 128 columns
    ("finegrained_scaled", W.scaled_down(W.WORKLOADS["finegrained"])),  # shared experts; all on tiles of 128 columns
    # few tokens on wide experts: dH cuts its tiles along k, on arrival counters that every replay finds as the last left them
    ("split", W.Workload("split", W.MoEShape(16, 4096, 2048, 4, 1), "router")),
]
ALL_GEMMS = ("gate_up", "down", "dh", "dx")
TILES = {"tiny": (("down", "dh", "dx"), ("gate_up",)), "imbalance_scaled": ((), ALL_GEMMS), "finegrained_scaled": ((), ALL_GEMMS),
         "split": (("gate_up", "down"), ("dx",))}   # (on 64-row tiles, on tiles of 128 columns)


def _tensors(buf, with_router):
    names = ["topk_idx", "topk_w", "counts", "offsets", "row_of_slot", "slot_of_row", "x_perm", "y_perm", "out",
             "dy_perm", "dtopk_w", "dx_perm", "dx", "dw_gate", "dw_up", "dw_down"]
    if with_router:
        names += ["probs", "dlogits"]
    return {n: getattr(buf, n) for n in names}


@pytest.mark.parametrize("name,wl", CASES, ids=[c[0] for c in CASES])
def test_graph_replays_match_eager(moe, name, wl):
    sh = wl.shape
    s = moe.Shape.of(sh)
    assert (moe.grouped_ffn_small_tiles(s), moe.grouped_ffn_mid_tiles(s)) == TILES[name]
    inp = W.make_layer_inputs(wl, seed=0)
    if "logits" not in inp:
        pytest.skip("workload without router logits")
    x, dout, logits = dev_bf16(inp["x"]), dev_bf16(inp["dout"]), dev(inp["logits"])
    wg, wu, wd = dev_bf16(inp["w_gate"]), dev_bf16(inp["w_up"]), dev_bf16(inp["w_down"])
    buf_graph, buf_eager = moe.MoeLayerBuffers(s), moe.MoeLayerBuffers(s)
    step = moe.CapturedLayerStep(buf_graph, x, dout, wg, wu, wd, logits=logits)
    for replay in range(3):
        print(f"[graph] {name}: replay {replay}", flush=True)
        other = W.make_layer_inputs(wl, seed=10 + replay)      # new inputs, and with them another routing
        x.copy_(dev_bf16(other["x"])); dout.copy_(dev_bf16(other["dout"])); logits.copy_(dev(other["logits"]))
        step.replay()
        torch.cuda.synchronize()
        moe.layer_forward(buf_eager, x, wg, wu, wd, logits)
        moe.layer_backward(buf_eager, dout, wg, wu, wd)
        torch.cuda.synchronize()
        got, ref = _tensors(buf_graph, True), _tensors(buf_eager, True)
        for n in got:
            a, b = got[n], ref[n]
            if a.dtype == torch.bfloat16:
                a, b = a.view(torch.int16), b.view(torch.int16)
            assert torch.equal(a, b), f"{name}: replay {replay}: {n} differs from the eager result"
        assert int(buf_graph.counts.sum()) == s.N


def test_replays_of_tiles_cut_along_k(moe):
    """dH and dX of one backward both cut their tiles along k, on the same arrival counters, which every replay finds as the last left them."""
    counts = [9, 20]
    s, x, dy, off, w, ws, y, sg, su = ffn_on_device(moe, 4096, 6400, counts)
    assert (moe.grouped_ffn_small_tiles(s), moe.grouped_ffn_mid_tiles(s)) == (("gate_up", "down"), ())

    def call(ws, y, g, u, dx, dw):
        moe.moe_grouped_ffn_fwd(s, x, off, *w, y, g, u, ws)
        moe.moe_grouped_ffn_bwd(s, dy, x, off, *w, g, u, dx, *dw, False, ws)

    def buffers():
        return (torch.empty_like(ws), *(torch.full_like(t, float("nan")) for t in (y, sg, su, x)), [torch.full(t.shape, float("nan"), device="cuda") for t in w])

    replayed, eager = buffers(), buffers()
    call(*replayed)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(*replayed)
    for replay in range(3):
        print(f"[graph] cut along k: replay {replay}", flush=True)
        g = torch.Generator(device="cuda").manual_seed(replay)
        for t in (x, dy):
            t.copy_(torch.randn(t.shape, device="cuda", generator=g))
        for t in (*replayed[1:5], *replayed[5]):
            t.fill_(float("nan"))
        graph.replay()
        call(*eager)
        torch.cuda.synchronize()
        for a, b in zip((*replayed[1:5], *replayed[5]), (*eager[1:5], *eager[5])):
            assert bool(torch.isfinite(a).all()) and torch.equal(a, b)
