"""The work that is measured: what a user of the MoE expert layer has it do, as calls of the package's entry points.

A case is a dict of plain values.  `kind` says which calls one pass makes:

  step      forward + backward of one layer (layer_forward, layer_backward), the training step.  routing: "router" (the
            layer closed from x: router weight -> logits -> top-k, and back to dx and the router weight's gradient),
            "logits" (gate logits given) or "given" (an expert-parallel shard: expert ids and gate weights arrive with
            the rows).  captured: the step is one HIP graph replay.
  forward   the forward half alone, closed from x (evaluation, generation).
  micro     two micro-batches of gradient accumulation under activation checkpointing: the forward keeps x_perm only, the
            backward recomputes G and U; the first overwrites the weight gradients, the second adds to them.
  ffn       the grouped expert FFN alone, forward + backward, on rows that are already grouped by expert (the
            expert-GEMM sweep's benchmark).
  movement  permute, combine and the backward of both (the permute/combine bandwidth benchmark).

load: how tokens spread over the experts: "even" (i.i.d. logits), "bias" (per-expert bias ~ N(0, 0.5)), "forced" (10 % of
the experts get 60 % of the slots, 20 % get none), "zipf" (popularity ~ rank^-1.2).  x, dout ~ N(0,1), weights ~ N(0,0.02),
all bf16; weight gradients fp32.
"""
import math

import torch

import paper_2605_05049_amd as moe

_ZIPF = 1.2
_HOT_LOG_RATIO = 2.4      # hot : warm log-popularity of the forced imbalance


def _case(name, kind, T, d, f, E, k, Es=0, renorm=True, routing="router", load="even", captured=False):
    return {"name": name, "kind": kind, "T": T, "d": d, "f": f, "E": E, "k": k, "Es": Es, "renorm": renorm, "routing": routing,
            "load": load, "captured": captured}


def listed():
    return [
        # the smallest training step: ~20 dependent launches of little work each, bound by latency
        _case("step_tiny", "step", 256, 512, 1024, 8, 2),
        # the same step as a user with launch overhead to save runs it: one graph replay
        _case("replay_tiny", "step", 256, 512, 1024, 8, 2, captured=True),
        # generation: a few tokens, every active expert's weights streamed for a handful of rows
        _case("forward_few", "forward", 16, 2048, 1408, 64, 6, Es=2),
        # nothing a multiple of a tile: odd token count, odd expert count, a shared expert, gate weights not renormalised
        _case("step_odd", "step", 1003, 1088, 1984, 13, 3, Es=1, renorm=False, load="bias"),
        # wide experts with 64 rows each: forward and backward bound by weights and their gradients
        _case("ffn_64_rows", "ffn", 512, 4096, 14336, 8, 1, routing="given"),
        # gradient accumulation with recomputed activations on fine-grained experts
        _case("micro_finegrained", "micro", 2048, 2048, 1408, 64, 6, Es=2, routing="logits", load="bias"),
        # the fine-grained layer: 64 routed experts, top-6, two shared ones, mild imbalance
        _case("step_finegrained", "step", 8192, 2048, 1408, 64, 6, Es=2, load="bias"),
        # one expert-parallel shard: 32 local experts, popularity so skewed that some get a few rows
        _case("step_shard", "step", 4096, 7168, 2048, 32, 1, routing="given", load="zipf"),
        # many experts, forced imbalance
        _case("step_imbalance", "step", 16384, 4096, 1024, 128, 4, routing="logits", load="forced"),
        # few wide experts, near-uniform load: the headline benchmark's layer
        _case("step_wide", "step", 4096, 4096, 14336, 8, 2, routing="logits"),
        # evaluation of a long odd prompt on the same layer
        _case("forward_long", "forward", 3001, 4096, 14336, 8, 2),
        # the permute/combine bandwidth benchmark
        _case("movement", "movement", 16384, 4096, 1024, 128, 4, routing="logits", load="forced"),
    ]


_MAX_FLOPS = 18.0 * 4096 * 14336 * 8192     # of the largest listed case
_MAX_WEIGHTS = 8 * 3 * 4096 * 14336         # its expert weights, in elements


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: 1 to 16384 tokens, widths 512 .. 7168 and 512 .. 14336 in multiples of 64, 4 to 128 experts."""
    kind = rng.choice(["step"] * 5 + ["forward"] * 2 + ["micro", "ffn", "movement"])
    while True:
        T = _log_int(rng, 1 if kind == "forward" else 64, 16384)
        d = 64 * _log_int(rng, 8, 112)
        f = 64 * _log_int(rng, 8, 224)
        E = _log_int(rng, 4, 128)
        k = 1 if kind == "ffn" else rng.randint(1, min(8, E))
        Es = 0 if kind == "ffn" else rng.choice([0, 0, 1, 2])
        K = k + Es
        weights = 3 * (E + Es) * d * f if kind != "movement" else 0
        flops = 18.0 * d * f * T * K if kind != "movement" else 0.0
        # the whole pass stays below the largest listed one: arithmetic, weights, rows and fp32 gradients
        if flops + 500.0 * 18 * weights > _MAX_FLOPS or weights > _MAX_WEIGHTS or T * K > 65536 or T * K * max(d, f) > 65536 * 4096:
            continue
        break
    routing = "given" if kind == "ffn" else "router" if kind == "forward" else rng.choice(["router", "logits", "given"])
    if kind in ("micro", "movement") and routing == "router":
        routing = "logits"
    if routing == "given" and (k > 1 or Es > 0):
        routing = "logits"
    load = rng.choice(["even", "zipf"]) if routing == "given" else rng.choice(["even", "bias"]) if routing == "router" else rng.choice(["even", "bias", "forced"])
    c = _case("", kind, T, d, f, E, k, Es, rng.random() < 0.75, routing, load, kind == "step" and rng.random() < 0.2)
    del c["name"]
    return c


def _shape(c):
    return moe.Shape(c["T"], c["d"], c["f"], c["E"], c["k"], c["Es"], 1 if c["renorm"] else 0)


def _zipf_counts(E, total, gen):
    p = torch.arange(1, E + 1, dtype=torch.float64) ** -_ZIPF
    p = (p / p.sum())[torch.randperm(E, generator=gen)]
    n = (p * total).floor().to(torch.int64)
    n[int(n.argmax())] += total - int(n.sum())
    return n


def prepare(case, seed):
    s = _shape(case)
    T, d, f, E, Et = s.T, s.d_model, s.d_ffn, s.E, s.E_total
    kind = case["kind"]
    host = torch.Generator().manual_seed(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*size, std=1.0):
        return torch.randn(*size, device="cuda", generator=gen).mul_(std).to(torch.bfloat16)

    def weights(a, b):
        w = torch.empty(Et, a, b, dtype=torch.bfloat16, device="cuda")
        for e in range(Et):
            w[e] = normal(a, b, std=0.02)
        return w

    st = {"case": dict(case), "shape": s}
    if kind != "movement":
        st["w_gate"], st["w_up"], st["w_down"] = weights(d, f), weights(d, f), weights(f, d)
    if kind == "ffn":
        n = _zipf_counts(E, T, host) if case["load"] == "zipf" else torch.full((E,), T // E, dtype=torch.int64)
        n[0] += T - int(n.sum())
        st["offsets"] = torch.cat([torch.zeros(1, dtype=torch.int64), n.cumsum(0)]).to(torch.int32).cuda()
        st["x"], st["dy"] = normal(T, d), normal(T, d)
        bf = dict(dtype=torch.bfloat16, device="cuda")
        st["y"], st["dx"] = torch.empty(T, d, **bf), torch.empty(T, d, **bf)
        st["g"], st["u"] = torch.empty(T, f, **bf), torch.empty(T, f, **bf)
        st["dw_gate"] = torch.empty(E, d, f, device="cuda")
        st["dw_up"] = torch.empty(E, d, f, device="cuda")
        st["dw_down"] = torch.empty(E, f, d, device="cuda")
        st["ws"] = torch.empty(moe.workspace_bytes(s), dtype=torch.uint8, device="cuda")
        return st

    batches = []
    for _ in range(2 if kind == "micro" else 1):
        b = {"x": normal(T, d), "dout": normal(T, d)}
        if case["routing"] == "given":
            if case["load"] == "zipf":
                p = torch.arange(1, E + 1, dtype=torch.float64) ** -_ZIPF
                ids = torch.multinomial(p[torch.randperm(E, generator=host)], T, replacement=True, generator=host)
            else:
                ids = torch.randint(E, (T,), generator=host)
            b["topk_idx"] = ids.to(torch.int32).reshape(T, 1).cuda()
            b["topk_w"] = torch.rand(T, 1, device="cuda", generator=gen)
        elif case["routing"] == "logits":
            z = torch.randn(T, E, device="cuda", generator=gen) * (0.02 * math.sqrt(d))
            if case["load"] == "bias":
                z += 0.5 * torch.randn(E, device="cuda", generator=gen)
            elif case["load"] == "forced":
                order = torch.randperm(E, generator=host).cuda()
                n_dead = min(int(round(0.2 * E)), E - s.k)
                n_hot = min(max(1, int(round(0.1 * E))), E - n_dead)
                base = torch.zeros(E, device="cuda")
                base[order[:n_hot]] = _HOT_LOG_RATIO
                base[order[n_hot:n_hot + n_dead]] = -1e30
                u = torch.rand(T, E, device="cuda", generator=gen).clamp_(1e-30, 1 - 1e-7)
                z = base - torch.log(-torch.log(u))
            b["logits"] = z.contiguous()
        batches.append(b)
    st["batches"] = batches
    if case["routing"] == "router":
        st["w_router"] = normal(E, d, std=0.02)
        if case["load"] == "bias":   # a popular expert's row has a part along the mean token
            batches[0]["x"] += 0.25
            st["w_router"] += 0.5 / (0.25 * d) * torch.randn(E, 1, device="cuda", generator=gen)
    if kind == "movement":
        bf = dict(dtype=torch.bfloat16, device="cuda")
        i32 = dict(dtype=torch.int32, device="cuda")
        st.update(topk_idx=torch.empty(T, s.K_slots, **i32), topk_w=torch.empty(T, s.K_slots, device="cuda"), counts=torch.empty(Et, **i32),
                  offsets=torch.empty(Et + 1, **i32), row_of_slot=torch.empty(s.N, **i32), slot_of_row=torch.empty(s.N, **i32),
                  x_perm=torch.empty(s.N, d, **bf), y_perm=normal(s.N, d), out=torch.empty(T, d, **bf), dy_perm=torch.empty(s.N, d, **bf),
                  dtopk_w=torch.empty(T, s.K_slots, device="cuda"), dx=torch.empty(T, d, **bf),
                  ws=torch.empty(moe.workspace_bytes(s), dtype=torch.uint8, device="cuda"))
        b = batches[0]
        if case["routing"] == "given":
            st["topk_idx"], st["topk_w"] = b["topk_idx"], b["topk_w"]
        else:
            moe.moe_route_topk(s, b["logits"], st["topk_idx"], st["topk_w"], None)
        return st
    buf = moe.MoeLayerBuffers(s, with_backward=kind != "forward", with_router=case["routing"] != "given")
    st["buf"] = buf
    if case["routing"] == "given":
        buf.topk_idx.copy_(batches[0]["topk_idx"])
        buf.topk_w.copy_(batches[0]["topk_w"])
    if case["captured"]:
        b = batches[0]
        st["graph"] = moe.CapturedLayerStep(buf, b["x"], b["dout"], st["w_gate"], st["w_up"], st["w_down"], logits=b.get("logits"),
                                            w_router=st.get("w_router"), with_router=case["routing"] != "given")
    return st


def run(st):
    case, s = st["case"], st["shape"]
    kind = case["kind"]
    if kind == "ffn":
        moe.moe_grouped_ffn_fwd(s, st["x"], st["offsets"], st["w_gate"], st["w_up"], st["w_down"], st["y"], st["g"], st["u"], st["ws"])
        moe.moe_grouped_ffn_bwd(s, st["dy"], st["x"], st["offsets"], st["w_gate"], st["w_up"], st["w_down"], st["g"], st["u"], st["dx"],
                                st["dw_gate"], st["dw_up"], st["dw_down"], False, st["ws"])
        return {n: st[n] for n in ("y", "g", "u", "dx", "dw_gate", "dw_up", "dw_down")}
    b = st["batches"][0]
    if kind == "movement":
        moe.moe_permute(s, b["x"], st["topk_idx"], st["x_perm"], st["counts"], st["offsets"], st["row_of_slot"], st["slot_of_row"], st["ws"])
        moe.moe_unpermute_combine(s, st["y_perm"], st["row_of_slot"], st["topk_w"], st["out"])
        moe.moe_unpermute_combine_bwd(s, b["dout"], st["y_perm"], st["row_of_slot"], st["topk_w"], st["dy_perm"], st["dtopk_w"])
        moe.moe_permute_bwd(s, st["dy_perm"], st["row_of_slot"], st["dx"])
        return {n: st[n] for n in ("x_perm", "counts", "offsets", "row_of_slot", "slot_of_row", "out", "dy_perm", "dtopk_w", "dx")}
    buf, w = st["buf"], (st["w_gate"], st["w_up"], st["w_down"])
    if kind == "forward":
        return {"out": moe.layer_forward(buf, b["x"], *w, logits=b.get("logits"), w_router=st.get("w_router")), "logits": buf.logits,
                "topk_w": buf.topk_w}
    gated = case["routing"] != "given"
    if kind == "step":
        if case["captured"]:
            st["graph"].replay()
        else:
            moe.layer_forward(buf, b["x"], *w, logits=b.get("logits"), w_router=st.get("w_router"))
            moe.layer_backward(buf, b["dout"], *w, with_router=gated, x=b["x"] if "w_router" in st else None, w_router=st.get("w_router"))
        got = {n: getattr(buf, n) for n in ("out", "dx", "dtopk_w", "dw_gate", "dw_up", "dw_down")}
        if gated:
            got["dlogits"] = buf.dlogits
        if "w_router" in st:
            got["dw_router"] = buf.dw_router
        return got
    for i, b in enumerate(st["batches"]):
        if gated:
            moe.moe_route_topk(s, b["logits"], buf.topk_idx, buf.topk_w, buf.probs)
        moe.moe_permute(s, b["x"], buf.topk_idx, buf.x_perm, buf.counts, buf.offsets, buf.row_of_slot, buf.slot_of_row, buf.ws)
        moe.moe_grouped_ffn_fwd(s, buf.x_perm, buf.offsets, *w, buf.y_perm, None, None, buf.ws)
        moe.moe_unpermute_combine(s, buf.y_perm, buf.row_of_slot, buf.topk_w, buf.out)
        moe.moe_unpermute_combine_bwd(s, b["dout"], buf.y_perm, buf.row_of_slot, buf.topk_w, buf.dy_perm, buf.dtopk_w)
        moe.moe_grouped_ffn_bwd_recompute(s, buf.dy_perm, buf.x_perm, buf.offsets, *w, buf.dx_perm, buf.dw_gate, buf.dw_up, buf.dw_down, i > 0,
                                          buf.ws)
        moe.moe_permute_bwd(s, buf.dx_perm, buf.row_of_slot, buf.dx)
        if gated:
            moe.moe_route_topk_bwd(s, buf.dtopk_w, buf.topk_idx, buf.topk_w, buf.probs, buf.dlogits)
    return {n: getattr(buf, n) for n in ("out", "dx", "dtopk_w", "dw_gate", "dw_up", "dw_down")}


def work(case):
    """Arithmetic of the GEMMs, and the bytes of the pass's inputs and outputs, each once (what lies between them, the
    permuted rows and the activations, is left out where a pass makes and uses it itself; weights of experts that the
    rows cannot all reach are counted for the experts that they can)."""
    s = _shape(case)
    T, d, f, N, E, Et = s.T, s.d_model, s.d_ffn, s.N, s.E, s.E_total
    kind = case["kind"]
    rows, tok = 2 * d * N, 2 * d * T
    if kind == "movement":
        # permute: read x, write x_perm; combine: read y, write out; its backward: read dout and y, write dy; permute
        # backward: read dy, write dx (four calls, each of which has to read and write its own tensors)
        return {"bytes": 5 * rows + 4 * tok + 8 * 4 * N, "flops": 2 * d * N * 4}
    live = E if case["load"] != "forced" else E - int(round(0.2 * E))
    if T * s.k < 4 * E:   # few tokens: the expected number of experts with a row
        live = live * (1 - (1 - 1 / max(live, 1)) ** (T * s.k))
    live += case["Es"]
    weights = 3 * live * d * f * 2
    grads = 3 * Et * d * f * 4
    gate = 4 * T * E if case["routing"] == "logits" else 2 * E * d if case["routing"] == "router" else 8 * T
    if kind == "forward":
        return {"bytes": weights + 2 * tok + gate, "flops": 6.0 * d * f * N + 2.0 * T * E * d}
    if kind == "ffn":
        return {"bytes": weights + grads + 4 * tok + 2 * T * f * 2, "flops": 18.0 * d * f * N}
    router = 6.0 * T * E * d if case["routing"] == "router" else 0.0
    if kind == "micro":
        return {"bytes": weights + grads + 2 * (4 * tok + gate), "flops": 2 * 22.0 * d * f * N}
    return {"bytes": weights + grads + 4 * tok + 2 * gate, "flops": 18.0 * d * f * N + router}


def tolerance(case):
    if case["kind"] == "movement":
        # copies are exact; sums of up to 10 terms in fp32, rounded to bf16 once (in the reverse order 1e-5 to 2e-5, and at
        # most one bf16 step, 8e-3, in one element), dot products in fp32 (1e-7)
        return {"rel": 1e-4, "max": 2e-2}
    # Against the same step in 64 bits: out 2.9e-3, dx 3.4e-3 to 3.8e-3, gradients of the weights 2.5e-3 to 3.5e-3, of the
    # logits 2.2e-3 to 2.5e-3 (bf16 roundings of G, U, H, Y, dG, dU, dX); largest element 0.11 of the rms (an expert with few
    # rows among many-row ones)
    return {"rel": 1.2e-2, "max": 0.3}
