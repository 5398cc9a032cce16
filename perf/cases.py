"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is a dict of plain values.  ``path`` says which calls one pass makes:

    layer      one MoE layer on one GPU as bench.py runs it: the predictor of the next layer, the router, permute,
               grouped FFN, combine; the options below choose among the library's forms of these calls
    route      the router alone, fp32 gate and full probabilities (scoring and evaluation runs)
    residual   the lookahead predictor with its residual MLP (Eq. 7 in full)
    dispatch   the sending side of the exchange: greedy plan, this rank's dispatch plan, rows grouped by destination

Shapes are those of the configurations in paper_2602_00509_amd/workload.py, of the tests, or generic.  Everything
lives on the GPU, is made from the seed alone, and outputs and workspaces are allocated once, as a serving program
does.
"""
import math

import numpy as np
import torch

from paper_2602_00509_amd import probe, workload

RANKS = 8          # expert-parallel ranks of the dispatch path


def _layer(name, T, H, E, k, F, E_loc, n_rep, zipf, chunk=0, *, gate="packed", gather=False, fused=False,
           grouped=False, shared=False, graph=False):
    """chunk: tokens per popularity order (0 = one order); gate: "packed" planes or the "fp32" matrix; gather: rows
    read on load instead of permuted; fused: router and predictor in one call; grouped: group-limited sigmoid gate;
    shared: a shared expert on every token; graph: the pass recorded once and replayed."""
    return dict(name=name, path="layer", T=T, H=H, E=E, k=k, F=F, E_loc=E_loc, n_rep=n_rep, zipf=zipf, chunk=chunk,
                gate=gate, gather=gather, fused=fused, grouped=grouped, shared=shared, graph=graph)


def listed():
    return [
        # a small model's layer: nothing but launches and latency
        _layer("tiny_layer", 256, 512, 8, 2, 1024, 8, 1, 1.2),
        # one sequence generating on one GPU that holds every expert of an 8-expert model
        _layer("decode_8x_one_token", 1, 4096, 8, 2, 14336, 8, 2, 1.0),
        # a decode step of a 128-expert model on one of eight ranks, replayed from a graph as serving loops do
        _layer("decode_128x_graph", 128, 4096, 128, 8, 1536, 16, 2, 1.1, graph=True),
        # a decode step of a 256-expert model with its own gate (8 groups of which 4, sigmoid) and a shared expert,
        # at a batch that is no multiple of anything
        _layer("decode_256x_grouped_shared", 75, 7168, 256, 8, 2048, 32, 4, 1.1, gather=True, grouped=True,
               shared=True),
        # the decode batch the paper measures (768 per rank), top-4 of 128, hidden size 2880
        _layer("decode_128x_768", 768, 2880, 128, 4, 2880, 16, 2, 1.1),
        # a mixed batch (decode and a piece of a prompt) of ragged size, router and predictor in one pass
        _layer("mixed_128x_2500", 2500, 4096, 128, 8, 1536, 16, 2, 1.1, fused=True),
        # prefill of an 8-expert model, the popular experts move every 512 tokens
        _layer("prefill_8x_4096", 4096, 4096, 8, 2, 14336, 8, 2, 1.0, 512),
        # prefill chunk on one of eight ranks of a 256-expert model: the benchmark's own workload
        _layer("prefill_256x_8192", 8192, 7168, 256, 8, 2048, 32, 4, 1.1),
        # the largest: a 16K-token chunk, a quarter of 256 experts, strong skew
        _layer("prefill_256x_16384", 16384, 7168, 256, 8, 2048, 64, 0, 1.5, 1024),
        # a router on odd sizes, fp32 gate handed over per call, all probabilities out
        dict(name="route_odd_probs", path="route", T=3001, H=1000, E=60, k=6, renorm=False),
        # the distilled predictor during prefill
        dict(name="predict_residual_8192", path="residual", T=8192, H=7168, E=256, k=8, D=256),
        # plan for the next layer and rows grouped for the exchange, on the sending rank
        dict(name="plan_and_dispatch_3000", path="dispatch", T=3000, H=4096, E=128, k=8, zipf=1.1),
    ]


# (H, E, k, F, E_loc, n_rep) of the shapes above; draw() adds generic ones
_SHAPES = [(4096, 8, 2, 14336, 8, 2), (7168, 256, 8, 2048, 32, 4), (4096, 128, 8, 1536, 16, 2),
           (2880, 128, 4, 2880, 16, 2), (7168, 256, 8, 2048, 64, 0)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer"] * 9 + ["route", "residual", "dispatch"])
    if kind == "route":
        E = rng.randint(8, 256)
        H = 8 * _log(rng, 16, 896) if rng.random() < 0.5 else 64 * _log(rng, 4, 112)
        return dict(path="route", T=_log(rng, 1, 16384), H=H, E=E, k=rng.randint(1, min(8, E)),
                    renorm=rng.random() < 0.5)
    if kind == "residual":
        return dict(path="residual", T=_log(rng, 64, 12000), H=64 * _log(rng, 8, 112), E=rng.choice([64, 128, 200, 256]),
                    k=rng.choice([4, 6, 8]), D=rng.choice([64, 128, 256, 512]))
    if kind == "dispatch":
        return dict(path="dispatch", T=_log(rng, 64, 8192), H=64 * _log(rng, 16, 112), E=rng.choice([64, 128, 256]),
                    k=rng.choice([4, 6, 8]), zipf=round(rng.uniform(0.8, 1.5), 2))
    if rng.random() < 0.75:
        H, E, k, F, E_loc, n_rep = rng.choice(_SHAPES)
        T = _log(rng, 1, 4096 if E == 8 else 8192)
    else:
        E = 16 * rng.randint(1, 16)
        k = rng.randint(2, 8)
        H, F = 64 * _log(rng, 8, 80), 64 * _log(rng, 8, 48)
        E_loc = E // rng.choice([1, 2, 4, 8])
        while E_loc > 64:
            E_loc //= 2
        n_rep = rng.randint(0, 3)
        T = _log(rng, 1, 8192)
        while T * k * H * F * E_loc / E > 2e11:      # stays below the largest listed case
            T //= 2
    c = _layer("", T, H, E, k, F, E_loc, n_rep, round(rng.uniform(1.0, 1.5), 2),
               rng.choice([0, 0, 512]), gate=rng.choice(["packed", "packed", "fp32"]), gather=rng.random() < 0.3)
    c["grouped"] = E >= 64 and E % 64 == 0 and rng.random() < 0.25
    c["fused"] = not c["grouped"] and rng.random() < 0.25
    c["shared"] = E > 8 and T <= 4096 and rng.random() < 0.2
    c["graph"] = T <= 512 and rng.random() < 0.3
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs

def _config(c):
    return workload.LayerConfig(0, "", c["T"], c["H"], c["E"], c["k"], c["F"], c["E_loc"], c["n_rep"], c["zipf"],
                                c["chunk"], 1, max(c["E"] // c["E_loc"], 1))


def _zipf_bias(rng, groups, E, s):
    """-s ln(rank) under a fresh popularity order per group: softmax prior ~ rank^-s, fp32 [groups, E]."""
    rank = np.stack([rng.permutation(E) for _ in range(groups)]) + 1.0
    return (-s * np.log(rank)).astype(np.float32)


def _normal(gen, shape, scale, dtype):
    """N(0, scale^2), drawn in fp32 and rounded to dtype."""
    return (torch.randn(shape, generator=gen, device="cuda") * scale).to(dtype)


def _expert(gen, H, F):
    return _normal(gen, (2 * F, H), 0.02, torch.bfloat16), _normal(gen, (H, F), 0.02, torch.bfloat16)


def _empty(shape, dtype):
    return torch.empty(shape, dtype=dtype, device="cuda")


def _route_out(T, k, E, probs=False):
    out = dict(idx=_empty((T, k), torch.int32), w=_empty((T, k), torch.float32), counts=_empty((E,), torch.int32))
    if probs:
        out["probs"] = _empty((T, E), torch.float32)
    return out


def _permute_out(T, k, H, S, copy):
    N = T * k
    out = dict(slot_counts=_empty((S,), torch.int32), slot_offsets=_empty((S + 1,), torch.int32),
               row_pair=_empty((N,), torch.int32), pair_row=_empty((T, k), torch.int32),
               n_local=_empty((1,), torch.int32))
    if copy:
        out["xp"] = torch.zeros((N, H), dtype=torch.bfloat16, device="cuda")
    return out


def _prepare_layer(c, seed):
    cfg = _config(c)
    T, H, E, k, F, S = cfg.T, cfg.H, cfg.E, cfg.k, cfg.F, cfg.S
    rng = np.random.default_rng([seed, 1])
    gen = torch.Generator(device="cuda").manual_seed(seed)
    s = dict(case=c, k=k, tpg=c["chunk"] or T, x=_normal(gen, (T, H), 1.0, torch.bfloat16))
    gates = [_normal(gen, (E, H), 0.02, torch.float32) for _ in range(2)]
    bias = [_zipf_bias(rng, cfg.G, E, cfg.zipf_s) for _ in range(2)]
    s["bias"], s["bias_next"] = (torch.from_numpy(b).cuda() for b in bias)
    s["select_bias"] = _normal(gen, (E,), 0.01, torch.float32) if c["grouped"] else None
    # the plan that was made for this batch: the host recipe of the workload on the batch's expected expert loads
    logits = s["x"].float() @ gates[0].t() + s["bias"][torch.arange(T, device="cuda") // s["tpg"]]
    counts = torch.bincount(logits.topk(k, dim=1).indices.flatten(), minlength=E).cpu().numpy()
    plan = workload.build_plan(cfg, counts)
    s["plan"] = probe.Plan(plan["rep_off"], plan["rep_slot"], plan["rep_weight"], plan["num_slots"], "cuda")
    # slot weights; a replica holds a copy of its expert's
    own = {int(e): _expert(gen, H, F) for e in sorted(set(plan["slot_expert"].tolist()))}
    seen, w13, w2 = set(), [], []
    for e in plan["slot_expert"].tolist():
        a, b = own[e]
        w13.append(a.clone() if e in seen else a)
        w2.append(b.clone() if e in seen else b)
        seen.add(e)
    s["weights"] = probe.WeightTable(w13, w2)
    if c["fused"]:
        s["gate"], s["gate_next"] = (probe.PackedGate(*gates), None) if c["gate"] == "packed" else gates
        need = probe.route_predict_topk_workspace_bytes(T, H, E, k)
    else:
        s["gate"], s["gate_next"] = map(probe.PackedGate, gates) if c["gate"] == "packed" else gates
        need = probe.route_topk_workspace_bytes(T, H, E, k)
    s["ws_route"] = _empty((max(need, 256),), torch.uint8)
    s["ws_permute"] = _empty((max(probe.permute_workspace_bytes(T, E, k, S), 256),), torch.uint8)
    s["ws_ffn"] = _empty((probe.grouped_ffn_workspace_bytes(S, H, F, T * k),), torch.uint8)
    s["routed"], s["predicted"] = _route_out(T, k, E), _route_out(T, k, E)
    s["permuted"] = _permute_out(T, k, H, S, not c["gather"])
    s["y"], s["out"] = _empty((T * k, H), torch.bfloat16), _empty((T, H), torch.bfloat16)
    if c["shared"]:
        a, b = _expert(gen, H, F)
        s["shared"] = dict(weights=probe.WeightTable([a], [b]), y=_empty((T, H), torch.bfloat16),
                           offsets=torch.tensor([0, T], dtype=torch.int32, device="cuda"),
                           ws=_empty((probe.grouped_ffn_workspace_bytes(1, H, F, T),), torch.uint8))
    if c["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _run_layer(s)                # the first call of a process sets the kernels up, outside the capture
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"], stream=side):
                s["result"] = _run_layer(s)
        torch.cuda.current_stream().wait_stream(side)
    return s


def prepare(case, seed):
    path = case["path"]
    if path == "layer":
        return _prepare_layer(case, seed)
    T, H, E, k = case["T"], case["H"], case["E"], case["k"]
    rng = np.random.default_rng([seed, 2])
    gen = torch.Generator(device="cuda").manual_seed(seed)
    s = dict(case=case, k=k, x=_normal(gen, (T, H), 1.0, torch.bfloat16))
    if path == "dispatch":
        # this rank's routing, and the predicted tokens per expert that every rank sent
        bias = torch.from_numpy(_zipf_bias(rng, 1, E, case["zipf"])).cuda()
        logits = _normal(gen, (RANKS * T, E), 1.3, torch.float32) + bias
        chosen = logits.topk(k, dim=1).indices.to(torch.int32)
        s["idx"] = chosen[:T].contiguous()
        s["n_hat"] = torch.stack([torch.bincount(chosen[r * T:(r + 1) * T].flatten(), minlength=E)
                                  for r in range(RANKS)]).to(torch.int32)
        s["ws_plan"] = _empty((probe.lib().probe_plan_greedy_workspace_bytes(RANKS, E),), torch.uint8)
        s["slots"] = E + RANKS * 3
        s["ws_permute"] = _empty((max(probe.permute_workspace_bytes(T, E, k, s["slots"]), 256),), torch.uint8)
        s["permuted"] = _permute_out(T, k, H, s["slots"], True)
        return s
    s["gate"] = _normal(gen, (E, H), 0.02, torch.float32)
    s["bias"] = torch.from_numpy(_zipf_bias(rng, 1, E, 1.1)).cuda()
    s["out"] = _route_out(T, k, E, probs=True)
    if path == "residual":
        D = case["D"]
        s["w1"] = _normal(gen, (D, H), 1.5 / math.sqrt(H), torch.bfloat16)
        s["w2"] = _normal(gen, (E, D), 0.3 / math.sqrt(D), torch.float32)
        s["ws"] = _empty((probe.predict_topk_residual_workspace_bytes(T, H, E, k, D),), torch.uint8)
    else:
        s["ws"] = _empty((max(probe.route_topk_workspace_bytes(T, H, E, k), 256),), torch.uint8)
    return s


# ------------------------------------------------------------------ one pass

def _run_layer(s):
    c, x, k, tpg = s["case"], s["x"], s["k"], s["tpg"]
    routed, predicted, permuted = s["routed"], s["predicted"], s["permuted"]
    if c["fused"]:
        probe.route_predict_topk(x, s["gate"], s["bias"], s["gate_next"], s["bias_next"], tpg, k, True, out=routed,
                                 pred_out=predicted, workspace=s["ws_route"])
    else:
        probe.predict_topk(x, s["gate_next"], s["bias_next"], tpg, k, True, out=predicted, workspace=s["ws_route"])
        if c["grouped"]:
            probe.route_grouped(x, s["gate"], s["bias"], tpg, s["select_bias"], scoring="sigmoid", n_group=8,
                                topk_group=4, group_top=2, k=k, renormalize=True, routed_scale=2.5, out=routed,
                                workspace=s["ws_route"])
        else:
            probe.route_topk(x, s["gate"], s["bias"], tpg, k, True, out=routed, workspace=s["ws_route"])
    probe.permute(routed["idx"], s["plan"], x, out=permuted, workspace=s["ws_permute"], copy_rows=not c["gather"])
    if c["gather"]:
        probe.grouped_ffn_gather(x, permuted["row_pair"], k, permuted["slot_offsets"], s["weights"], out=s["y"],
                                 workspace=s["ws_ffn"])
    else:
        probe.grouped_ffn(permuted["xp"], permuted["slot_offsets"], s["weights"], out=s["y"], workspace=s["ws_ffn"])
    if c["shared"]:
        e = s["shared"]
        probe.grouped_ffn(x, e["offsets"], e["weights"], out=e["y"], workspace=e["ws"])
        probe.combine_shared(s["y"], permuted["pair_row"], routed["w"], e["y"], out=s["out"])
    else:
        probe.combine(s["y"], permuted["pair_row"], routed["w"], out=s["out"])
    # the expert counts are the histograms of the two idx, the permute outputs follow from idx and the plan
    return dict(out=s["out"], idx=routed["idx"], w=routed["w"], pred_idx=predicted["idx"], pred_w=predicted["w"])


def run(state):
    s, c = state, state["case"]
    path = c["path"]
    if path == "layer":
        if not c["graph"]:
            return _run_layer(s)
        s["graph"].replay()
        return s["result"]
    if path == "route":
        o = probe.route_topk(s["x"], s["gate"], s["bias"], None, s["k"], c["renorm"], want_probs=True, out=s["out"],
                             workspace=s["ws"])
        return dict(idx=o["idx"], w=o["w"], probs=o["probs"])
    if path == "residual":
        o = probe.predict_topk_residual(s["x"], s["gate"], s["bias"], None, s["w1"], s["w2"], s["k"], True,
                                        out=s["out"], workspace=s["ws"])
        return dict(idx=o["idx"], w=o["w"])
    greedy = probe.plan_greedy(s["n_hat"], c["E"] // RANKS, rank=0, max_replicas=3, budget=3, k_max=16, n0=64, g_num=1,
                               g_den=4, want_assignment=True, workspace=s["ws_plan"])
    sent = probe.plan_dispatch(greedy["n"], greedy["delta_in"], c["E"] // RANKS, 0)
    p = probe.permute(s["idx"], sent["plan"], s["x"], out=s["permuted"], workspace=s["ws_permute"])
    return dict(n=greedy["n"], moves=greedy["moves"], stats=greedy["stats"], rank_off=sent["rank_off"],
                slot_expert=sent["slot_expert"], slot_offsets=p["slot_offsets"], row_pair=p["row_pair"],
                pair_row=p["pair_row"], xp=p["xp"])


# ------------------------------------------------------------------ work and tolerance

def _rows_and_slots(c):
    """Local rows and active slots of a layer pass: counted on at most 1024 tokens whose logits have the spread that
    the gate gives them, and scaled up."""
    cfg = _config(c)
    if c["T"] == 0:
        return 0, 0
    rng = np.random.default_rng(7)
    t = min(c["T"], 1024)
    groups = min(cfg.G, t)
    bias = _zipf_bias(rng, groups, cfg.E, cfg.zipf_s)
    logits = rng.standard_normal((t, cfg.E)) * 0.02 * math.sqrt(cfg.H) + bias[np.arange(t) * groups // t]
    counts = np.bincount(np.argpartition(-logits, cfg.k - 1, axis=1)[:, :cfg.k].ravel(), minlength=cfg.E)
    plan = workload.build_plan(cfg, counts)
    rows, slots = 0.0, 0
    for e in range(cfg.E):
        i = slice(plan["rep_off"][e], plan["rep_off"][e + 1])
        weight, local = plan["rep_weight"][i], plan["rep_slot"][i] >= 0
        part = counts[e] * weight * local / weight.sum()
        rows += part.sum()
        slots += min(int((part > 0).sum()), int(counts[e]))
    return int(round(rows * c["T"] / t)), slots


def work(case):
    c, path = case, case["path"]
    T, H, E, k = c["T"], c["H"], c["E"], c["k"]
    gate = 2 * T * H * E
    if path == "route":
        return dict(bytes=2 * T * H + 4 * E * H + 4 * T * E + 8 * T * k, flops=gate)
    if path == "residual":
        D = c["D"]
        return dict(bytes=2 * T * H + 4 * E * H + 2 * D * H + 4 * E * D + 8 * T * k,
                    flops=gate + 2 * T * D * (H + E))
    if path == "dispatch":
        return dict(bytes=2 * T * H + 2 * T * k * H + 12 * T * k + 4 * RANKS * E * (RANKS + 1), flops=0)
    rows, slots = _rows_and_slots(c)
    F, per_gate = c["F"], (6 if c["gate"] == "packed" else 4) * E * H
    n_bytes = 2 * T * H + 2 * per_gate + 16 * T * k + slots * 6 * H * F + 2 * T * H
    flops = 2 * gate + 6 * rows * H * F
    if c["shared"]:
        n_bytes += 6 * H * F
        flops += 6 * T * H * F
    return dict(bytes=n_bytes, flops=flops)


def tolerance(case):
    if case["path"] == "dispatch":
        return "exact"                       # integers and copied rows
    if case["path"] != "layer":
        # fp32 sums over H terms: against the same in 64 bits, weights and probabilities are off by rel 1e-7 to 6e-7,
        # max 4e-6.  A token whose neighbouring logits differ by less than that may list them the other way round.
        return dict(rel=3e-6, max=3e-5, differ=2e-3)
    # bf16 activations, h and y rounded to bf16 between the GEMMs: rel 3e-3, max 2e-2 against 64 bits.  A near tie at
    # rank k that goes the other way puts another expert's row into one token's sum, hence the bound on elements.
    return dict(rel=1e-2, max=0.9, differ=2e-3)
