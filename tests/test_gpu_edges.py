"""GPU edge cases through the C ABI: empty and degenerate inputs, determinism, plan
invariance, the predictor identity, HIP-graph replay of the five-call sequence."""
import numpy as np
import pytest
import torch

from paper_2602_00509_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def probe():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2602_00509_amd import probe as p
    p.lib()
    return p


@pytest.fixture(scope="module")
def G():
    import gpu_util
    return gpu_util


def _layer(G, probe, cfg, batch=0):
    L = G.Layer(cfg, batch)
    r = probe.route_topk(L.d_x, L.d_wg, L.d_bias, L.tpg, cfg.k, True, want_probs=True)
    torch.cuda.synchronize()
    return L, r


def test_empty_batch(probe):
    print("case empty batch", flush=True)
    dev = "cuda"
    H, E, k, S, F = 64, 8, 2, 3, 64
    x = torch.empty((0, H), dtype=torch.bfloat16, device=dev)
    wg = torch.zeros((E, H), dtype=torch.float32, device=dev)
    r = probe.route_topk(x, wg, None, None, k, True, out=dict(counts=torch.full((E,), 7, dtype=torch.int32, device=dev)))
    assert r["idx"].shape == (0, k) and int(r["counts"].abs().sum()) == 0
    plan = probe.Plan(np.arange(E + 1), np.array([0, 1, 2, -1, -1, -1, -1, -1]), np.ones(E), S)
    p = probe.permute(r["idx"], plan, x)
    torch.cuda.synchronize()
    assert int(p["n_local"]) == 0 and p["slot_offsets"].tolist() == [0] * (S + 1) and p["slot_counts"].tolist() == [0] * S
    w13 = [torch.zeros((2 * F, H), dtype=torch.bfloat16, device=dev) for _ in range(S)]
    w2 = [torch.zeros((H, F), dtype=torch.bfloat16, device=dev) for _ in range(S)]
    y = probe.grouped_ffn(p["xp"], p["slot_offsets"], probe.WeightTable(w13, w2))
    out = probe.combine(y, p["pair_row"], r["w"])
    torch.cuda.synchronize()
    assert y.shape == (0, H) and out.shape == (0, H)


def test_all_remote_and_zero_weight_replica(oracle, probe, G):
    print("case all remote / zero weight", flush=True)
    cfg = wl.small_config(T=200, H=128, E=12, k=3, F=128, E_loc=4, n_rep=2, ep=3, chunk=0, cid=80)
    L, r = _layer(G, probe, cfg)
    E, S = cfg.E, cfg.S
    # every expert remote: no rows, pair_row all -1, combine gives zeros, FFN launches do nothing
    plan = probe.Plan(np.arange(E + 1), -np.ones(E), np.ones(E), S)
    p = probe.permute(r["idx"], plan, L.d_x)
    L.load_weights(np.arange(S) % E, probe)
    y = torch.full((cfg.N, cfg.H), float("nan"), dtype=torch.bfloat16, device="cuda")
    probe.grouped_ffn(p["xp"], p["slot_offsets"], L.weights, out=y)
    out = probe.combine(torch.zeros_like(y), p["pair_row"], r["w"])
    torch.cuda.synchronize()
    assert int(p["n_local"]) == 0 and bool((p["pair_row"] == -1).all()) and bool((p["row_pair"] == -1).all())
    assert bool(torch.isnan(y.float()).all()) and float(out.float().abs().max()) == 0.0
    # a zero-weight replica receives nothing; its partner takes everything
    g_idx = r["idx"].cpu().numpy()
    rep_off = np.r_[0, 2, np.arange(3, E + 2)]
    rep_slot = np.r_[0, 4, np.where(np.arange(1, E) < 4, np.arange(1, E), -1)]
    rep_weight = np.r_[0, 5, np.ones(E - 1, np.int64)]
    plan = probe.Plan(rep_off, rep_slot, rep_weight, S)
    p = probe.permute(r["idx"], plan, L.d_x)
    torch.cuda.synchronize()
    o = oracle.permute(g_idx, rep_off.astype(np.int32), rep_slot.astype(np.int32), rep_weight.astype(np.int32), S, L.x)
    assert int(p["slot_counts"][0]) == 0 and int(p["slot_counts"][4]) == int((g_idx == 0).sum())
    np.testing.assert_array_equal(p["pair_row"].cpu().numpy(), o["pair_row"])
    np.testing.assert_array_equal(p["row_pair"].cpu().numpy(), o["row_pair"])
    np.testing.assert_array_equal(p["slot_offsets"].cpu().numpy(), o["slot_offsets"])


@pytest.mark.parametrize("T,k,E,S,H", [(1, 1, 1, 1, 8), (1024, 1, 256, 64, 16), (1025, 1, 9, 65, 8), (341, 3, 130, 20, 24), (342, 3, 130, 20, 24),
                                       (1024, 8, 256, 1000, 72), (1025, 8, 33, 7, 8), (2048, 8, 64, 63, 8), (2049, 8, 64, 66, 8),
                                       (4096, 4, 8, 12, 8), (1639, 5, 200, 30, 40), (32768, 8, 128, 24, 8), (40, 7, 12, 30, 4104),
                                       (1024, 2, 16, 12, 2048), (1025, 2, 16, 12, 2048), (700, 1, 20, 12, 3000)])
def test_permute_on_both_sides_of_every_block_count(oracle, probe, G, T, k, E, S, H):
    """1, 2, 8, 9, 16, 17 and 256 blocks of 1024 pairs, tokens that straddle blocks, replicas with equal, unequal and no weight, remote
    experts, a replica list longer than the staged one, with the row copy (4 MB of x and a row more) and without: every output
    bit for bit the oracle's."""
    print("case permute T=%d k=%d E=%d S=%d" % (T, k, E, S), flush=True)
    rng = np.random.default_rng(T * k + E)
    popularity = rng.permutation(E)
    idx = np.minimum(rng.geometric(min(4.0 / E, 0.9), size=(T, k)) - 1, E - 1)
    idx = popularity[idx].astype(np.int32)
    reps = rng.integers(1, 4 if E < 256 else 20, E)                       # 256 experts: more entries than are staged
    rep_off = np.r_[0, np.cumsum(reps)].astype(np.int32)
    slots = np.full(rep_off[-1], -1, np.int32)
    local = rng.permutation(rep_off[-1])[:min(S, rep_off[-1])]            # a slot belongs to one replica
    slots[local] = rng.permutation(S)[:local.size]
    weight = rng.integers(0, 4, rep_off[-1]).astype(np.int32)
    weight[rep_off[:-1]] += 1                                              # every expert has some weight
    x = wl.f32_to_bf16_bits(rng.standard_normal((T, H)).astype(np.float32))
    o = oracle.permute(idx, rep_off, slots, weight, S, x)
    d_idx, d_x = torch.from_numpy(idx).cuda(), G.dev_bf16(x)
    plan = probe.Plan(rep_off, slots, weight, S)
    full = probe.permute(d_idx, plan, d_x)
    lean = probe.permute(d_idx, plan, d_x, copy_rows=False)
    torch.cuda.synchronize()
    n = o["n_local"]
    for got in (full, lean):
        assert int(got["n_local"].item()) == n
        for key in ("slot_counts", "slot_offsets", "pair_row", "row_pair"):
            np.testing.assert_array_equal(got[key].cpu().numpy(), o[key], err_msg=key)
    np.testing.assert_array_equal(G.bits_of(full["xp"])[:n], o["xp"][:n])


def test_topk_equals_all_experts_and_predictor_identity(oracle, probe, G):
    print("case k == E, predictor identity", flush=True)
    cfg = wl.small_config(T=77, H=64, E=8, k=8, F=64, E_loc=8, n_rep=0, ep=1, chunk=0, cid=81)
    L, r = _layer(G, probe, cfg)
    o = oracle.route_topk(L.x, L.wg, L.bias, L.tpg, cfg.k, True)
    G.check_route(r, o, cfg.k, True)
    assert bool((torch.sort(r["idx"], dim=1).values == torch.arange(8, device="cuda", dtype=torch.int32)).all())
    np.testing.assert_allclose(r["w"].sum(1).cpu().numpy(), 1.0, atol=1e-6)
    assert r["counts"].tolist() == [cfg.T] * 8
    # Sec. 4.2: at the zero-initialised residual the predictor is the cloned router
    pr = probe.predict_topk(L.d_x, L.d_wg, L.d_bias, L.tpg, cfg.k, True, want_probs=True)
    torch.cuda.synchronize()
    for key in ("idx", "w", "probs", "counts"):
        assert torch.equal(r[key], pr[key]), key


@pytest.mark.parametrize("T,H,E,k", [(150, 72, 20, 3), (300, 200, 130, 8), (64, 8, 5, 2), (129, 1000, 256, 8)])
def test_route_when_hidden_size_is_not_a_multiple_of_64(oracle, probe, G, T, H, E, k):
    """H % 8 == 0 is all the router asks for; these shapes take the kernel that zero-fills the K tail."""
    print("case route H=%d" % H, flush=True)
    rng = np.random.default_rng(H)
    x = wl.f32_to_bf16_bits(rng.standard_normal((T, H), dtype=np.float32))
    wg = (rng.standard_normal((E, H), dtype=np.float32) * np.float32(0.05))
    b = rng.standard_normal((2, E)).astype(np.float32)
    tpg = 100
    g = probe.route_topk(G.dev_bf16(x), torch.from_numpy(wg).cuda(), torch.from_numpy(b).cuda(), tpg, k, True,
                         want_probs=True)
    torch.cuda.synchronize()
    o = oracle.route_topk(x, wg, b, tpg, k, True)
    G.check_route(g, o, k, True)
    np.testing.assert_array_equal(g["counts"].cpu().numpy(), np.bincount(g["idx"].cpu().numpy().ravel(), minlength=E))


@pytest.mark.parametrize("T,H,E,k", [(1, 64, 16, 8), (16, 1000, 17, 3), (17, 8, 60, 6), (32, 4096, 9, 2), (33, 520, 130, 8),
                                     (65, 7168, 256, 8), (129, 1024, 128, 4), (513, 328, 16, 2), (9000, 192, 8, 2),
                                     (257, 512, 128, 8), (2049, 4104, 16, 2), (3100, 4096, 8, 2), (9001, 2880, 13, 3),
                                     (12001, 2048, 8, 2), (40003, 1024, 16, 2)])
def test_route_small_batches_and_small_gates(oracle, probe, G, T, H, E, k):
    """The kernel that goes from global memory to the matrix cores: one to eight token fragments per workgroup (by the batch, or
    by the gate where it has at most 16 experts), batches and gates on both sides of where it hands over to the tiled ones, expert counts that leave a partial fragment or
    partial 16-byte pieces; every token against the oracle, the packed gate bit for bit the fp32 one."""
    print("case small route T=%d H=%d E=%d" % (T, H, E), flush=True)
    rng = np.random.default_rng(T + E)
    x = wl.f32_to_bf16_bits(rng.standard_normal((T, H), dtype=np.float32))
    wg = (rng.standard_normal((E, H), dtype=np.float32) * np.float32(0.05))
    b = rng.standard_normal((2, E)).astype(np.float32)
    tpg = max(T // 2, 1)
    d_x, d_w, d_b = G.dev_bf16(x), torch.from_numpy(wg).cuda(), torch.from_numpy(b).cuda()
    g = probe.route_topk(d_x, d_w, d_b, tpg, k, True, want_probs=True)
    p = probe.route_topk(d_x, probe.PackedGate(d_w), d_b, tpg, k, True, want_probs=True)
    torch.cuda.synchronize()
    for key in ("idx", "w", "probs", "counts"):
        assert torch.equal(g[key], p[key]), key
    o = oracle.route_topk(x, wg, b, tpg, k, True)
    G.check_route(g, o, k, True)
    np.testing.assert_array_equal(g["counts"].cpu().numpy(), np.bincount(g["idx"].cpu().numpy().ravel(), minlength=E))
    if 2 * k <= E:   # both gates in one pass: the second is this one with its experts in reverse order
        r, q = probe.route_predict_topk(d_x, d_w, d_b, d_w.flip(0).contiguous(), d_b.flip(1).contiguous(), tpg, k, True)
        torch.cuda.synchronize()
        G.check_route(r, o, k, True)
        rev = oracle.route_topk(x, wg[::-1].copy(), b[:, ::-1].copy(), tpg, k, True)
        G.check_route(q, rev, k, True)


@pytest.mark.parametrize("T,H,E,k", [(1, 1024, 60, 5), (128, 1024, 64, 4), (129, 1024, 64, 4), (255, 512, 90, 3), (256, 2048, 128, 8),
                                     (257, 2048, 128, 8), (512, 1024, 256, 8), (513, 1024, 256, 8), (66, 2048, 7, 2),
                                     (2049, 1024, 128, 6), (3073, 1024, 64, 2), (6145, 512, 132, 4), (96, 4096, 60, 4), (97, 4096, 60, 4),
                                     (192, 4096, 126, 8), (193, 4096, 126, 8), (512, 2560, 250, 8), (513, 2560, 250, 8),
                                     (512, 1728, 250, 8)])
def test_route_topk_a_wave_or_sixteen_lanes_per_token(oracle, probe, G, T, H, E, k):
    """Both sides of the lines between a wave and sixteen lanes per token and between one and two tokens per row, alone and
    with two gates in one launch, one of them misaligned where E % 4 != 0; every token against the oracle."""
    print("case topk T=%d H=%d E=%d" % (T, H, E), flush=True)
    rng = np.random.default_rng(T + E)
    x = wl.f32_to_bf16_bits(rng.standard_normal((T, H), dtype=np.float32))
    wg = (rng.standard_normal((E, H), dtype=np.float32) * np.float32(0.05))
    b = rng.standard_normal((2, E)).astype(np.float32)
    tpg = max((T + 1) // 2, 1)
    d_x, d_w, d_b = G.dev_bf16(x), torch.from_numpy(wg).cuda(), torch.from_numpy(b).cuda()
    one = probe.route_topk(d_x, d_w, d_b, tpg, k, False, want_probs=True)
    r, q = probe.route_predict_topk(d_x, d_w, d_b, d_w.flip(0).contiguous(), d_b.flip(1).contiguous(), tpg, k, True,
                                    want_probs=True)
    torch.cuda.synchronize()
    o = oracle.route_topk(x, wg, b, tpg, k, True)
    rev = oracle.route_topk(x, wg[::-1].copy(), b[:, ::-1].copy(), tpg, k, True)
    G.check_route(one, oracle.route_topk(x, wg, b, tpg, k, False), k, False)
    for got, ora in ((r, o), (q, rev)):
        G.check_route(got, ora, k, True)
        np.testing.assert_allclose(got["probs"].cpu().numpy(), ora["probs"], rtol=0, atol=G.PROB_ATOL)
        np.testing.assert_array_equal(got["counts"].cpu().numpy(),
                                      np.bincount(got["idx"].cpu().numpy().ravel(), minlength=E))


@pytest.mark.parametrize("T,H,E,k", [
    (1000, 1024, 128, 8), (1025, 1024, 128, 8), (1000, 960, 128, 8),  # one k32 per wave: the most logits, too many, too short an H
    (384, 2880, 96, 4), (1300, 1088, 100, 4),                         # one and two; a last expert fragment of four
    (640, 2880, 96, 4), (640, 2880, 95, 4),                           # two: the emptiest column of experts, emptier
    (768, 2048, 128, 8), (769, 2048, 128, 8),                         # two: the most logits, too many
    (512, 4096, 128, 8), (513, 4096, 128, 8),                         # two and three
    (256, 4096, 224, 8), (257, 4096, 224, 8), (140, 2880, 256, 8)])   # two columns: two token blocks and three
def test_route_more_logits_without_lds(oracle, probe, G, T, H, E, k):
    """Either side of the lines up to which gates of more than 32768 logits go from global memory to the matrix cores: every token
    against the oracle, the packed gate bit for bit the fp32 one, a batch in the workspace of exactly its size, and under capture."""
    print("case more logits T=%d H=%d E=%d" % (T, H, E), flush=True)
    rng = np.random.default_rng(T + E)
    x = wl.f32_to_bf16_bits(rng.standard_normal((T, H), dtype=np.float32))
    wg = (rng.standard_normal((E, H), dtype=np.float32) * np.float32(0.05))
    d_x, d_w = G.dev_bf16(x), torch.from_numpy(wg).cuda()
    ws = torch.full((probe.route_topk_workspace_bytes(T, H, E, k),), 0xff, dtype=torch.uint8, device="cuda")
    g = probe.route_topk(d_x, d_w, None, None, k, True, want_probs=True, workspace=ws)
    p = probe.route_topk(d_x, probe.PackedGate(d_w), None, None, k, True, want_probs=True)
    torch.cuda.synchronize()
    for key in ("idx", "w", "probs", "counts"):
        assert torch.equal(g[key], p[key]), key
    o = oracle.route_topk(x, wg, None, T, k, True)
    G.check_route(g, o, k, True)
    np.testing.assert_allclose(g["probs"].cpu().numpy(), o["probs"], rtol=0, atol=G.PROB_ATOL)
    out = {key: torch.empty_like(g[key]) for key in ("idx", "w", "counts")}
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        probe.route_topk(d_x, d_w, None, None, k, True, out=out, workspace=ws)
    for _ in range(3):
        for key in out:
            out[key].zero_()
        graph.replay()
        torch.cuda.synchronize()
        for key in out:
            assert torch.equal(out[key], g[key]), key


def test_route_small_gate_on_more_token_blocks_than_65535(oracle, probe, G):
    """A gate of at most 16 experts takes 32 tokens per workgroup at any batch: more of them than the y and z dimensions of a
    launch can hold.  Every token bit for bit as in batches of a million, the last ones against the oracle."""
    T, H, E, k = 2 ** 21 + 45, 64, 8, 2
    g = torch.Generator(device="cuda").manual_seed(9)
    x = torch.randn((T, H), generator=g, device="cuda").to(torch.bfloat16)
    w = torch.randn((E, H), generator=g, device="cuda") * 0.2
    print("case small gate T=%d" % T, flush=True)
    r = probe.route_topk(x, w, None, None, k, True)
    torch.cuda.synchronize()
    assert int(r["counts"].sum()) == T * k
    for t0, t1 in ((0, 2 ** 20), (2 ** 20, 2 ** 21), (2 ** 21 - 10000, T)):
        part = probe.route_topk(x[t0:t1], w, None, None, k, True)
        for key in ("idx", "w"):
            assert torch.equal(part[key], r[key][t0:t1]), (key, t0)
    n = 200
    o = oracle.route_topk(x[-n:].view(torch.int16).cpu().numpy().view(np.uint16), w.cpu().numpy(), None, n, k, True)
    G.check_route({key: r[key][-n:] for key in ("idx", "w")}, o, k, True)


@pytest.mark.parametrize("T,H,E,k", [(8200, 256, 256, 8), (4100, 1024, 200, 6), (2049, 128, 130, 4)])
def test_route_on_256_token_tiles_with_a_ragged_last_tile(oracle, probe, G, T, H, E, k):
    """Large batches take the 256-token tile of the gate GEMM; T is not a multiple of the tile, E not
    always one of 128, and the K range of one split is as short as one step."""
    print("case route T=%d H=%d E=%d" % (T, H, E), flush=True)
    rng = np.random.default_rng(T)
    x = wl.f32_to_bf16_bits(rng.standard_normal((T, H), dtype=np.float32))
    wg = (rng.standard_normal((E, H), dtype=np.float32) * np.float32(0.05))
    b = rng.standard_normal((3, E)).astype(np.float32)
    tpg = 1500
    g = probe.route_topk(G.dev_bf16(x), torch.from_numpy(wg).cuda(), torch.from_numpy(b).cuda(), tpg, k, True,
                         want_probs=True)
    torch.cuda.synchronize()
    o = oracle.route_topk(x, wg, b, tpg, k, True)
    G.check_route(g, o, k, True)
    np.testing.assert_allclose(g["probs"].cpu().numpy(), o["probs"], rtol=0, atol=G.PROB_ATOL)
    np.testing.assert_array_equal(g["counts"].cpu().numpy(), np.bincount(g["idx"].cpu().numpy().ravel(), minlength=E))


@pytest.mark.parametrize("T,H,E,k", [(600, 1024, 128, 4), (2049, 320, 130, 4), (5500, 512, 256, 8), (9001, 1024, 130, 6),
                                     (16385, 512, 130, 2), (16129, 2048, 130, 2)])
def test_route_tile_heights_and_slices(oracle, probe, G, T, H, E, k):
    """128- and 256-token tiles with ragged last tiles and slices, sums by k-step and in the accumulators; a sample of the tokens and all
    of the last tile's against the oracle, all probabilities against the product in 64 bits."""
    print("case tiles T=%d H=%d E=%d" % (T, H, E), flush=True)
    rng = np.random.default_rng(T + E)
    x = wl.f32_to_bf16_bits(rng.standard_normal((T, H), dtype=np.float32))
    wg = (rng.standard_normal((E, H), dtype=np.float32) * np.float32(0.05))
    b = rng.standard_normal((2, E)).astype(np.float32)
    tpg = (T + 1) // 2
    d_x, d_w, d_b = G.dev_bf16(x), torch.from_numpy(wg).cuda(), torch.from_numpy(b).cuda()
    g = probe.route_topk(d_x, d_w, d_b, tpg, k, True, want_probs=True)
    torch.cuda.synchronize()
    tokens = np.unique(np.concatenate([rng.choice(T, 300, replace=False), np.arange(T - min(T, 256), T)]))
    o = oracle.route_topk(x[tokens], wg, G.gather_bias(b, tpg, tokens), 1, k, True)
    sub = {key: g[key][torch.from_numpy(tokens).cuda()] for key in ("idx", "w", "probs")}
    G.check_route(sub, o, k, True, tokens=None)
    np.testing.assert_array_equal(g["counts"].cpu().numpy(), np.bincount(g["idx"].cpu().numpy().ravel(), minlength=E))
    logits = d_x.double() @ d_w.double().t() + d_b.double()[torch.arange(T, device="cuda") // tpg]
    np.testing.assert_allclose(g["probs"].cpu().numpy(), torch.softmax(logits, 1).cpu().numpy(), rtol=0, atol=G.PROB_ATOL)


def test_determinism_and_plan_invariance(oracle, probe, G):
    """Two runs are bit-identical; with every replica local, any plan gives the same layer output."""
    print("case determinism / plan invariance", flush=True)
    cfg = wl.small_config(T=900, H=256, E=6, k=2, F=320, E_loc=6, n_rep=2, ep=1, chunk=256, cid=82)
    L, r = _layer(G, probe, cfg)
    counts = r["counts"].cpu().numpy()

    def run(plan):
        d_plan = probe.Plan(plan["rep_off"], plan["rep_slot"], plan["rep_weight"], plan["num_slots"])
        p = probe.permute(r["idx"], d_plan, L.d_x)
        L.load_weights(plan["slot_expert"], probe)
        y = torch.zeros((cfg.N, cfg.H), dtype=torch.bfloat16, device="cuda")
        probe.grouped_ffn(p["xp"], p["slot_offsets"], L.weights, out=y)
        out = probe.combine(y, p["pair_row"], r["w"])
        torch.cuda.synchronize()
        return p, y, out

    base = wl.no_replica_plan(cfg)
    rep = wl.build_plan(cfg, counts)
    p0, y0, out0 = run(base)
    p0b, y0b, out0b = run(base)
    assert torch.equal(out0, out0b) and torch.equal(y0, y0b) and torch.equal(p0["row_pair"], p0b["row_pair"])
    p1, y1, out1 = run(rep)
    assert int(p1["n_local"]) == cfg.N == int(p0["n_local"])
    assert bool((p1["slot_counts"][cfg.E_loc:] > 0).all())
    # neither plan's call cuts a contraction or takes items of few rows: a row's sum does not depend on where the row sits
    assert torch.equal(out0, out1)


def test_predictor_overlap_matches_oracle(oracle, probe, G):
    """Top-k overlap of the lookahead predictor against the next layer's router: the GPU's
    integer metric equals the oracle's on unambiguous tokens; drift 0 gives overlap 1."""
    print("case predictor overlap", flush=True)
    cfg = wl.small_config(T=512, H=256, E=64, k=8, F=64, E_loc=16, n_rep=0, ep=4, chunk=128, cid=83)
    h = wl.activations(cfg, 0)
    wn, bn = wl.gate_weights(cfg, 1), wl.zipf_bias(cfg, 0, 1)
    d_w, d_b = torch.from_numpy(wn).cuda(), torch.from_numpy(bn).cuda()
    tpg = wl.tokens_per_group(cfg)
    for alpha, lo, hi in ((0.0, 1.0, 1.0), (0.2, 0.6, 1.0), (0.5, 0.4, 0.95)):
        h2 = wl.drifted_activations(cfg, h, alpha, 0) if alpha > 0 else h
        pred = probe.predict_topk(G.dev_bf16(h), d_w, d_b, tpg, cfg.k, True)
        true = probe.route_topk(G.dev_bf16(h2), d_w, d_b, tpg, cfg.k, True)
        torch.cuda.synchronize()
        g_ov = oracle.topk_overlap(pred["idx"].cpu().numpy(), true["idx"].cpu().numpy())
        o_pred = oracle.predict_topk(h, wn, bn, tpg, cfg.k, True)
        o_true = oracle.route_topk(h2, wn, bn, tpg, cfg.k, True)
        o_ov = oracle.topk_overlap(o_pred["idx"], o_true["idx"])
        amb = G.ambiguous_tokens(o_pred["logits"], cfg.k) | G.ambiguous_tokens(o_true["logits"], cfg.k)
        assert abs(g_ov - o_ov) <= amb.sum() * cfg.k / (cfg.T * cfg.k) + 1e-12
        assert lo <= g_ov <= hi, (alpha, g_ov)


def test_graph_replay(oracle, probe, G):
    """The five calls record into a HIP graph (no allocation, no host sync, no memset nodes);
    every replay, with eager work in between, reproduces the eager results."""
    print("case graph replay", flush=True)
    cfg = wl.small_config(T=300, H=128, E=16, k=4, F=128, E_loc=8, n_rep=2, ep=2, chunk=0, cid=84)
    L, r0 = _layer(G, probe, cfg)
    plan = wl.build_plan(cfg, r0["counts"].cpu().numpy())
    d_plan = probe.Plan(plan["rep_off"], plan["rep_slot"], plan["rep_weight"], plan["num_slots"])
    L.load_weights(plan["slot_expert"], probe)
    T, H, E, k, S, F, N = cfg.T, cfg.H, cfg.E, cfg.k, cfg.S, cfg.F, cfg.N
    dev = "cuda"
    mk = lambda shape, dt: torch.zeros(shape, dtype=dt, device=dev)
    bufs = dict(r=dict(idx=mk((T, k), torch.int32), w=mk((T, k), torch.float32), counts=mk((E,), torch.int32)),
                pr=dict(idx=mk((T, k), torch.int32), w=mk((T, k), torch.float32), counts=mk((E,), torch.int32)),
                p=dict(slot_counts=mk((S,), torch.int32), slot_offsets=mk((S + 1,), torch.int32),
                       row_pair=mk((N,), torch.int32), pair_row=mk((T, k), torch.int32),
                       xp=mk((N, H), torch.bfloat16), n_local=mk((1,), torch.int32)),
                y=mk((N, H), torch.bfloat16), out=mk((T, H), torch.bfloat16))
    ws_r = torch.empty(probe.route_topk_workspace_bytes(T, H, E, k), dtype=torch.uint8, device=dev)
    ws_p = torch.empty(max(256, probe.permute_workspace_bytes(T, E, k, S)), dtype=torch.uint8, device=dev)
    ws_f = torch.empty(probe.grouped_ffn_workspace_bytes(S, H, F, N), dtype=torch.uint8, device=dev)

    def step():
        probe.predict_topk(L.d_x, L.d_wg, L.d_bias, L.tpg, k, True, out=bufs["pr"], workspace=ws_r)
        probe.route_topk(L.d_x, L.d_wg, L.d_bias, L.tpg, k, True, out=bufs["r"], workspace=ws_r)
        probe.permute(bufs["r"]["idx"], d_plan, L.d_x, out=bufs["p"], workspace=ws_p)
        probe.grouped_ffn(bufs["p"]["xp"], bufs["p"]["slot_offsets"], L.weights, out=bufs["y"], workspace=ws_f)
        probe.combine(bufs["y"], bufs["p"]["pair_row"], bufs["r"]["w"], out=bufs["out"])

    step()                                   # eager (also the one-time LDS opt-in of the FFN kernels)
    torch.cuda.synchronize()
    ref = {k_: bufs[k_].clone() for k_ in ("y", "out")}
    ref_idx, ref_rows = bufs["r"]["idx"].clone(), bufs["p"]["row_pair"].clone()
    nl = int(bufs["p"]["n_local"])
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            step()
    torch.cuda.synchronize()
    for i in range(3):
        for t in (bufs["y"], bufs["out"], bufs["r"]["idx"], bufs["p"]["row_pair"]):
            t.fill_(0)                       # eager work between replays
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(bufs["r"]["idx"], ref_idx) and torch.equal(bufs["p"]["row_pair"], ref_rows), i
        assert torch.equal(bufs["y"][:nl], ref["y"][:nl]) and torch.equal(bufs["out"], ref["out"]), i


def test_ffn_every_way_a_slot_is_cut_into_tiles(oracle, probe, G):
    """Slot sizes on both sides of every tile-height boundary of the standard cut, empty slots in between, so many that no other cut
    is taken: every output element against the oracle, and every slot's tiles."""
    sizes = [0, 1, 63, 64, 65, 128, 129, 191, 192, 193, 255, 256, 257, 0, 300, 320, 321, 384, 385, 449,
             512, 513, 576, 577, 640, 641, 700, 768 + 1, 768 + 65, 768 + 129, 768 + 192, 768 + 193, 1024 + 130, 7]
    print("case every cut", flush=True)
    table = _tall_tiles(oracle, probe, G, sizes, 448, 512, sum(sizes) + 9, 0, n_weights=4)
    assert table[1:3] == (False, True)
    assert _slots_in_order(table, sizes, 192)


def _ffn_against_oracle(oracle, probe, G, cfg, sizes, n_weights, seed, extra_rows=9, workspace=None):
    """probe_grouped_ffn on slots of the given sizes, every output element against the oracle."""
    S = len(sizes)
    so = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(so[-1])
    ws = wl.expert_weights_many(cfg, list(range(n_weights)))
    rng = np.random.default_rng(seed)
    xp = wl.f32_to_bf16_bits(rng.standard_normal((n + extra_rows, cfg.H)).astype(np.float32))
    d_w = {e: (G.dev_bf16(ws[e][0]), G.dev_bf16(ws[e][1])) for e in range(n_weights)}
    tab = probe.WeightTable([d_w[s % n_weights][0] for s in range(S)], [d_w[s % n_weights][1] for s in range(S)])
    y = torch.full((n + extra_rows, cfg.H), 7.0, dtype=torch.bfloat16, device="cuda")
    probe.grouped_ffn(G.dev_bf16(xp), torch.from_numpy(so).cuda(), tab, out=y, workspace=workspace)
    torch.cuda.synchronize()
    ref = oracle.grouped_ffn(xp, so, [ws[s % n_weights][0] for s in range(S)], [ws[s % n_weights][1] for s in range(S)])
    got = G.f64_of(y)
    err = G.rel_err(got[:n], ref)
    assert err < G.BF16_RTOL, err
    assert (got[n:] == 7.0).all()          # rows past the last slot are not written
    return err


def _tile_table(ws, F, cap):
    """What the schedule kernel left in a call's workspace: tiles, whether gemm1 and gemm2 take narrow column blocks, and a row
    (first row, rows to the slot's end, height, slot) per tile."""
    at = (cap * F * 2 + 255) // 256 * 256
    head = ws[at:at + 128].cpu().numpy().view(np.int32)
    n = int(head[0])
    return n, bool(head[1]), bool(head[2]), ws[at + 128:at + 128 + 32 * n].cpu().numpy().view(np.int32).reshape(n, 8)[:, :4]


def _cut(m, cap):
    """Heights of a slot's tiles, first row first: as many of 320 rows as leave whole ones of 256 and no rest, or one short tile at the end;
    with a cap tiles of that height and a shorter one."""
    u = (m + 63) // 64
    if cap:
        return [cap] * (64 * u // cap) + ([64 * u % cap] if 64 * u % cap else [])
    for a in range(u // 5, -1, -1):
        if (u - 5 * a) % 4 == 0:
            return [320] * a + [256] * ((u - 5 * a) // 4)
    return {1: [64], 2: [128], 3: [192], 6: [256, 128], 7: [320, 128], 11: [320, 256, 128]}[u]


def _tall_tiles(oracle, probe, G, sizes, H, F, cap, height, n_weights=3):
    """One call on the tall tiles, every output element against the oracle.  Asserts that each slot is cut as `height` says (0 = the standard
    cut) and returns the tile table."""
    assert cap > 64 * len(sizes) and (cap // 64 + len(sizes)) * (F // 64) > 512        # past the decode schedule
    cfg = wl.small_config(T=64, H=H, E=4, k=2, F=F, cid=120)
    ws = torch.zeros(probe.grouped_ffn_workspace_bytes(len(sizes), H, F, cap), dtype=torch.uint8, device="cuda")
    _ffn_against_oracle(oracle, probe, G, cfg, sizes, n_weights, seed=H + F, extra_rows=cap - sum(sizes), workspace=ws)
    table = _tile_table(ws, F, cap)
    _check_cut(table, sizes, height)
    return table


def _check_cut(table, sizes, height):
    tiles = table[3]
    first = np.r_[0, np.cumsum(sizes)]
    for q, m in enumerate(sizes):
        mine = tiles[tiles[:, 3] == q]
        mine = mine[np.argsort(mine[:, 0])]
        want = _cut(m, height)
        assert mine[:, 2].tolist() == want, (q, m, mine)
        at = np.cumsum([0] + want[:-1]) if want else np.zeros(0, int)
        assert mine[:, 0].tolist() == (first[q] + at).tolist() and mine[:, 1].tolist() == (m - at).tolist()
    assert table[0] == sum(len(_cut(m, height)) for m in sizes)


def _slots_in_order(table, sizes, single):
    """Slots of more than `single` rows stand by descending rows, each one's tiles together but for single short tiles in between."""
    several = [int(q) for q in table[3][:, 3] if sizes[q] > single]
    runs = [q for i, q in enumerate(several) if i == 0 or q != several[i - 1]]
    return runs == sorted((q for q, m in enumerate(sizes) if m > single), key=lambda q: (-sizes[q], q))


def test_ffn_decode_schedule_every_element(oracle, probe, G):
    """A decode-sized row space (at most 64 rows per slot on average): the call takes the schedule of skinny
    tiles (64 rows x 64 h columns / 128 output columns).  Slot sizes around the 64-row tile boundary, empty
    slots, slots of several row tiles; F and H that leave a partial last column block."""
    for (H, F, cid) in ((192, 320, 96), (128, 64, 97), (256, 448, 98)):
        cfg = wl.small_config(T=64, H=H, E=4, k=2, F=F, cid=cid)
        sizes = [0, 1, 40, 63, 64, 65, 0, 130, 17, 33, 5, 0, 90, 2]
        assert sum(sizes) + 9 <= 64 * len(sizes)
        print("case decode schedule H=%d F=%d" % (H, F), flush=True)
        _ffn_against_oracle(oracle, probe, G, cfg, sizes, 4, seed=H + F)


@pytest.mark.parametrize("sizes,H,F", [([1], 4096, 4160), ([75], 6016, 192), ([1, 0, 0, 2], 320, 5120), ([64, 65], 4480, 256),
                                       ([300], 4096, 576), ([0, 17, 0], 8192, 64)])
def test_ffn_few_tiles_every_element(oracle, probe, G, sizes, H, F):
    """So few tiles that the contraction is cut into pieces whose sums a second kernel adds: one, some or all
    of the two GEMMs, pieces of unequal length, a last column block that is not full."""
    cfg = wl.small_config(T=64, H=H, E=4, k=2, F=F, cid=100)
    print("case few tiles", sizes, H, F, flush=True)
    _ffn_against_oracle(oracle, probe, G, cfg, sizes, len(sizes), seed=H + F, extra_rows=0 if sizes == [1] else 9)


@pytest.mark.parametrize("sizes,H,F", [([1, 0, 0, 2], 4160, 320), ([75], 4096, 192), ([2, 0, 5], 320, 5120)])
def test_ffn_few_tiles_gathered_on_load_and_in_a_graph(oracle, probe, G, sizes, H, F):
    """Pieces of K with the activation rows gathered on load (two rows per token, out of order): bit for bit the call on the
    gathered copy, every element against the oracle; recorded once and replayed on other rows, with eager calls between."""
    cfg = wl.small_config(T=64, H=H, E=4, k=2, F=F, cid=104)
    S, n, k = len(sizes), sum(sizes), 2
    rng = np.random.default_rng(n + H)
    so = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    T = n // 2 + 3
    pairs = np.full(n + 5, -1, np.int32)
    pairs[:n] = rng.permutation(T * k)[:n]
    ws = wl.expert_weights_many(cfg, list(range(S)))
    tab = probe.WeightTable([G.dev_bf16(w[0]) for w in ws], [G.dev_bf16(w[1]) for w in ws])
    rows = lambda: wl.f32_to_bf16_bits(rng.standard_normal((T, H)).astype(np.float32))
    x = rows()
    d_x, d_so, d_pairs = G.dev_bf16(x), torch.from_numpy(so).cuda(), torch.from_numpy(pairs).cuda()
    y = torch.full((n + 5, H), 7.0, dtype=torch.bfloat16, device="cuda")
    work = torch.empty(probe.grouped_ffn_workspace_bytes(S, H, F, n + 5), dtype=torch.uint8, device="cuda")
    call = lambda out: probe.grouped_ffn_gather(d_x, d_pairs, k, d_so, tab, out=out, workspace=work)
    print("case gather few tiles", sizes, H, F, flush=True)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call(y)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            call(y)
    torch.cuda.current_stream().wait_stream(side)
    for replay in range(3):
        if replay:
            x = rows()
            d_x.copy_(G.dev_bf16(x))
        xp = np.zeros((n + 5, H), np.uint16)
        xp[:n] = x[pairs[:n] // k]
        copied = torch.full_like(y, 7.0)
        probe.grouped_ffn(G.dev_bf16(xp), d_so, tab, out=copied)
        y.fill_(7.0)
        work.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, copied), replay
        ref = oracle.grouped_ffn(xp, so, [w[0] for w in ws], [w[1] for w in ws])
        assert G.rel_err(G.f64_of(y)[:n], ref) < G.BF16_RTOL
        assert (y[n:] == 7.0).all()


@pytest.mark.parametrize("sizes,H,F", [([1, 0, 0, 2], 4096, 2112), ([3], 4160, 3136), ([64, 65], 4096, 2112), ([0, 1], 320, 14336),
                                       ([2, 3], 2048, 4160), ([64], 1024, 4160), ([9, 0, 1, 30], 4224, 1984), ([75], 7168, 2048),
                                       ([1, 0, 0, 2], 4096, 1600), ([64, 65], 4096, 1600), ([9, 0, 1, 30], 4224, 1472),
                                       ([1] * 8, 4096, 1536), ([32], 1024, 4160), ([1, 2], 4096, 8192),
                                       ([1] * 9, 1024, 2560), ([1] * 10, 1024, 2560), ([64, 64], 2880, 2880), ([64] * 6, 1024, 2880),
                                       ([30] * 6, 1024, 2880), ([31] * 6, 1024, 2880), ([64, 65], 1024, 2880), ([64], 2048, 2048),
                                       ([64], 2176, 2048), ([64, 64], 2048, 2496), ([64, 64], 2048, 2560)])
def test_ffn_second_contraction_cut_repeats_bit_for_bit(oracle, probe, G, sizes, H, F):
    """gemm2 in pieces that the last workgroup of an item adds (32 to 128 k-steps in two to five pieces; one row, full tiles; 72
    items of one row and 46 of 64 rows, the most there are; 30 rows in each of 48 items, 64 rows in 16 items of 32 k-steps and in
    32 of 40), in pieces that the adding kernel adds (fourteen of one row, four of 64 rows), and not cut (31 k-steps and fewer; 80
    items of one row, 48 of 64 rows, 31 rows in each of 48 items, 64 rows in 17 items of 32 k-steps and in 32 of 39).  Every element
    against the oracle; workspaces full of zeros, ones and noise and repeated calls give the same bits."""
    cfg = wl.small_config(T=64, H=H, E=4, k=2, F=F, cid=104)
    print("case last adds", sizes, H, F, flush=True)
    _ffn_against_oracle(oracle, probe, G, cfg, sizes, 2, seed=H + F, extra_rows=0)
    n, S = sum(sizes), len(sizes)
    gen = torch.Generator(device="cuda").manual_seed(F)
    x = torch.randn((n, H), generator=gen, device="cuda").to(torch.bfloat16)
    w = (torch.randn((2 * F, H), generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16),
         torch.randn((H, F), generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16))
    tab = probe.WeightTable([w[0]] * S, [w[1]] * S)
    so = torch.from_numpy(np.r_[0, np.cumsum(sizes)].astype(np.int32)).cuda()
    need = probe.grouped_ffn_workspace_bytes(S, H, F, n)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    ys = []
    for fill in (0, 255, None, 127):
        if fill is None:
            ws.random_(0, 256, generator=gen)
        else:
            ws.fill_(fill)
        for _ in range(3):
            ys.append(probe.grouped_ffn(x, so, tab, workspace=ws))
    torch.cuda.synchronize()
    assert all(torch.equal(ys[0], y) for y in ys[1:])


@pytest.mark.parametrize("n,H,F", [
    (13, 2560, 1280),     # 260 items of either GEMM: 19 of 20 column blocks are halved
    (8, 6016, 3008),      # 376 of either GEMM: the most of a single round
    (29, 1664, 832),      # 377 of either: not
    (12, 3456, 1728),     # 324 of either, gemm2 of 27 k-steps
    (11, 3840, 1728),     # 330 of gemm2, of 27 k-steps: not
    (13, 2880, 2624),     # 299 of gemm2, whose last block has 64 columns; 533 of gemm1: a last round of 21
    (16, 896, 1280),      # 320 of gemm1, of 14 k-steps: not
    (16, 2048, 2432),     # 608 of gemm1: the most of a second round; 256 of gemm2: one to a CU
    (14, 2432, 2816),     # 616 of gemm1: not
    (257, 64, 64)])       # one block of columns each, of one k-step
def test_ffn_decode_schedule_halves_blocks(oracle, probe, G, n, H, F):
    """Decode schedule: numbers of items at the limits between which column blocks are halved; every output element against the
    oracle, and the rows gathered on load bit for bit the same."""
    cfg = wl.small_config(T=64, H=H, E=4, k=2, F=F, cid=107)
    sizes = [1 + 7 * i % 5 for i in range(n)]
    sizes[n // 2] = 64
    print("case halves", n, H, F, flush=True)
    _ffn_against_oracle(oracle, probe, G, cfg, sizes, 3, seed=H + F)
    gen = torch.Generator(device="cuda").manual_seed(F)
    rows = sum(sizes)
    x = torch.randn((rows + 5, H), generator=gen, device="cuda").to(torch.bfloat16)
    w = (torch.randn((2 * F, H), generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16),
         torch.randn((H, F), generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16))
    tab = probe.WeightTable([w[0]] * n, [w[1]] * n)
    so = torch.from_numpy(np.r_[0, np.cumsum(sizes)].astype(np.int32)).cuda()
    order = torch.randperm(rows + 5, device="cuda", generator=gen).to(torch.int32)
    plain = probe.grouped_ffn(x[order.long()].contiguous(), so, tab)
    gathered = probe.grouped_ffn_gather(x, order, 1, so, tab)
    torch.cuda.synchronize()
    assert torch.equal(plain[:rows], gathered[:rows])


@pytest.mark.parametrize("n,H,F", [
    (13, 2560, 1280),     # 260 items of either GEMM
    (14, 4096, 1536),     # 336 of gemm1
    (15, 3072, 2560),     # 360 of gemm2; 600 of gemm1, of up to 32 rows per tile
    (13, 2880, 2624),     # 299 of gemm2; 533 of gemm1
    (17, 2048, 2048)])    # 544 of gemm1; 272 of gemm2, of 32 k-steps
def test_ffn_bits_of_a_row_do_not_follow_the_number_of_tiles(probe, n, H, F):
    """Decode schedule, no contraction cut: a row has the same bits in a call whose column blocks are halved to fill the CUs and in calls
    of fewer slots, whose blocks are whole."""
    print("case bits of a row", n, H, F, flush=True)
    sizes = [17 + 5 * i % 29 for i in range(n)]     # more rows than the items of few rows take
    gen = torch.Generator(device="cuda").manual_seed(n + H)
    x = torch.randn((sum(sizes), H), generator=gen, device="cuda").to(torch.bfloat16)
    w13 = [torch.randn((2 * F, H), generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16) for _ in range(3)]
    w2 = [torch.randn((H, F), generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16) for _ in range(3)]
    up = lambda b: (b + 255) // 256 * 256

    def call(lo, hi):
        rows = sum(sizes[lo:hi])
        first = sum(sizes[:lo])
        so = torch.from_numpy(np.r_[0, np.cumsum(sizes[lo:hi])].astype(np.int32)).cuda()
        tab = probe.WeightTable([w13[i % 3] for i in range(lo, hi)], [w2[i % 3] for i in range(lo, hi)])
        ws = torch.empty(up(rows * F * 2) + up(128 + 32 * (rows // 64 + hi - lo)), dtype=torch.uint8, device="cuda")  # no room for pieces
        return probe.grouped_ffn(x[first:first + rows].contiguous(), so, tab, workspace=ws)

    few = 256 // max(F // 64, (H + 127) // 128)     # slots that make one item per CU at most
    whole = call(0, n)
    parts = torch.cat([call(lo, min(lo + few, n)) for lo in range(0, n, few)])
    torch.cuda.synchronize()
    assert torch.equal(whole, parts)


@pytest.mark.parametrize("sizes,H,F", [
    ([16, 1, 0, 9], 64, 64),          # two steps of 32 for eight waves
    ([16, 3], 1088, 2048),            # 64 items of gemm1, 34 steps of 32: six waves of five, one of four
    ([17, 3], 1088, 2048),            # a row too many
    ([3, 16], 2048, 2112),            # 66 items of gemm1: too many; 32 of gemm2, of 33 k-steps
    ([4, 0, 4, 4, 4, 4], 1024, 1280), # 100 items of gemm1, of 16 k-steps, up to four rows
    ([4, 5, 4, 4, 4], 1024, 1280),    # a row too many
    ([4, 1, 2, 4], 1152, 2048),       # 128 items of gemm1
    ([2, 1, 4], 960, 2112),           # 99 items of gemm1, of 15 k-steps: neither
    ([3] + [0] * 127, 320, 192),      # the most slots that every wave scans for itself
    ([3] + [0] * 128, 320, 192)])     # one more: not
def test_ffn_few_rows_in_every_slot(oracle, probe, G, sizes, H, F):
    """Either side of the lines up to which items of few rows are a quarter as wide and stream straight to registers: every output
    element against the oracle, and the rows gathered on load bit for bit the same."""
    cfg = wl.small_config(T=64, H=H, E=4, k=2, F=F, cid=111)
    print("case few rows", len(sizes), H, F, flush=True)
    _ffn_against_oracle(oracle, probe, G, cfg, sizes, 3, seed=H + F)
    n, rows = len(sizes), sum(sizes)
    gen = torch.Generator(device="cuda").manual_seed(F)
    x = torch.randn((rows + 5, H), generator=gen, device="cuda").to(torch.bfloat16)
    w = (torch.randn((2 * F, H), generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16),
         torch.randn((H, F), generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16))
    tab = probe.WeightTable([w[0]] * n, [w[1]] * n)
    so = torch.from_numpy(np.r_[0, np.cumsum(sizes)].astype(np.int32)).cuda()
    order = torch.randperm(rows + 5, device="cuda", generator=gen).to(torch.int32)
    plain = probe.grouped_ffn(x[order.long()].contiguous(), so, tab)
    gathered = probe.grouped_ffn_gather(x, order, 1, so, tab)
    torch.cuda.synchronize()
    assert torch.equal(plain[:rows], gathered[:rows])


@pytest.mark.parametrize("S,H,F,rows", [(40, 1152, 2496, 40), (40, 1088, 2496, 64), (27, 1152, 2560, 52), (27, 1088, 2560, 64),
                                        (16, 1152, 4096, 64), (16, 128, 4096, 64)])
def test_ffn_either_side_of_the_decode_schedule(oracle, probe, G, S, H, F, rows):
    """The last capacity that takes the decode schedule, which leaves no tile table, and the first that takes tall tiles, with 1560, 1080 and
    1024 column blocks of all slots, and H on either side of the line from which more blocks count: every output element of both
    against the oracle."""
    cfg = wl.small_config(T=64, H=H, E=4, k=2, F=F, cid=109)
    sizes = [(5 * i) % 17 for i in range(S)]
    sizes[3] = 70
    for cap in (rows * S, rows * S + 1):
        print("case either side", S, H, F, cap, flush=True)
        ws = torch.full((probe.grouped_ffn_workspace_bytes(S, H, F, cap),), 0xff, dtype=torch.uint8, device="cuda")
        _ffn_against_oracle(oracle, probe, G, cfg, sizes, 2, seed=F, extra_rows=cap - sum(sizes), workspace=ws)
        at = (cap * F * 2 + 255) // 256 * 256
        assert (int(ws[at:at + 4].cpu().numpy().view(np.int32)[0]) > 0) == (cap > rows * S)


def test_ffn_contraction_is_not_cut_where_every_slot_can_hold_rows(oracle, probe, G):
    """At 40 rows of capacity per slot no adding kernel is launched although one slot alone holds rows: the call gives the
    same bits with and without room for partial sums.  Every element against the oracle."""
    cfg = wl.small_config(T=64, H=4096, E=4, k=2, F=1408, cid=103)
    S, cap, n = 12, 480, 3
    w13, w2 = wl.expert_weights_many(cfg, [0])[0]
    d13, d2 = G.dev_bf16(w13), G.dev_bf16(w2)
    tab = probe.WeightTable([d13] * S, [d2] * S)
    x = np.zeros((cap, cfg.H), np.uint16)
    x[:n] = wl.f32_to_bf16_bits(np.random.default_rng(4).standard_normal((n, cfg.H)).astype(np.float32))
    so = torch.tensor([0] * 5 + [n] * (S - 4), dtype=torch.int32, device="cuda")
    need = probe.grouped_ffn_workspace_bytes(S, cfg.H, cfg.F, cap)
    print("case no cut", S, cap, flush=True)
    ys = [probe.grouped_ffn(G.dev_bf16(x), so, tab, workspace=torch.empty(b, dtype=torch.uint8, device="cuda"))[:n]
          for b in (need, need - (8 << 20))]
    torch.cuda.synchronize()
    assert torch.equal(ys[0], ys[1])
    off = np.array([0] * 5 + [n] * (S - 4), np.int32)
    ref = oracle.grouped_ffn(x[:n], off, [w13] * S, [w2] * S)
    assert G.rel_err(G.f64_of(ys[0]), ref) < G.BF16_RTOL


@pytest.mark.parametrize("sizes,H,F,height,tall,by_height", [
    # every height; 14 tall tiles in 8 narrow column blocks of gemm1, 33 tiles
    ([384, 190, 130, 30, 64, 30, 321, 190, 256, 250, 30, 577, 192, 321, 1, 321, 130, 30, 250, 300, 30, 30, 65, 512, 577, 65], 1088, 512, 0, 14, True),
    # 16 tall tiles in 16 column blocks: the most
    ([384, 200, 512, 450, 190, 128, 190, 200, 200, 190, 450, 384, 512, 256, 1, 512], 704, 2048, 0, 16, True),
    # 19 in 14: one more than 256 items
    ([192, 250, 577, 128, 640, 1, 300, 64, 320, 65, 384, 450, 1, 300, 130, 190, 250, 256, 0, 577, 300, 300, 320, 30, 320], 704, 1792, 0, 19, False),
    # seven tiles of 256 rows in a lower cut
    ([130, 190, 256, 128, 300, 1, 450, 1, 30, 1, 300, 30, 192, 30, 577, 0, 64, 0, 64], 1344, 768, 256, 7, True),
    # 256 items of gemm1: no second round
    ([190, 192, 1, 250, 1, 0, 190, 65, 1, 128, 65, 128, 250, 1, 1, 64, 192], 1536, 1024, 0, 2, False)])
def test_ffn_tall_tiles_first_every_element(oracle, probe, G, sizes, H, F, height, tall, by_height):
    """More items of gemm1 than CUs (256), and tiles of more than 192 rows that all start at once: the table goes by descending height.
    Otherwise the slots stay in order.  Tiles of one height in several slots, empty slots, every element."""
    print("case tall first", sizes, flush=True)
    table = _tall_tiles(oracle, probe, G, sizes, H, F, max(sum(sizes) + 9, 65 * len(sizes)), height)
    tiles = table[3]
    cols = F // 64 if table[1] else (F + 127) // 128
    assert (tiles[:, 2] > 192).sum() == tall
    assert by_height == (tall * cols <= 256 < len(tiles) * cols)
    falls = (np.diff(tiles[:, 2]) <= 0).all()
    assert falls == by_height
    if by_height:    # tiles of one height by their slots' rows
        keys = [(-t[2], -sizes[t[3]], t[3], t[0]) for t in tiles.tolist()]
        assert keys == sorted(keys)
    else:
        assert _slots_in_order(table, sizes, 192)


@pytest.mark.parametrize("sizes,H,F,cut", [
    ([320, 256, 192, 128, 64, 37, 0, 321] * 4, 1344, 960, (0, False, True)),    # every height, partial last column blocks
    ([320, 256, 192, 128, 64, 37, 0, 321], 1088, 1344, (64, False, True)),      # partial last column blocks
    ([100] * 14, 2432, 2048, (0, False, False)), ([100] * 15, 2560, 2048, (0, False, False)),   # uniform tiles, 224 and 240 items of gemm1
    ([130] * 16, 2560, 768, (0, True, False)), ([130] * 17, 2560, 768, (0, True, False)),       # 192 and 204 of gemm1, 160 and 170 of gemm2
    ([130] * 16, 2560, 192, None), ([130] * 17, 2560, 192, None),               # the decode schedule with three tiles to a slot
    ([70, 0, 300], 64, 14400, (64, False, True))])                              # one k-step; more column blocks than tiles
def test_ffn_wide_and_narrow_column_blocks(oracle, probe, G, sizes, H, F, cut):
    """Wide and narrow column blocks of either GEMM: every output element against the oracle, and the rows gathered on load bit for
    bit the same.  `cut`: the height of the tiles and whether the blocks of gemm1 and gemm2 are narrow, as the table says."""
    cfg = wl.small_config(T=64, H=H, E=4, k=2, F=F, cid=103)
    print("case narrow", len(sizes), H, F, flush=True)
    n = sum(sizes)
    if cut:
        assert _tall_tiles(oracle, probe, G, sizes, H, F, n + 9, cut[0])[1:3] == cut[1:]
    else:
        _ffn_against_oracle(oracle, probe, G, cfg, sizes, 3, seed=H + F)
    gen = torch.Generator(device="cuda").manual_seed(H)
    x = torch.randn((n + 9, H), generator=gen, device="cuda").to(torch.bfloat16)
    w = [(torch.randn((2 * F, H), generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16),
          torch.randn((H, F), generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16)) for _ in range(2)]
    tab = probe.WeightTable([w[i % 2][0] for i in range(len(sizes))], [w[i % 2][1] for i in range(len(sizes))])
    so = torch.from_numpy(np.r_[0, np.cumsum(sizes)].astype(np.int32)).cuda()
    rows = torch.randperm(n + 9, device="cuda", generator=gen).to(torch.int32)
    plain = probe.grouped_ffn(x[rows.long()].contiguous(), so, tab)
    gathered = probe.grouped_ffn_gather(x, rows, 1, so, tab)
    torch.cuda.synchronize()
    assert torch.equal(plain[:n], gathered[:n])


@pytest.mark.parametrize("sizes,H,F,cut", [
    ([100] * 26, 1216, 768, (0, False, False)),                                                     # 156 / 130 items
    ([450, 190, 64, 64, 70, 450, 64, 450, 200, 3, 512], 704, 1792, (0, False, True)),               # 210 / 90
    ([30, 3, 64, 128, 450, 512, 200, 190, 3, 0, 128, 3, 70, 450, 200, 30], 2496, 832, (0, True, False)),
    ([64, 190, 130, 130, 130, 30, 3, 190], 1920, 1600, (0, True, True)),
    ([320] + [5] * 14, 3200, 1408, (64, False, False)),                                             # 209 / 247
    ([64] * 20 + [320], 1088, 1152, (64, False, True)),
    ([320, 320] + [1] * 6, 1728, 1216, (128, True, True)),
    ([190, 30, 130, 128, 3, 3, 577, 450, 390, 3, 3, 256, 300, 30, 3], 1408, 1024, (128, False, False)),
    ([130, 390, 3, 30, 64, 333, 3, 70, 333, 30, 512, 200, 70, 3, 70, 70], 1856, 1344, (192, False, False)),
    ([64, 30, 3, 128, 128, 3, 512, 577, 30, 30, 200, 256, 577], 1856, 640, (192, True, False)),
    ([0, 0, 512, 256, 70, 130, 0, 450, 130, 200, 200, 70, 390, 3], 768, 1600, (256, False, True)),
    ([70, 130, 128, 390, 200, 64, 30, 300, 200, 70, 390, 512, 70, 3], 2496, 768, (256, True, False))])
def test_ffn_column_blocks_by_estimated_time(oracle, probe, G, sizes, H, F, cut):
    """The standard cut and lower ones, each GEMM with wide or narrow column blocks, as the estimate of the launches takes them: every output
    element against the oracle, the cut and the widths from the table."""
    print("case estimated time", sizes, H, F, flush=True)
    cap = max(sum(sizes) + 9, 65 * len(sizes), 1600)
    assert _tall_tiles(oracle, probe, G, sizes, H, F, cap, cut[0])[1:3] == cut[1:]


@pytest.mark.parametrize("sizes,H,F,spare,items", [
    ([50], 64, 64, 36000, (1, 1)),
    ([90] * 9, 832, 576, 4000, (162, 126)),          # 18 tiles of 64 rows: a third group of two tiles, column groups that end early
    ([70] * 51, 64, 320, 9, (255, 51)),              # one item to a workgroup but the last, one to every
    ([70] * 64, 448, 256, 9, (256, 256)),
    ([130] * 43, 384, 768, 9, (258, 129)),           # the first two that are drawn
    ([70] * 83 + [130], 320, 192, 9, (255, 255)),
    ([300, 90, 200, 300, 70, 300, 70, 190, 200, 200, 130, 70, 190, 300, 70, 300, 200, 90, 190, 300, 200, 300, 200, 90, 130, 70, 190, 90, 200],
     704, 320, 9, (215, 258)),
    ([70, 300, 0, 90] * 11, 320, 2112, 9, (935, 165))])
def test_ffn_every_item_of_the_queue_is_run_once(oracle, probe, G, sizes, H, F, spare, items):
    """Tall tiles at numbers of items of gemm1 and gemm2 around one per workgroup, where the first ones are dealt without a draw, and with
    groups of tiles and columns that are not full: every output element against the oracle."""
    cap = max(sum(sizes) + spare, 65 * len(sizes))
    print("case queue", len(sizes), H, F, flush=True)
    cfg = wl.small_config(T=64, H=H, E=4, k=2, F=F, cid=106)
    assert (cap // 64 + len(sizes)) * (F // 64) > 512                                          # past the decode schedule
    ws = torch.zeros(probe.grouped_ffn_workspace_bytes(len(sizes), H, F, cap), dtype=torch.uint8, device="cuda")
    _ffn_against_oracle(oracle, probe, G, cfg, sizes, 3, seed=H + F, extra_rows=cap - sum(sizes), workspace=ws)
    n, narrow1, narrow2, _ = _tile_table(ws, F, cap)
    assert items == (n * (F // 64 if narrow1 else (F + 127) // 128), n * ((H + 127) // 128 if narrow2 else (H + 255) // 256))


@pytest.mark.parametrize("sizes,H,F,height,least_height", [
    ([3, 200, 0, 3, 200, 70, 130, 130, 30], 64, 1600, 64, 128),                    # 19 tiles, room for 12 in the least workspace
    ([577, 3, 0, 70, 64, 390, 130, 190, 0, 190, 0, 130, 30], 64, 832, 64, 192),
    ([200, 64, 200, 64, 333, 577, 30], 64, 1152, 64, 256),
    ([450, 512, 450, 512, 70], 256, 2176, 64, 0),
    ([256, 200, 450, 64, 512, 200], 448, 1216, 128, 0),
    ([200, 130, 200, 0, 450, 390, 512, 256, 333], 192, 704, 128, 192),
    ([64, 450, 70, 512, 200, 450], 1344, 1152, 192, 0)])
def test_ffn_tile_heights_by_estimated_time(oracle, probe, G, sizes, H, F, height, least_height):
    """Tiles of lower heights than the standard cut's where the estimate of the launches takes them: every output element against the
    oracle, and the same bits from the least workspace, whose tile table has no room for them and takes another cut."""
    S, n = len(sizes), sum(sizes)
    cap = max(n + 9, 65 * S)
    print("case heights", S, H, F, flush=True)
    _tall_tiles(oracle, probe, G, sizes, H, F, cap, height)
    gen = torch.Generator(device="cuda").manual_seed(H)
    x = torch.randn((cap, H), generator=gen, device="cuda").to(torch.bfloat16)
    w = (torch.randn((2 * F, H), generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16),
         torch.randn((H, F), generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16))
    so = torch.from_numpy(np.r_[0, np.cumsum(sizes)].astype(np.int32)).cuda()
    tab = probe.WeightTable([w[0]] * S, [w[1]] * S)
    up = lambda b: (b + 255) // 256 * 256
    ys = []
    for b, h in ((probe.grouped_ffn_workspace_bytes(S, H, F, cap), height), (up(cap * F * 2) + up(128 + 32 * (cap // 256 + S)), least_height)):
        ws = torch.zeros(b, dtype=torch.uint8, device="cuda")
        ys.append(probe.grouped_ffn(x, so, tab, workspace=ws)[:n])
        _check_cut(_tile_table(ws, F, cap), sizes, h)
    assert torch.equal(ys[0], ys[1])


@pytest.mark.parametrize("sizes,H,F,spare,tiles", [
    ([111, 244, 557, 236, 391, 208], 704, 1024, 0, 16),      # tiles of 128 rows; 12 would be the room of the standard cut
    ([190, 0, 130, 0, 200, 200], 512, 2048, 9, 14)])         # tiles of 64 rows
def test_ffn_workspace_of_the_query_holds_the_chosen_cut(probe, sizes, H, F, spare, tiles):
    """More room than the query asks for changes nothing: the same tiles, and the same bits."""
    cap = sum(sizes) + spare
    print("case room", sizes, H, F, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(H)
    x = torch.randn((cap, H), generator=gen, device="cuda").to(torch.bfloat16)
    w = (torch.randn((2 * F, H), generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16),
         torch.randn((H, F), generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16))
    so = torch.from_numpy(np.r_[0, np.cumsum(sizes)].astype(np.int32)).cuda()
    tab = probe.WeightTable([w[0]] * len(sizes), [w[1]] * len(sizes))
    tables, ys = [], []
    for more in (0, 1 << 16):
        ws = torch.zeros(probe.grouped_ffn_workspace_bytes(len(sizes), H, F, cap) + more, dtype=torch.uint8, device="cuda")
        ys.append(probe.grouped_ffn(x, so, tab, workspace=ws)[:sum(sizes)])
        tables.append(_tile_table(ws, F, cap))
    assert tables[0][0] == tables[1][0] == tiles
    assert tables[0][1:3] == tables[1][1:3] and np.array_equal(tables[0][3], tables[1][3])
    assert torch.equal(ys[0], ys[1])


@pytest.mark.parametrize("sizes,H,F,height", [
    ([70, 70, 100, 30, 200, 100, 0, 0, 30, 30, 0, 190], 128, 1472, 64),                                # 216 items of gemm1
    ([100, 70, 130, 70, 30, 130, 260, 130, 0, 130, 100], 128, 1216, 64),                               # 494
    ([450, 200, 100, 70, 450, 200, 200, 320, 100, 70, 100, 0], 128, 704, 128),                         # 242
    ([30, 200, 70, 260, 130, 130, 450, 260, 450, 200, 0, 200, 130, 100], 192, 1280, 128),              # 290
    ([122, 0, 226, 159, 98, 111, 135, 0, 118, 139, 0, 232, 522, 135, 299], 832, 2816, 192)])           # 374
def test_ffn_tiles_of_a_slot_stay_together_in_lower_cuts(oracle, probe, G, sizes, H, F, height):
    """Tiles of at most 192 rows: but for single tiles between them a slot's tiles stand side by side, and the slots of several tiles by
    descending rows, whatever the number of items.  Every output element against the oracle."""
    print("case together", sizes, H, F, flush=True)
    table = _tall_tiles(oracle, probe, G, sizes, H, F, max(sum(sizes) + 9, 65 * len(sizes)), height)
    assert _slots_in_order(table, sizes, height)


@pytest.mark.parametrize("H,F,n", [(4096, 2048, 75), (2880, 2880, 40)])
def test_ffn_workspace_of_a_larger_call_serves_a_smaller_one(oracle, probe, G, H, F, n):
    """A workspace sized for more rows serves fewer as their own does, bit for bit, also where only the smaller call keeps partial
    sums in it (one slot: 1100 rows take the tall tiles, 75 and 40 rows the pieces of K); one without that room is accepted."""
    cfg = wl.small_config(T=64, H=H, E=4, k=2, F=F, cid=101)
    big = 1100
    own, larger = (probe.grouped_ffn_workspace_bytes(1, cfg.H, cfg.F, r) for r in (n, big))
    assert own <= larger
    w13, w2 = wl.expert_weights_many(cfg, [0])[0]
    tab = probe.WeightTable([G.dev_bf16(w13)], [G.dev_bf16(w2)])
    x = wl.f32_to_bf16_bits(np.random.default_rng(3).standard_normal((n, cfg.H)).astype(np.float32))
    so = torch.tensor([0, n], dtype=torch.int32, device="cuda")
    print("case workspace of a larger call", flush=True)
    ys = [probe.grouped_ffn(G.dev_bf16(x), so, tab, workspace=torch.empty(b, dtype=torch.uint8, device="cuda"))
          for b in (own, larger, own - (8 << 20))]
    torch.cuda.synchronize()
    assert torch.equal(ys[0], ys[1])
    ref = oracle.grouped_ffn(x, np.array([0, n], np.int32), [w13], [w2])
    for y in ys:
        assert G.rel_err(G.f64_of(y), ref) < G.BF16_RTOL


def test_ffn_every_tile_height_at_full_depth(oracle, probe, G):
    """One slot per tile height (320, 256, 192, 128, 64 rows) and a ragged one, at the depth of the benchmark's
    main configuration (K = 7168 in the first GEMM, 2048 in the second: 112 and 32 steps of the main loop):
    every output element against the oracle."""
    print("case full-depth tile heights", flush=True)
    sizes = [320, 256, 192, 128, 64, 37, 0, 321]
    _tall_tiles(oracle, probe, G, sizes, wl.CONFIGS[3].H, wl.CONFIGS[3].F, sum(sizes) + 9, 0)


@pytest.mark.parametrize("H,F", [(64, 256), (320, 64), (256, 128)])
def test_ffn_every_tile_height_at_shallow_depth(oracle, probe, G, H, F):
    """Forty slots per tile height, with which the standard cut is taken, at depths of 1, 2, 4 and 5 steps of the main loop, where its first
    and last steps (which load fewer tiles ahead) are all there is: every output element against the oracle.  A single slot of
    each takes the decode schedule, whose main loop is the 64-row tile's."""
    print("case shallow depth H=%d F=%d" % (H, F), flush=True)
    sizes = [320, 256, 192, 128, 64, 37, 0, 321]
    _tall_tiles(oracle, probe, G, sizes * 40, H, F, 40 * sum(sizes) + 9, 0, n_weights=4)
    cfg = wl.small_config(T=64, H=H, E=4, k=2, F=F, cid=99)
    _ffn_against_oracle(oracle, probe, G, cfg, sizes, 4, seed=H * 7 + F)


@pytest.mark.parametrize("cid", [1, 4])
def test_ffn_with_rows_gathered_on_load_equals_ffn_on_the_permuted_copy(oracle, probe, G, cid):
    """probe_permute without the row copy + probe_grouped_ffn_gather give bit for bit the y of the standard
    pair (same kernels, only the source of the activation rows differs), and match the oracle."""
    cfg = wl.CONFIGS[cid]
    L, r = _layer(G, probe, cfg)
    counts = r["counts"].cpu().numpy()
    plan = wl.build_plan(cfg, counts)
    d_plan = probe.Plan(plan["rep_off"], plan["rep_slot"], plan["rep_weight"], plan["num_slots"])
    full = probe.permute(r["idx"], d_plan, L.d_x)
    lean = probe.permute(r["idx"], d_plan, L.d_x, copy_rows=False)
    assert "xp" not in lean
    for key in ("slot_counts", "slot_offsets", "pair_row", "n_local"):
        assert torch.equal(full[key], lean[key]), key
    nl = int(full["n_local"].item())
    assert torch.equal(full["row_pair"][:nl], lean["row_pair"][:nl])
    L.load_weights(plan["slot_expert"], probe)
    y0 = torch.full((cfg.N, cfg.H), 3.0, dtype=torch.bfloat16, device="cuda")
    y1 = torch.full((cfg.N, cfg.H), 3.0, dtype=torch.bfloat16, device="cuda")
    probe.grouped_ffn(full["xp"], full["slot_offsets"], L.weights, out=y0)
    probe.grouped_ffn_gather(L.d_x, lean["row_pair"], cfg.k, lean["slot_offsets"], L.weights, out=y1)
    torch.cuda.synchronize()
    assert torch.equal(y0, y1)
    ws = [wl.expert_weights(cfg, int(e)) for e in plan["slot_expert"]]
    o_p = oracle.permute(r["idx"].cpu().numpy(), plan["rep_off"], plan["rep_slot"], plan["rep_weight"],
                         plan["num_slots"], L.x)
    ref = oracle.grouped_ffn(o_p["xp"], o_p["slot_offsets"], [w[0] for w in ws], [w[1] for w in ws])
    assert G.rel_err(G.f64_of(y1)[:nl], ref) < G.BF16_RTOL


def test_largest_slot_and_expert_counts(oracle, probe, G):
    """The limits of the build at once: 256 experts, top-8, 1024 weight slots (four local copies of every
    expert with unequal shares).  Permute is checked completely, the FFN on a row sample from every slot."""
    E, k, T, H, F, S = 256, 8, 2048, 64, 64, 1024
    cfg = wl.small_config(T=T, H=H, E=E, k=k, F=F, E_loc=E, n_rep=0, zipf_s=1.0, chunk=0, ep=1, cid=95)
    L, r = _layer(G, probe, cfg)
    rep_off = np.arange(0, 4 * E + 1, 4, dtype=np.int32)
    rng = np.random.default_rng(95)
    rep_slot = rng.permutation(S).astype(np.int32)                  # copies of an expert sit in scattered slots
    rep_weight = rng.integers(0, 4, size=S).astype(np.int32)
    rep_weight[::4] = np.maximum(rep_weight[::4], 1)                # every expert keeps a positive share
    slot_expert = np.empty(S, np.int32)
    slot_expert[rep_slot] = np.repeat(np.arange(E, dtype=np.int32), 4)
    plan = probe.Plan(rep_off, rep_slot, rep_weight, S)
    p = probe.permute(r["idx"], plan, L.d_x)
    torch.cuda.synchronize()
    idx = r["idx"].cpu().numpy()
    o = oracle.permute(idx, rep_off, rep_slot, rep_weight, S, L.x)
    for key in ("slot_counts", "slot_offsets", "pair_row"):
        np.testing.assert_array_equal(p[key].cpu().numpy(), o[key])
    nl = int(o["n_local"])
    assert int(p["n_local"].item()) == nl == T * k
    np.testing.assert_array_equal(p["row_pair"].cpu().numpy()[:nl], o["row_pair"][:nl])
    np.testing.assert_array_equal(G.bits_of(p["xp"][:nl]), o["xp"][:nl])
    ws = wl.expert_weights_many(cfg, list(range(E)))
    d_w = [(G.dev_bf16(a), G.dev_bf16(b)) for a, b in ws]
    tab = probe.WeightTable([d_w[e][0] for e in slot_expert], [d_w[e][1] for e in slot_expert])
    y = probe.grouped_ffn(p["xp"], p["slot_offsets"], tab)
    torch.cuda.synchronize()
    so = o["slot_offsets"]
    rows = np.unique(np.concatenate([so[:-1][np.diff(so) > 0], so[1:][np.diff(so) > 0] - 1,
                                     rng.choice(nl, 512, replace=False)])).astype(np.int32)
    ref = oracle.grouped_ffn(o["xp"], so, [ws[e][0] for e in slot_expert], [ws[e][1] for e in slot_expert], rows=rows)
    got = G.f64_of(y[torch.from_numpy(rows.astype(np.int64)).cuda()])
    assert G.rel_err(got, ref) < G.BF16_RTOL
    assert (np.diff(so) == 0).any() and (np.diff(so) > 64).any()    # empty slots and slots of several tiles' worth


def test_more_tokens_than_one_pass_of_any_grid(oracle, probe, G):
    """140001 tokens: the top-k kernel's grid covers 131072 tokens per pass and wraps, permute walks 274 blocks
    of pairs, the FFN table holds hundreds of tiles.  Routing and permutation are checked completely, the
    floating-point stages on samples."""
    cfg = wl.small_config(T=140001, H=64, E=16, k=2, F=64, E_loc=8, n_rep=2, zipf_s=1.1, chunk=0, ep=2, cid=96)
    print("case many tokens", flush=True)
    res = G.run_layer_parity(oracle, probe, cfg, batch=0, route_sample=None, ffn_sample=64, seed=96)
    assert res["n_local"] > 100000


def test_graph_replay_of_the_variant_entry_points(oracle, probe, G):
    """The planner, the dispatch plan, the group-limited gate, permute without the row copy, the FFN with rows
    gathered on load and the combine with a shared expert record into one HIP graph; every replay, with eager
    work in between, reproduces the eager results bit for bit."""
    print("case graph replay, variants", flush=True)
    cfg = wl.small_config(T=384, H=128, E=32, k=4, F=128, E_loc=8, n_rep=0, ep=4, chunk=0, cid=98)
    T, H, E, k, F, R, E_loc = cfg.T, cfg.H, cfg.E, cfg.k, cfg.F, 4, 8
    L = G.Layer(cfg, 0)
    rng = np.random.default_rng(98)
    nh = torch.from_numpy(rng.poisson(60, size=(R, E)).astype(np.int32)).cuda()
    nh[:, 3] *= 6                                                  # a hot expert, so that the planner moves something
    sb = torch.from_numpy((rng.standard_normal(E) * 0.05).astype(np.float32)).cuda()
    kw = dict(max_replicas=2, budget=2, k_max=8, n0=16, g_num=1, g_den=2)
    S = E_loc + 2
    ws = wl.expert_weights_many(cfg, list(range(E)))
    d_w = [(G.dev_bf16(a), G.dev_bf16(b)) for a, b in ws]
    shared_tab = probe.WeightTable([d_w[0][0]], [d_w[0][1]])
    so_shared = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    res = {}

    def step():
        g = probe.plan_greedy(nh, E_loc, rank=0, want_assignment=True, **kw)
        d = probe.plan_dispatch(g["n"], g["delta_in"], E_loc, 0)
        r = probe.route_grouped(L.d_x, L.d_wg, None, None, sb, scoring="sigmoid", n_group=4, topk_group=2, group_top=2,
                                k=k, renormalize=True, routed_scale=2.5)
        p = probe.permute(r["idx"], g["plan"], L.d_x, copy_rows=False)
        res.update(g=g, d=d, r=r, p=p)
        return g, d, r, p

    # the weight table follows the planner's slot_expert, which is fixed for a fixed n_hat: build it once, eagerly
    g0, _, _, _ = step()
    torch.cuda.synchronize()
    se = g0["slot_expert"].cpu().numpy()
    assert (se[E_loc:] >= 0).any()
    tab = probe.WeightTable([d_w[max(int(e), 0)][0] for e in se], [d_w[max(int(e), 0)][1] for e in se])

    def full():
        g, d, r, p = step()
        y = probe.grouped_ffn_gather(L.d_x, p["row_pair"], k, p["slot_offsets"], tab)
        shared = probe.grouped_ffn(L.d_x, so_shared, shared_tab)
        y0 = torch.where(torch.arange(y.shape[0], device="cuda")[:, None] < p["n_local"], y, torch.zeros_like(y))
        out = probe.combine_shared(y0, p["pair_row"], r["w"], shared, 1.0)
        res.update(out=out, y0=y0)

    full()
    torch.cuda.synchronize()
    ref = dict(out=res["out"].clone(), idx=res["r"]["idx"].clone(), rows=res["p"]["pair_row"].clone(),
               rep_w=res["g"]["rep_weight"].clone(), dslot=res["d"]["rep_slot"].clone(), y0=res["y0"].clone())
    assert (ref["rows"] >= 0).any() and ref["out"].float().abs().sum() > 0
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            full()
    torch.cuda.synchronize()
    cap = dict(out=res["out"], idx=res["r"]["idx"], rows=res["p"]["pair_row"], rep_w=res["g"]["rep_weight"],
               dslot=res["d"]["rep_slot"], y0=res["y0"])
    used = int(res["g"]["rep_off"][-1])
    for i in range(3):
        for t in cap.values():
            t.zero_()                        # eager work between replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(cap["idx"], ref["idx"]) and torch.equal(cap["rows"], ref["rows"]), i
        assert torch.equal(cap["rep_w"][:used], ref["rep_w"][:used]) and torch.equal(cap["dslot"][:used], ref["dslot"][:used]), i
        assert torch.equal(cap["y0"], ref["y0"]) and torch.equal(cap["out"], ref["out"]), i
