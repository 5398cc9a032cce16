"""GPU parity of probe_plan_greedy (Algorithm 1 as one workgroup) against the sequential oracle: every
integer output bit-exact, and the device-resident loop predict -> plan -> permute."""
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


def _random_nhat(seed, R, E, scale=200, zipf=1.2):
    rng = np.random.default_rng(seed)
    pop = (np.arange(1, E + 1) ** -zipf)[rng.permutation(E)]
    lam = scale * pop / pop.mean()
    return rng.poisson(lam, size=(R, E)).astype(np.int32)


def _compare(probe, oracle, nh, E_loc, ranks, **kw):
    R, E = nh.shape
    o = oracle.plan_greedy(nh, E_loc, **kw)
    d_nh = torch.from_numpy(nh).cuda()
    for rank in ranks:
        g = probe.plan_greedy(d_nh, E_loc, rank=rank, want_assignment=True, **kw)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(g["moves"].cpu().numpy(), o["moves"])
        np.testing.assert_array_equal(g["delta_in"].cpu().numpy(), o["delta_in"])
        np.testing.assert_array_equal(g["delta_out"].cpu().numpy(), o["delta_out"])
        np.testing.assert_array_equal(g["n"].cpu().numpy(), o["n"])
        assert g["stats"].cpu().tolist() == [o["L_before"], o["L_after"], o["max_load"], o["n_moves"]]
        p = oracle.plan_for_rank(o["n"], o["delta_in"], E_loc, rank)
        used = int(p["rep_off"][E])
        np.testing.assert_array_equal(g["rep_off"].cpu().numpy(), p["rep_off"])
        np.testing.assert_array_equal(g["rep_slot"].cpu().numpy()[:used], p["rep_slot"])
        np.testing.assert_array_equal(g["rep_weight"].cpu().numpy()[:used], p["rep_weight"])
        np.testing.assert_array_equal(g["slot_expert"].cpu().numpy(), p["slot_expert"])
    return o


@pytest.mark.parametrize("seed,R,E,E_loc", [(1, 4, 16, 4), (2, 8, 64, 8), (3, 8, 256, 32), (4, 3, 10, 4),
                                            (5, 16, 128, 8), (6, 16, 256, 16), (7, 1, 8, 8), (8, 2, 3, 2)])
@pytest.mark.parametrize("cost", [dict(n0=0, g_num=0, g_den=1), dict(n0=64, g_num=1, g_den=4),
                                  dict(n0=16, g_num=3, g_den=2, eps=40)])
def test_planner_matches_oracle_bit_for_bit(oracle, probe, seed, R, E, E_loc, cost):
    print("case planner R=%d E=%d" % (R, E), flush=True)
    nh = _random_nhat(seed, R, E)
    o = _compare(probe, oracle, nh, E_loc, ranks=sorted({0, R // 2, R - 1}), max_replicas=3, budget=2, k_max=16, **cost)
    if R >= 4 and cost.get("eps", 0) == 0:
        assert o["n_moves"] >= 2          # the cases exercise the loop, not only its exit


@pytest.mark.parametrize("R,E,E_loc", [(11, 256, 24), (12, 256, 22), (16, 135, 9), (16, 136, 9), (5, 250, 50),
                                          (12, 240, 20), (12, 241, 21)])
def test_planner_on_both_sides_of_the_assignment_in_lds(oracle, probe, R, E, E_loc):
    """The largest assignments that lie in LDS (of all, 12 ranks of 240 experts take the most) and the smallest that lie in the
    workspace; budgets that run out, so that pairs become invalid between moves."""
    print("case planner R=%d E=%d" % (R, E), flush=True)
    for seed, budget in ((11, 1), (12, 8)):
        o = _compare(probe, oracle, _random_nhat(seed, R, E, scale=3000, zipf=1.4), E_loc, ranks=[R - 1], max_replicas=budget,
                     budget=budget, k_max=64, n0=64, g_num=1, g_den=4)
        assert o["n_moves"] >= 2


def test_planner_hand_worked_example_and_limits(oracle, probe):
    """The three-rank example worked out by hand in the oracle's pins, then the exits of the loop."""
    nh = np.array([[20, 0, 0], [30, 10, 0], [40, 0, 10]], np.int32)
    g = probe.plan_greedy(torch.from_numpy(nh).cuda(), 1, rank=1, max_replicas=2, budget=2, k_max=16)
    torch.cuda.synchronize()
    assert g["stats"].cpu().tolist() == [90, 50, 50, 2]
    assert g["moves"].cpu().numpy()[:2].tolist() == [[0, 0, 1], [0, 1, 2]]
    assert g["rep_weight"].cpu().numpy()[:5].tolist() == [20, 30, 40, 10, 10]
    assert g["rep_slot"].cpu().numpy()[:5].tolist() == [-1, 1, -1, 0, -1]
    big = _random_nhat(11, 8, 64)
    for kw in (dict(max_replicas=3, budget=0, k_max=16), dict(max_replicas=0, budget=3, k_max=16),
               dict(max_replicas=3, budget=3, k_max=0), dict(max_replicas=8, budget=8, k_max=64),
               dict(max_replicas=1, budget=3, k_max=16, n0=32, g_num=1, g_den=1)):
        _compare(probe, oracle, big, 8, ranks=[0, 5], **kw)
    # all-zero prediction: nothing to plan, every expert keeps a unit weight at home
    z = np.zeros((4, 16), np.int32)
    o = _compare(probe, oracle, z, 4, ranks=[2], max_replicas=2, budget=2, k_max=16)
    assert o["n_moves"] == 0


def test_predict_plan_permute_stays_on_the_device(oracle, probe, G):
    """Predicted top-k of 8 virtual source ranks -> n_hat -> plan on the device -> permute of the real routing
    with that plan; the permutation is checked against the oracle fed with the oracle's plan."""
    cfg = wl.small_config(T=2048, H=128, E=64, k=4, F=128, E_loc=8, n_rep=0, zipf_s=1.3, ep=8, cid=94)
    R, E, E_loc, k, T = 8, cfg.E, 8, cfg.k, cfg.T
    L = G.Layer(cfg, 0)
    pred = probe.predict_topk(L.d_x, L.d_wg, L.d_bias, L.tpg, k, True)
    # tokens are dealt to source ranks in contiguous chunks of T / R (test plumbing, not part of the path)
    chunk = T // R
    onehot = torch.zeros((R, E), dtype=torch.int32, device="cuda")
    src = (torch.arange(T, device="cuda") // chunk).clamp(max=R - 1).repeat_interleave(k)
    onehot.index_put_((src, pred["idx"].reshape(-1).long()), torch.ones(T * k, dtype=torch.int32, device="cuda"),
                      accumulate=True)
    kw = dict(max_replicas=3, budget=3, k_max=16, n0=16, g_num=1, g_den=2)
    g = probe.plan_greedy(onehot, E_loc, rank=0, **kw)
    route = probe.route_topk(L.d_x, L.d_wg, L.d_bias, L.tpg, k, True)
    perm = probe.permute(route["idx"], g["plan"], L.d_x)
    torch.cuda.synchronize()
    nh = onehot.cpu().numpy()
    np.testing.assert_array_equal(nh.sum(0), pred["counts"].cpu().numpy())
    o = oracle.plan_greedy(nh, E_loc, **kw)
    assert o["n_moves"] >= 1 and g["stats"].cpu().tolist()[3] == o["n_moves"]
    p = oracle.plan_for_rank(o["n"], o["delta_in"], E_loc, 0)
    o_p = oracle.permute(route["idx"].cpu().numpy(), p["rep_off"], p["rep_slot"], p["rep_weight"], p["num_slots"], L.x)
    np.testing.assert_array_equal(perm["pair_row"].cpu().numpy(), o_p["pair_row"])
    np.testing.assert_array_equal(perm["slot_counts"].cpu().numpy(), o_p["slot_counts"])
    nl = o_p["n_local"]
    np.testing.assert_array_equal(G.bits_of(perm["xp"][:nl]), o_p["xp"][:nl])
    # rank 0's replica slots received rows exactly when the plan gave them a positive share
    se = g["slot_expert"].cpu().numpy()
    for s in range(E_loc, E_loc + 3):
        if se[s] >= 0:
            assert o_p["slot_counts"][s] > 0


@pytest.mark.parametrize("seed,R,E,E_loc", [(1, 4, 16, 4), (2, 8, 64, 8), (3, 8, 256, 32), (5, 16, 128, 8), (8, 2, 3, 2)])
def test_dispatch_plan_matches_oracle(oracle, probe, seed, R, E, E_loc):
    """probe_plan_dispatch for every source rank, bit for bit against the oracle."""
    nh = _random_nhat(seed, R, E)
    kw = dict(max_replicas=3, budget=2, k_max=16, n0=16, g_num=1, g_den=4)
    o = oracle.plan_greedy(nh, E_loc, **kw)
    g = probe.plan_greedy(torch.from_numpy(nh).cuda(), E_loc, rank=0, want_assignment=True, **kw)
    for rs in range(R):
        d = probe.plan_dispatch(g["n"], g["delta_in"], E_loc, rs)
        torch.cuda.synchronize()
        od = oracle.plan_dispatch(o["n"], o["delta_in"], E_loc, rs)
        used = int(od["rep_off"][E])
        np.testing.assert_array_equal(d["rep_off"].cpu().numpy(), od["rep_off"])
        np.testing.assert_array_equal(d["rep_slot"].cpu().numpy()[:used], od["rep_slot"])
        np.testing.assert_array_equal(d["rep_weight"].cpu().numpy()[:used], od["rep_weight"])
        np.testing.assert_array_equal(d["rank_off"].cpu().numpy(), od["rank_off"])
        np.testing.assert_array_equal(d["slot_expert"].cpu().numpy()[:used], od["slot_expert"])


def test_source_side_grouping_by_destination_rank(oracle, probe, G):
    """One source rank's own tokens: route -> counts of every source rank -> plan -> dispatch plan -> permute.
    When the prediction is the routing itself, the send counts are exactly the planned ones, tokens of an expert
    this rank holds stay here, rows are grouped by destination rank and inside a rank by expert, and everything
    matches the oracle."""
    cfg = wl.small_config(T=1024, H=64, E=32, k=4, F=64, E_loc=4, n_rep=0, zipf_s=1.3, ep=8, cid=97)
    R, E, E_loc, k, me = 8, cfg.E, 4, cfg.k, 3
    L = G.Layer(cfg, 0)
    route = probe.route_topk(L.d_x, L.d_wg, L.d_bias, L.tpg, k, True)
    mine = route["counts"].cpu().numpy().astype(np.int32)
    nh = np.stack([mine if r == me else _random_nhat(40 + r, 1, E, scale=100)[0] for r in range(R)]).astype(np.int32)
    kw = dict(max_replicas=3, budget=3, k_max=16, n0=16, g_num=1, g_den=2)
    g = probe.plan_greedy(torch.from_numpy(nh).cuda(), E_loc, rank=me, want_assignment=True, **kw)
    d = probe.plan_dispatch(g["n"], g["delta_in"], E_loc, me)
    perm = probe.permute(route["idx"], d["plan"], L.d_x)
    torch.cuda.synchronize()
    o = oracle.plan_greedy(nh, E_loc, **kw)
    assert o["n_moves"] >= 1
    od = oracle.plan_dispatch(o["n"], o["delta_in"], E_loc, me)
    idx = route["idx"].cpu().numpy()
    o_p = oracle.permute(idx, od["rep_off"], od["rep_slot"], od["rep_weight"], od["num_slots"], L.x)
    for key in ("slot_counts", "slot_offsets", "pair_row"):
        np.testing.assert_array_equal(perm[key].cpu().numpy(), o_p[key])
    assert int(perm["n_local"].item()) == cfg.T * k                     # every pair has a destination
    np.testing.assert_array_equal(G.bits_of(perm["xp"]), o_p["xp"])
    # send counts per destination rank = what the planner assigned to this origin
    so, ro = o_p["slot_offsets"], od["rank_off"]
    np.testing.assert_array_equal(so[ro[1:]] - so[ro[:-1]], o["n"][me].sum(0))
    # rows of a slot carry that slot's expert; locality first: pairs of an expert that this rank holds stay here
    used = int(od["rep_off"][E])
    row_slot = np.searchsorted(so[:used + 1], np.arange(cfg.T * k), side="right") - 1
    row_expert = idx.ravel()[o_p["row_pair"]]
    np.testing.assert_array_equal(od["slot_expert"][row_slot], row_expert)
    dest = np.searchsorted(ro, row_slot, side="right") - 1
    held = set(range(me * E_loc, (me + 1) * E_loc)) | {int(e) for e in o["delta_in"][me] if e >= 0}
    for e in held:
        assert (dest[row_expert == e] == me).all()
