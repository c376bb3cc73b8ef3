"""GPU parity: every entry point of the C-ABI library against the CPU oracle on the same seeded
inputs.  Integer results (counts, plans, permutation indices, gathered rows) must be bit-exact;
floating-point results must be within relative L2 5e-3 of the oracle, which computes in double
precision on the same bf16-rounded inputs."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_2605_08639_amd as rl

pytestmark = pytest.mark.gpu
TOL = 5e-3
DEV = "cuda"


def rel_l2(got, want):
    got = got.double().cpu().numpy() if torch.is_tensor(got) else np.asarray(got, np.float64)
    want = np.asarray(want, np.float64)
    den = np.linalg.norm(want)
    return float(np.linalg.norm(got - want) / den) if den > 0 else float(np.linalg.norm(got))


def dev_i32(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(DEV)


def routing(cfg):
    ids, gates = zip(*[wl.make_routing(cfg, mb) for mb in range(cfg.n_mb)])
    return np.stack(ids), np.stack(gates)


# ------------------------------------------------------------------ histogram
@pytest.mark.parametrize("kw", [
    dict(), dict(T=513, k=3, E=12, EP=4),                       # T*k not a multiple of 4: scalar loads
    dict(T=20000, k=8, E=256, EP=8, n_mb=2), dict(T=1, k=1, E=4, EP=4, n_mb=1)])
def test_route_hist_bit_exact(kw):
    cfg = wl.small_config(**kw)
    ids, _ = routing(cfg)
    want, _ = oracle.route_hist(ids, cfg.E)
    err = rl.new_err_flag()
    got = rl.relibra_route_hist(torch.from_numpy(ids).to(DEV), cfg.E, err_flag=err)
    assert np.array_equal(got.cpu().numpy(), want)
    assert err.item() == 0


def test_route_hist_flags_bad_ids_and_handles_empty():
    ids = torch.zeros((1, 64, 2), dtype=torch.int32, device=DEV)
    ids[0, 5, 1] = 9
    ids[0, 6, 0] = -1
    err = rl.new_err_flag()
    got = rl.relibra_route_hist(ids, 8, err_flag=err)
    assert err.item() == rl.ERR_ID_RANGE
    assert got.sum().item() == 126 and got[0, 0].item() == 126
    got = rl.relibra_route_hist(torch.zeros((2, 0, 2), dtype=torch.int32, device=DEV), 8)
    assert got.shape == (2, 8) and got.sum().item() == 0


def test_per_source_histogram_bit_exact():
    """x[j][e] of Section 4.1 (tokens on source rank j routed to e): the histogram kernel on the ids
    viewed as [n_mb*EP, T/EP, k] against the oracle's definition."""
    cfg = wl.small_config(T=1024, k=4, E=32, EP=8, n_mb=2)
    ids, _ = routing(cfg)
    err = rl.new_err_flag()
    got = rl.relibra_route_hist_src(torch.from_numpy(ids).to(DEV), cfg.E, cfg.EP, err_flag=err).cpu().numpy()
    assert err.item() == 0 and got.shape == (cfg.n_mb, cfg.EP, cfg.E)
    for mb in range(cfg.n_mb):
        assert np.array_equal(got[mb], oracle.route_hist_src(ids[mb], cfg.E, cfg.EP))


def test_histograms_of_several_layers_in_one_launch():
    """Replayed routing of every layer is known before training (Section 3): the histograms of
    [layers, n_mb] micro-batches come from one launch over ids of [layers * n_mb, T, k]."""
    layers = 3
    cfgs = [wl.small_config(T=640, k=4, E=64, EP=8, n_mb=4, index=90 + l) for l in range(layers)]
    ids = np.concatenate([routing(c)[0] for c in cfgs])                    # [layers * n_mb, T, k]
    got = rl.relibra_route_hist(torch.from_numpy(ids).to(DEV), 64).cpu().numpy().reshape(layers, 4, 64)
    for l, c in enumerate(cfgs):
        assert np.array_equal(got[l], oracle.route_hist(routing(c)[0], 64)[0])
    skew, inter = rl.relibra_load_stats(got[0], top=8)
    s_or, i_or = oracle.load_stats(got[0], top=8)
    assert np.allclose(skew, s_or, rtol=1e-14, atol=0) and np.array_equal(inter, i_or)


# ------------------------------------------------------------------ plan + permute
def plan_both(cfg, counts):
    want = oracle.plan(counts, cfg.EP, cfg.rpn, cfg.r)
    got = rl.relibra_plan(counts, cfg.k, cfg.EP, cfg.rpn, cfg.r)
    for key in ("expert_to_slot", "replica_expert", "inst_ptr", "inst_rank", "inst_rows", "inst_group",
                "group_expert", "group_offset"):
        assert np.array_equal(got[key], want[key]), key
    return got


@pytest.mark.parametrize("kw", [
    dict(), dict(E=8, k=2, EP=4, r=1, T=512, n_mb=1, routing="single"),
    dict(E=128, k=8, EP=8, r=2, T=3000, n_mb=2, h=64),
    dict(E=16, k=8, EP=8, r=2, T=1000, n_mb=2, routing="stress", zipf_s=1.5, h=64),
    dict(E=5, k=5, EP=1, r=0, T=37, n_mb=1, h=8)])
def test_hist_plan_permute_bit_exact(kw):
    cfg = wl.small_config(**kw)
    ids, _ = routing(cfg)
    counts = rl.relibra_route_hist(torch.from_numpy(ids).to(DEV), cfg.E).cpu().numpy()
    p = plan_both(cfg, counts)
    for mb in range(cfg.n_mb):
        X, _ = wl.make_tokens(cfg, mb)
        want_row, want_src = oracle.permute(ids[mb], cfg.E, p["inst_ptr"][mb], p["inst_rows"][mb],
                                            p["inst_group"][mb], p["group_offset"][mb])
        err = rl.new_err_flag()
        row_of, src_of, Xrows = rl.relibra_permute(
            torch.from_numpy(ids[mb]).to(DEV), dev_i32(p["inst_ptr"][mb]), dev_i32(p["inst_rows"][mb]),
            dev_i32(p["inst_group"][mb]), dev_i32(p["group_offset"][mb]), X.to(DEV), cfg.E, cfg.G, err_flag=err)
        assert err.item() == 0
        assert np.array_equal(row_of.cpu().numpy(), want_row)
        assert np.array_equal(src_of.cpu().numpy(), want_src)
        want_rows = oracle.gather_rows(X, want_src, cfg.k)
        got_rows = Xrows.cpu().view(torch.int16).numpy().view(np.uint16)
        assert np.array_equal(got_rows, want_rows)                     # bit copy


@pytest.mark.parametrize("kw", [dict(E=16, k=2, EP=4, r=2, T=240, ranks_per_node=2),
                                dict(E=128, k=8, EP=8, r=2, T=3000, n_mb=2, h=64, ranks_per_node=4),
                                dict(E=16, k=8, EP=8, r=2, T=1000, n_mb=2, routing="stress", zipf_s=1.5, h=64, ranks_per_node=8)])
def test_source_aware_permute_bit_exact(kw):
    """Permutation under the per-source split of Section 5.2: indices and gathered rows identical
    to the oracle's, and every instance holds exactly the tokens of each source the split gave it."""
    cfg = wl.small_config(**kw)
    ids, _ = routing(cfg)
    counts = oracle.route_hist(ids, cfg.E)[0]
    p = plan_both(cfg, counts)
    for mb in range(cfg.n_mb):
        X, _ = wl.make_tokens(cfg, mb)
        x = oracle.route_hist_src(ids[mb], cfg.E, cfg.EP)
        ptr, rank, rows, grp, off = (p[key][mb] for key in ("inst_ptr", "inst_rank", "inst_rows", "inst_group", "group_offset"))
        y = oracle.assign_sources(x, cfg.rpn, ptr, rank, rows)
        want_row, want_src = oracle.permute_src(ids[mb], cfg.E, cfg.EP, ptr, grp, off, y)
        tabs = rl.relibra_assign_sources(x, cfg.rpn, ptr, rank, rows)
        err = rl.new_err_flag()
        row_of, src_of, Xrows = rl.relibra_permute_src(
            torch.from_numpy(ids[mb]).to(DEV), dev_i32(ptr), dev_i32(grp), dev_i32(off), cfg.EP,
            dev_i32(tabs["src_first"]), dev_i32(tabs["inst_src_rows"]), dev_i32(tabs["inst_src_base"]),
            X.to(DEV), cfg.E, cfg.G, err_flag=err)
        assert err.item() == 0
        assert np.array_equal(row_of.cpu().numpy(), want_row)
        assert np.array_equal(src_of.cpu().numpy(), want_src)
        got_rows = Xrows.cpu().view(torch.int16).numpy().view(np.uint16)
        assert np.array_equal(got_rows, oracle.gather_rows(X, want_src, cfg.k))
    # a split table that does not cover the routing is flagged and the assignment skipped
    bad = tabs["inst_src_rows"].copy()
    i, j = np.argwhere(bad > 0)[0]
    bad[i, j] -= 1
    err = rl.new_err_flag()
    row_of, _, _ = rl.relibra_permute_src(
        torch.from_numpy(ids[-1]).to(DEV), dev_i32(ptr), dev_i32(grp), dev_i32(off), cfg.EP,
        dev_i32(tabs["src_first"]), dev_i32(bad), dev_i32(tabs["inst_src_base"]), None, cfg.E, cfg.G, err_flag=err)
    # one token of source j fewer than routed: exactly the source's last assignment of that expert has no row
    e_bad = int(np.searchsorted(np.asarray(ptr), i, side="right") - 1)
    tps = cfg.T // cfg.EP
    flat = ids[-1].reshape(-1)
    a_of = np.flatnonzero((flat == e_bad) & (np.arange(flat.size) // cfg.k // tps == j))
    assert err.item() == rl.ERR_PLAN_COVER
    assert np.array_equal(np.flatnonzero(row_of.cpu().numpy() < 0), a_of[-1:])


def test_source_aware_permute_one_token_per_source():
    """Smallest shape the source-aware permutation accepts: T = EP tokens, k = 1."""
    E = EP = 4
    ids = np.array([[2], [2], [0], [2]], np.int32)
    x = oracle.route_hist_src(ids, E, EP)
    # expert 2 (home rank 2) has a replica on rank 0 taking one of its three tokens
    ptr, rank, rows, grp = [0, 1, 2, 4, 5], [0, 1, 0, 2, 3], [1, 0, 1, 2, 0], [0, 2, 1, 4, 6]
    off = [0, 1, 2, 2, 2, 4, 4, 4, 4]                       # G = 8 groups: (home, replica) per rank
    y = oracle.assign_sources(x, 4, ptr, rank, rows)
    want_row, want_src = oracle.permute_src(ids, E, EP, ptr, grp, off, y)
    tabs = rl.relibra_assign_sources(x, 4, ptr, rank, rows)
    err = rl.new_err_flag()
    row_of, src_of, _ = rl.relibra_permute_src(torch.from_numpy(ids).to(DEV), dev_i32(ptr), dev_i32(grp), dev_i32(off), EP,
                                               dev_i32(tabs["src_first"]), dev_i32(tabs["inst_src_rows"]),
                                               dev_i32(tabs["inst_src_base"]), None, E, 8, err_flag=err)
    assert err.item() == 0
    assert row_of.cpu().tolist() == want_row.tolist() and src_of.cpu().tolist() == want_src.tolist()
    assert want_row.tolist() == [1, 2, 0, 3]                # token 0 (source 0) is the one the replica on rank 0 serves


def test_timed_plan_drives_the_device_path():
    """Tables of the time-driven Algorithm 2 (equal to the oracle's, checked on the host) through
    permutation and expert FFN forward: indices bit-exact, outputs within the bar."""
    cfg = wl.small_config(E=32, k=4, EP=8, r=2, T=1024, n_mb=1, h=128, hff=192, ranks_per_node=4)
    ids, _ = routing(cfg)
    x = np.stack([oracle.route_hist_src(ids[0], cfg.E, cfg.EP)])
    model = rl.cost_model(cfg.EP, cfg.rpn, 2048, 768, 5e14, 4e11, 5e10)
    placed = (np.arange(cfg.E) // cfg.M).astype(np.int32)
    p = rl.relibra_plan_timed(x, cfg.k, model, cfg.r, placed)
    want = oracle.plan_comm(x, cfg.rpn, cfg.r, placed, oracle.cost_model(2048, 768, 5e14, 4e11, 5e10))
    for key in ("inst_ptr", "inst_rank", "inst_rows", "inst_group", "group_expert", "group_offset"):
        assert np.array_equal(p[key], want[key]), key
    X, _ = wl.make_tokens(cfg, 0)
    Wg, Wu, Wd = wl.make_weights(cfg)
    tabs = {key: dev_i32(p[key][0]) for key in ("inst_ptr", "inst_rows", "inst_group", "group_offset", "group_expert")}
    err = rl.new_err_flag()
    row_of, src_of, Xrows = rl.relibra_permute(torch.from_numpy(ids[0]).to(DEV), tabs["inst_ptr"], tabs["inst_rows"],
                                               tabs["inst_group"], tabs["group_offset"], X.to(DEV), cfg.E, cfg.G, err_flag=err)
    want_row, want_src = oracle.permute(ids[0], cfg.E, p["inst_ptr"][0], p["inst_rows"][0], p["inst_group"][0], p["group_offset"][0])
    assert err.item() == 0
    assert np.array_equal(row_of.cpu().numpy(), want_row) and np.array_equal(src_of.cpu().numpy(), want_src)
    Y = rl.relibra_moe_ffn_fwd(Xrows, tabs["group_offset"], tabs["group_expert"], Wg.to(DEV), Wu.to(DEV), Wd.to(DEV), err_flag=err)[3]
    Y_o = oracle.ffn_fwd(oracle.gather_rows(X, want_src, cfg.k), p["group_offset"][0], p["group_expert"][0], Wg, Wu, Wd)[3]
    assert err.item() == 0
    assert rel_l2(Y, Y_o) <= TOL


@pytest.mark.parametrize("E,k,T,EP", [(4, 1, 1, 4), (8, 1, 1025, 4), (8, 2, 2048, 4), (8, 1, 4097, 4), (512, 4, 1024, 8),
                                      (516, 2, 300, 4), (32, 4, 511, 8), (256, 2, 2048, 8), (512, 2, 1536, 8), (512, 1, 3073, 8)])
def test_permute_at_the_one_block_limits(E, k, T, EP):
    """Sizes around a wave's share and around the largest ones that one block permutes."""
    cfg = wl.small_config(E=E, k=k, EP=EP, r=1, T=T, n_mb=1, h=8)
    ids, _ = routing(cfg)
    p = plan_both(cfg, oracle.route_hist(ids, cfg.E)[0])
    X = torch.randn((T, 8), generator=torch.Generator().manual_seed(T)).to(torch.bfloat16)
    err = rl.new_err_flag()
    rl.prof_start(level=2, max_records=16)
    row_of, src_of, Xrows = rl.relibra_permute(torch.from_numpy(ids[0]).to(DEV), *(dev_i32(p[key][0]) for key in (
        "inst_ptr", "inst_rows", "inst_group", "group_offset")), X.to(DEV), cfg.E, cfg.G, err_flag=err)
    assert ("perm_small" in rl.prof_stop()) == (E <= 512 and k * T <= (4096 if E <= 256 else 3072))
    want_row, want_src = oracle.permute(ids[0], cfg.E, *(p[key][0] for key in ("inst_ptr", "inst_rows", "inst_group", "group_offset")))
    assert err.item() == 0
    assert np.array_equal(row_of.cpu().numpy(), want_row) and np.array_equal(src_of.cpu().numpy(), want_src)
    assert torch.equal(Xrows.cpu(), X[torch.from_numpy(want_src).long() // k])


@pytest.mark.parametrize("E,k,T,h", [(8, 2, 300, 8), (16, 4, 777, 264), (8, 8, 1024, 1024), (8, 8, 1024, 1032), (16, 9, 700, 2040)])
def test_row_gather_on_both_sides_of_its_rule(E, k, T, h):
    """Rows of up to 16 MiB and beyond, widths that no number of threads divides, more assignments per token than are
    looked up at a time."""
    cfg = wl.small_config(E=E, k=k, EP=4, r=1, T=T, n_mb=1, h=8)
    ids, _ = routing(cfg)
    p = plan_both(cfg, oracle.route_hist(ids, cfg.E)[0])
    tabs = [dev_i32(p[key][0]) for key in ("inst_ptr", "inst_rows", "inst_group", "group_offset")]
    X = torch.randn((T, h), generator=torch.Generator().manual_seed(h)).to(torch.bfloat16).to(DEV)
    Xrows = torch.full((T * k + 1, h), 7.0, dtype=torch.bfloat16, device=DEV)
    err = rl.new_err_flag()
    _, src_of, _ = rl.relibra_permute(torch.from_numpy(ids[0]).to(DEV), *tabs, X, cfg.E, cfg.G, Xrows=Xrows[:-1], err_flag=err)
    assert err.item() == 0
    assert torch.equal(Xrows[:-1], X[src_of.long() // k]) and (Xrows[-1] == 7.0).all()


def test_permute_flags_a_plan_that_does_not_cover_the_routing():
    cfg = wl.small_config(E=8, k=2, EP=4, r=1, T=200, n_mb=1, h=64)
    ids, _ = routing(cfg)
    counts, _ = oracle.route_hist(ids, cfg.E)
    p = rl.relibra_plan(counts, cfg.k, cfg.EP, cfg.rpn, cfg.r)
    rows = p["inst_rows"][0].copy()
    rows[p["inst_ptr"][0][3]] -= 1                                     # one row short for expert 3
    err = rl.new_err_flag()
    row_of, src_of, _ = rl.relibra_permute(
        torch.from_numpy(ids[0]).to(DEV), dev_i32(p["inst_ptr"][0]), dev_i32(rows), dev_i32(p["inst_group"][0]),
        dev_i32(p["group_offset"][0]), None, cfg.E, cfg.G, err_flag=err)
    assert err.item() & rl.ERR_PLAN_COVER
    assert (row_of == -1).sum().item() == 1


# ------------------------------------------------------------------ expert FFN
def ffn_case(seed, E, h, hff, rows, experts, wscale=0.05):
    rng = np.random.default_rng(seed)
    go = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    ge = np.array(experts, np.int32)
    N = int(go[-1])
    bf = lambda x: torch.from_numpy(np.asarray(x, np.float32)).to(torch.bfloat16)
    X = bf(rng.standard_normal((N, h)))
    dY = bf(rng.standard_normal((N, h)))
    Wg = bf(wscale * rng.standard_normal((E, hff, h)))
    Wu = bf(wscale * rng.standard_normal((E, hff, h)))
    Wd = bf(wscale * rng.standard_normal((E, h, hff)))
    return go, ge, X, dY, Wg, Wu, Wd


FFN_CASES = [
    # rows per group span: empty, 1, one short of a tile, a tile, one over, several tiles + tail
    dict(seed=1, E=4, h=256, hff=192, rows=(0, 1, 127, 128, 129, 300, 0, 65), experts=(0, 1, 2, 3, 0, 1, -1, 3)),
    dict(seed=2, E=3, h=128, hff=256, rows=(40, 513, 7), experts=(2, 0, 1)),
    dict(seed=3, E=2, h=64, hff=64, rows=(5, 3), experts=(1, 0)),
    dict(seed=4, E=2, h=320, hff=448, rows=(200, 0, 131), experts=(0, 1, 0)),
    # long groups: the large weight-gradient tile geometry (512 or more rows per group on average)
    dict(seed=7, E=2, h=128, hff=256, rows=(1100, 700), experts=(1, 0)),
    # widths of whole 512-column tiles (calls of so few tiles stay on the 256-column ones: see
    # test_wide_tiles_on_weights_as_stored for the others), ragged rows and a replica
    dict(seed=8, E=3, h=512, hff=512, rows=(1, 64, 65, 200, 0, 129), experts=(2, 0, 1, 0, -1, 2)),
    dict(seed=9, E=2, h=1024, hff=1536, rows=(300, 77), experts=(1, 0)),
    # the shortest contractions (two slabs: fewer than the ring holds): gate/up and dA over h = 64 with 512-wide
    # outputs, then down over h' = 64 and dX over two phases of two slabs
    dict(seed=10, E=2, h=64, hff=512, rows=(130, 64), experts=(1, 0)),
    dict(seed=11, E=2, h=512, hff=64, rows=(129, 3), experts=(0, 1)),
]


def dw_slots(ge, E):
    """Home group of an expert = its first group; later groups of the same expert are replicas."""
    seen, slots, nxt = set(), [], E
    for e in ge.tolist():
        if e < 0:
            slots.append(nxt); nxt += 1
        elif e in seen:
            slots.append(nxt); nxt += 1
        else:
            seen.add(e); slots.append(e)
    return np.array(slots, np.int32), nxt


@pytest.mark.parametrize("case", FFN_CASES)
def test_ffn_fwd_bwd_within_tolerance(case):
    go, ge, X, dY, Wg, Wu, Wd = ffn_case(**case)
    E, hff, h = Wg.shape
    Gt_o, U_o, A_o, Y_o = oracle.ffn_fwd(X, go, ge, Wg, Wu, Wd)
    dX_o, dWg_o, dWu_o, dWd_o = oracle.ffn_bwd(X, dY, go, ge, Wg, Wu, Wd)
    live = np.concatenate([np.arange(go[g], go[g + 1]) for g in range(len(ge)) if ge[g] >= 0]).astype(np.int64)

    d = lambda t: t.to(DEV)
    err = rl.new_err_flag()
    Xd, dYd, Wgd, Wud, Wdd = d(X), d(dY), d(Wg), d(Wu), d(Wd)
    god, ged = dev_i32(go), dev_i32(ge)
    N = X.shape[0]
    sentinel = lambda cols: torch.full((N, cols), 7.0, dtype=torch.bfloat16, device=DEV)
    Gt, U, A, Y = rl.relibra_moe_ffn_fwd(Xd, god, ged, Wgd, Wud, Wdd, Gt=sentinel(hff), U=sentinel(hff),
                                         A=sentinel(hff), Yrows=sentinel(h), err_flag=err)
    for name, got, want in (("Gt", Gt, Gt_o), ("U", U, U_o), ("A", A, A_o), ("Y", Y, Y_o)):
        assert rel_l2(got[live], want[live]) <= TOL, name
        for g in range(len(ge)):                                   # per group, so a bad tile cannot hide
            if ge[g] >= 0 and go[g + 1] > go[g]:
                assert rel_l2(got[go[g]:go[g + 1]], want[go[g]:go[g + 1]]) <= TOL, (name, g)
    dead = np.setdiff1d(np.arange(N), live)
    if dead.size:                                                   # rows of empty slots stay untouched
        assert (Y[dead].float() == 7.0).all()

    slots, n_slots = dw_slots(ge, E)
    mk = lambda *s: torch.full(s, 3.0, dtype=torch.float32, device=DEV)
    dWg, dWu, dWd = mk(n_slots, hff, h), mk(n_slots, hff, h), mk(n_slots, h, hff)
    dX = rl.relibra_moe_ffn_bwd(dYd, Xd, Gt, U, A, god, ged, dev_i32(slots), Wgd, Wud, Wdd, dWg, dWu, dWd,
                                dXrows=sentinel(h), err_flag=err)
    assert err.item() == 0
    assert rel_l2(dX[live], dX_o[live]) <= TOL
    used = sorted(set(e for e in ge.tolist() if e >= 0))
    for name, got, want in (("dWg", dWg, dWg_o), ("dWu", dWu, dWu_o), ("dWd", dWd, dWd_o)):
        for e in used:
            if np.linalg.norm(want[e]) > 0:
                assert rel_l2(got[e], want[e]) <= TOL, (name, e)
            else:
                assert (got[e] == 0).all(), (name, e)              # expert seen only through empty groups
    # bit-reproducible
    dWg2, dWu2, dWd2 = mk(n_slots, hff, h), mk(n_slots, hff, h), mk(n_slots, h, hff)
    dX2 = rl.relibra_moe_ffn_bwd(dYd, Xd, Gt, U, A, god, ged, dev_i32(slots), Wgd, Wud, Wdd, dWg2, dWu2, dWd2)
    assert torch.equal(dX2[live], dX[live])
    for a, b in ((dWg2, dWg), (dWu2, dWu), (dWd2, dWd)):
        assert torch.equal(a[:E][used], b[:E][used])
    # accumulate mode adds the same gradient on top
    before = [w[:E].clone() for w in (dWg, dWu, dWd)]
    rl.relibra_moe_ffn_bwd(dYd, Xd, Gt, U, A, god, ged, dev_i32(slots), Wgd, Wud, Wdd, dWg, dWu, dWd,
                           flags=rl.BWD_ACCUMULATE, err_flag=err)
    for w, b in zip((dWg, dWu, dWd), before):
        for e in used:
            assert rel_l2(w[e], 2 * b[e].double().cpu().numpy()) <= 1e-6
    assert err.item() == 0


def test_ffn_group_range_runs_one_ranks_share_only():
    go, ge, X, dY, Wg, Wu, Wd = ffn_case(seed=5, E=4, h=128, hff=128, rows=(30, 50, 0, 20, 140, 9),
                                         experts=(0, 1, 2, 3, 0, 1))
    _, _, _, Y_o = oracle.ffn_fwd(X, go, ge, Wg, Wu, Wd)
    d = lambda t: t.to(DEV)
    N, h = X.shape
    Y = torch.full((N, h), 7.0, dtype=torch.bfloat16, device=DEV)
    rl.relibra_moe_ffn_fwd(d(X), dev_i32(go), dev_i32(ge), d(Wg), d(Wu), d(Wd), g_begin=3, g_end=5, Yrows=Y)
    a, b = int(go[3]), int(go[5])
    assert rel_l2(Y[a:b], Y_o[a:b]) <= TOL
    assert (Y[:a].float() == 7.0).all() and (Y[b:].float() == 7.0).all()


def test_ffn_flags_inconsistent_group_tables_without_faulting():
    go, ge, X, dY, Wg, Wu, Wd = ffn_case(seed=6, E=2, h=64, hff=64, rows=(10, 10), experts=(0, 1))
    d = lambda t: t.to(DEV)
    err = rl.new_err_flag()
    bad_go = go.copy()
    bad_go[2] = 5000                                                 # beyond the row buffer
    rl.relibra_moe_ffn_fwd(d(X), dev_i32(bad_go), dev_i32(ge), d(Wg), d(Wu), d(Wd), err_flag=err)
    assert err.item() & rl.ERR_GROUP_TABLE
    err.zero_()
    rl.relibra_moe_ffn_fwd(d(X), dev_i32(go), dev_i32(np.array([0, 9], np.int32)), d(Wg), d(Wu), d(Wd), err_flag=err)
    assert err.item() & rl.ERR_GROUP_TABLE


class _ScheduleLaunches:
    """The calls inside launch the scheduling kernel this many times (each call without it schedules in its first kernel)."""

    def __init__(self, launches):
        self.launches = launches

    def __enter__(self):
        rl.prof_start(2, 256)

    def __exit__(self, kind, *_):
        seen = rl.prof_stop().get("sched", (0.0, 0))[1]
        assert kind is not None or seen == self.launches


@pytest.mark.parametrize("rows", [1024, 65536])                       # scheduled inside the first kernel, by the scheduling kernel
def test_ffn_row_tiles_of_overlapping_groups_end_with_the_lists(rows):
    """A corrupted table whose groups cover the same rows again and again has more row tiles than the workspace lists
    (which hold those of every table without overlap): flagged, and nothing is written behind the workspace."""
    groups = 64
    X, _, Wg, Wu, Wd = ffn_case(seed=12, E=2, h=64, hff=64, rows=(rows,), experts=(0,))[2:]
    go, ge = dev_i32(np.array([0, rows] * (groups // 2) + [0], np.int32)), dev_i32(np.arange(groups) % 2)
    need, guard = rl.workspace_bytes(rl.WS_FFN_FWD, rows, 1, 2, groups, 64, 64), 1 << 16
    ws = torch.full((need + guard,), 99, dtype=torch.uint8, device=DEV)
    err = rl.new_err_flag()
    with _ScheduleLaunches(0 if rows == 1024 else 1):
        rl.relibra_moe_ffn_fwd(X.to(DEV), go, ge, Wg.to(DEV), Wu.to(DEV), Wd.to(DEV), workspace=ws[:need], err_flag=err)
    assert err.item() == rl.ERR_GROUP_TABLE
    assert (ws[need:] == 99).all()


def _fwd_bwd(X, dY, W, counts, E, g_begin=0, g_end=None, out=None):
    """Forward and data gradients of groups of the given sizes (experts in turn); out: earlier results to write a range into."""
    go = dev_i32(np.concatenate([[0], np.cumsum(counts)]))
    ge = dev_i32(np.arange(len(counts)) % E)
    N, h, hff = X.shape[0], X.shape[1], W[0].shape[1]
    if out is None:
        out = [torch.full((N, w), 3.0, dtype=torch.bfloat16, device=DEV) for w in (hff, hff, hff, h, h)]
    Gt, U, A, Y, dX = out
    err = rl.new_err_flag()
    rl.relibra_moe_ffn_fwd(X, go, ge, *W, g_begin=g_begin, g_end=g_end, Gt=Gt, U=U, A=A, Yrows=Y, err_flag=err)
    rl.relibra_moe_ffn_bwd(dY, None, Gt, U, A, go, ge, ge, *W, None, None, None, g_begin=g_begin, g_end=g_end, flags=rl.BWD_DEFER_WGRAD,
                           dXrows=dX, err_flag=err, E=E)
    assert err.item() == 0
    return out


def _device_case(N, E, h, hff):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(N + h)
    draw = lambda std, *s: torch.empty(s, dtype=torch.bfloat16, device=DEV).normal_(0.0, std, generator=gen)
    return draw(1.0, N, h), draw(1.0, N, h), [draw(0.05, E, hff, h), draw(0.05, E, hff, h), draw(0.05, E, h, hff)]


SPARE_ROWS = 65536      # a buffer of so many rows may hold more than 504 row tiles, whatever its groups: the scheduling kernel's


def _with_spare_rows(t):
    return torch.cat([t, t.new_zeros((SPARE_ROWS - t.shape[0],) + t.shape[1:])])


@pytest.mark.parametrize("groups", [1, 251, 252, 253, 300])
def test_schedule_inside_the_first_kernel_equals_the_scheduling_kernel(groups):
    """Groups of up to 128 rows count as two row tiles each in the bound: 252 of them are the most that are scheduled
    inside.  The same rows range by range (always inside) and in a larger buffer (never inside) must come out bit for bit the
    same."""
    counts = np.full(groups, 128)
    if groups > 1:
        counts[::7] = 0
        counts[3::11] = 65
    X, dY, W = _device_case(int(128 * groups), 3, 64, 64)
    with _ScheduleLaunches(0 if groups <= 252 else 2):
        whole = _fwd_bwd(X, dY, W, counts, 3)
    parts = None
    with _ScheduleLaunches(0):
        for lo in range(0, groups, 100):
            parts = _fwd_bwd(X, dY, W, counts, 3, lo, min(lo + 100, groups), parts)
    with _ScheduleLaunches(2):
        spare = _fwd_bwd(_with_spare_rows(X), _with_spare_rows(dY), W, counts, 3)
    for a, b, c in zip(whole, parts, spare):
        assert torch.equal(a, b)
        assert torch.equal(a, c[:a.shape[0]]) and (c[a.shape[0]:] == 3.0).all()
    first = int(np.argmax(counts > 0))
    want = torch.nn.functional.silu(X[:int(counts[first])].float() @ W[0][first % 3].float().T)
    want = want * (X[:want.shape[0]].float() @ W[1][first % 3].float().T)
    assert rel_l2(whole[2][:want.shape[0]], want.cpu().numpy()) <= TOL


def _every_form(X, dY, gate, W, E, go, ge, slot, g_begin, g_end, rows):
    """Forward and data gradients in a buffer of `rows` rows: plain, gate-fused, with the replica slots' parameters."""
    go, ge, slot = dev_i32(go), dev_i32(ge), dev_i32(slot)
    N, h, hff, G = X.shape[0], X.shape[1], W[0].shape[1], len(ge)
    fill = lambda *widths: [torch.full((rows, w), 3.0, dtype=torch.bfloat16, device=DEV) for w in widths]
    pad = lambda t: torch.cat([t, t.new_zeros((rows - N,) + t.shape[1:])])
    own = [w[:E] for w in W]
    tok = (torch.arange(rows, dtype=torch.int32, device=DEV) * 7) % N
    dgate = torch.full((rows,), 3.0, device=DEV)
    scratch = torch.zeros(rl.workspace_bytes(rl.WS_DGATE, rows, 1, E, G, h, hff), dtype=torch.uint8, device=DEV)
    plain, gated, slots = fill(hff, hff, hff, h, h), fill(hff, hff, hff, h, h), fill(h)
    errs = [rl.new_err_flag() for _ in range(5)]
    share = dict(g_begin=g_begin, g_end=g_end)
    Gt, U, A, Y, dX = plain
    rl.relibra_moe_ffn_fwd(pad(X), go, ge, *own, Gt=Gt, U=U, A=A, Yrows=Y, err_flag=errs[0], **share)
    rl.relibra_moe_ffn_bwd(pad(dY), None, Gt, U, A, go, ge, slot, *own, None, None, None, flags=rl.BWD_DEFER_WGRAD, dXrows=dX, err_flag=errs[1], E=E, **share)
    rl.relibra_moe_ffn_bwd(pad(dY), None, Gt, U, A, go, ge, slot, *W, None, None, None, flags=rl.BWD_DEFER_WGRAD | rl.BWD_REPLICA_WEIGHTS, dXrows=slots[0],
                           err_flag=errs[2], E=E, **share)
    Gt, U, A, Y, dX = gated
    rl.relibra_moe_ffn_fwd_gated(X, tok, pad(gate), go, ge, *own, Gt=Gt, U=U, A=A, Ag=A, Yrows=Y, err_flag=errs[3], **share)
    rl.relibra_moe_ffn_bwd_gated(dY, tok, pad(gate), Gt, U, go, ge, slot, *own, dXrows=dX, dgate=dgate, dgate_scratch=scratch, err_flag=errs[4], E=E, **share)
    return plain + gated + slots + [dgate], [e.item() for e in errs]


BANDS = [0, 1, 129, 1153, 64, 65, 1024, 128, 2176, 0, 3]            # one row tile, bands of eight, a remainder of one and of two bands
SCHEDULE_CASES = [  # rows of the groups, expert width, first and last group of the call
    pytest.param([1], 320, 0, None, id="one-row"), pytest.param([129], 320, 0, None, id="two-row-tiles"),
    pytest.param(BANDS, 64, 0, None, id="bands-one-column-tile"), pytest.param(BANDS, 320, 0, None, id="bands-three-column-tiles"),
    pytest.param(BANDS, 320, 3, 9, id="bands-of-a-range"), pytest.param([(37 * i) % 97 for i in range(300)], 64, 0, None, id="more-than-256-groups")]


@pytest.mark.parametrize("counts,hff,g_begin,g_end", SCHEDULE_CASES)
def test_schedule_inside_the_first_kernel_over_bands_columns_and_forms(counts, hff, g_begin, g_end):
    """The same table in a buffer with spare rows goes through the scheduling kernel: bit for bit the same results, with several
    column tiles (of 128 in gate/up, of 256 in the activation backward), groups of more row tiles than a band has,
    gate-fused and with parameter blocks chosen by replica slot."""
    E, h, N, G = 5, 128, sum(counts), len(counts)
    X, dY, W = _device_case(N, E + 3, h, hff)
    gate = torch.linspace(0.1, 0.9, N, device=DEV)
    go, ge = np.concatenate([[0], np.cumsum(counts)]), np.arange(G) % E
    slot = np.where(np.arange(G) % 3 == 1, E + np.arange(G) % 3, ge)
    with _ScheduleLaunches(0):
        inside, err_in = _every_form(X, dY, gate, W, E, go, ge, slot, g_begin, g_end, N)
    with _ScheduleLaunches(5):
        outside, err_out = _every_form(X, dY, gate, W, E, go, ge, slot, g_begin, g_end, SPARE_ROWS)
    assert err_in == err_out == [0] * 5
    for a, b in zip(inside, outside):
        assert torch.equal(a, b[:N]) and (b[N:] == 3.0).all()
    assert not torch.equal(inside[4], inside[10]) or not (slot != ge)[np.asarray(counts) > 0].any()      # replica slots' parameters were read


def test_schedule_inside_the_first_kernel_skips_and_flags_the_same_groups():
    """Falling and negative offsets, experts and replica slots out of range: the same groups are skipped and the same calls flagged
    whichever kernel works the schedule out."""
    E, h, hff, N = 3, 64, 320, 900
    X, dY, W = _device_case(N, E + 2, h, hff)
    gate = torch.linspace(0.1, 0.9, N, device=DEV)
    good = dict(go=np.array([0, 40, 100, 300, 500, 700, 900]), ge=np.array([0, 1, 2, 0, -1, 2]), slot=np.array([0, 3, 2, 0, 0, 4]))
    bad = {"offset": dict(go=np.array([0, 40, -5, 300, 500, 700, 900])), "expert": dict(ge=np.array([0, 1, 7, -2, -1, 2])),
           "slot": dict(slot=np.array([0, 3, 5, -1, 99, 4]))}
    for what, change in [("none", {}), *bad.items()]:
        table = {**good, **change}
        with _ScheduleLaunches(0):
            inside, err_in = _every_form(X, dY, gate, W, E, *table.values(), 0, None, N)
        with _ScheduleLaunches(5):
            outside, err_out = _every_form(X, dY, gate, W, E, *table.values(), 0, None, SPARE_ROWS)
        flagged = {"none": [], "slot": [2]}.get(what, range(5))          # the slot table is read with the replica slots' parameters only
        assert err_in == err_out == [rl.ERR_GROUP_TABLE if i in flagged else 0 for i in range(5)], what
        for a, b in zip(inside, outside):
            assert torch.equal(a, b[:N]) and (b[N:] == 3.0).all(), what


@pytest.mark.parametrize("h,hff,rows", [(1024, 64, 16384), (64, 1024, 5376), (64, 1024, 8192)])
def test_more_rows_do_not_change_the_others(h, hff, rows):
    """128 more rows, up to which the results of a kernel fit the L2s (32 MiB) and beyond which they do not, must not change
    the others."""
    X, dY, W = _device_case(rows + 128, 3, h, hff)
    more = _fwd_bwd(X, dY, W, np.full(rows // 128 + 1, 128), 3)
    fewer = _fwd_bwd(X[:rows].contiguous(), dY[:rows].contiguous(), W, np.full(rows // 128, 128), 3)
    for a, b in zip(more, fewer):
        assert torch.equal(a[:rows], b)


# ------------------------------------------------------------------ combine
@pytest.mark.parametrize("T,k,h", [(97, 4, 256), (5, 1, 8), (300, 8, 2048)])
def test_combine_modes(T, k, h):
    rng = np.random.default_rng(T)
    N = T * k
    row_of = rng.permutation(N).astype(np.int32)
    bf = lambda x: torch.from_numpy(np.asarray(x, np.float32)).to(torch.bfloat16)
    Y = bf(rng.standard_normal((N, h)))
    dOut = bf(rng.standard_normal((T, h)))
    gates = rng.random((T, k)).astype(np.float32)
    gates /= gates.sum(1, keepdims=True)
    Yd, gd, rd = Y.to(DEV), torch.from_numpy(gates).to(DEV), dev_i32(row_of)
    err = rl.new_err_flag()
    out = rl.relibra_unpermute_combine(rl.COMBINE_FWD, Yd, rd, T, k, gates=gd, err_flag=err)
    assert rel_l2(out, oracle.combine_fwd(Y.double().numpy(), gates, row_of, T, k)) <= TOL
    out = rl.relibra_unpermute_combine(rl.COMBINE_SUM, Yd, rd, T, k, err_flag=err)
    assert rel_l2(out, oracle.combine_fwd(Y.double().numpy(), None, row_of, T, k)) <= TOL
    dY, dgate = rl.relibra_unpermute_combine(rl.COMBINE_BWD, Yd, rd, T, k, gates=gd, tok=dOut.to(DEV), err_flag=err)
    dY_o, dgate_o = oracle.combine_bwd(dOut.double().numpy(), Y.double().numpy(), gates, row_of, T, k)
    assert rel_l2(dY, dY_o) <= TOL and rel_l2(dgate, dgate_o) <= TOL
    assert err.item() == 0


# ------------------------------------------------------------------ whole path
def run_layer_gpu(cfg, mb, ids, gates, p, Wg, Wu, Wd, X, dOut, dW):
    """One micro-batch through every entry point; returns what the layer hands back."""
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    err = rl.new_err_flag()
    ids_d, gates_d = t(ids), t(gates)
    tabs = {key: dev_i32(p[key][mb]) for key in ("inst_ptr", "inst_rows", "inst_group", "group_offset",
                                                 "group_expert", "group_dw_slot")}
    row_of, src_of, Xrows = rl.relibra_permute(ids_d, tabs["inst_ptr"], tabs["inst_rows"], tabs["inst_group"],
                                               tabs["group_offset"], X, cfg.E, cfg.G, err_flag=err)
    Gt, U, A, Y = rl.relibra_moe_ffn_fwd(Xrows, tabs["group_offset"], tabs["group_expert"], Wg, Wu, Wd, err_flag=err)
    Out = rl.relibra_unpermute_combine(rl.COMBINE_FWD, Y, row_of, cfg.T, cfg.k, gates=gates_d, err_flag=err)
    dY, dgate = rl.relibra_unpermute_combine(rl.COMBINE_BWD, Y, row_of, cfg.T, cfg.k, gates=gates_d, tok=dOut,
                                             err_flag=err)
    dXrows = rl.relibra_moe_ffn_bwd(dY, Xrows, Gt, U, A, tabs["group_offset"], tabs["group_expert"],
                                    tabs["group_dw_slot"], Wg, Wu, Wd, *dW, err_flag=err)
    dX = rl.relibra_unpermute_combine(rl.COMBINE_SUM, dXrows, row_of, cfg.T, cfg.k, err_flag=err)
    assert err.item() == 0
    return Out, dgate, dX


def run_layer_oracle(cfg, mb, ids, gates, p, Wg, Wu, Wd, X, dOut):
    row_of, src_of = oracle.permute(ids, cfg.E, p["inst_ptr"][mb], p["inst_rows"][mb], p["inst_group"][mb],
                                    p["group_offset"][mb])
    Xrows = oracle.gather_rows(X, src_of, cfg.k)
    go, ge = p["group_offset"][mb], p["group_expert"][mb]
    _, _, _, Y = oracle.ffn_fwd(Xrows, go, ge, Wg, Wu, Wd)
    Out = oracle.combine_fwd(Y, gates, row_of, cfg.T, cfg.k)
    dY, dgate = oracle.combine_bwd(dOut.double().numpy(), Y, gates, row_of, cfg.T, cfg.k)
    # the oracle's backward takes bf16 rows: round the upstream row gradients once, as the path does
    dY16 = torch.from_numpy(dY).to(torch.bfloat16)
    dXrows, dWg, dWu, dWd = oracle.ffn_bwd(Xrows, dY16, go, ge, Wg, Wu, Wd)
    dX = oracle.combine_fwd(dXrows, None, row_of, cfg.T, cfg.k)
    return Out, dgate, dX, dWg, dWu, dWd


@pytest.mark.parametrize("cfg", [wl.CONFIGS[0],
                                 wl.small_config(E=16, k=4, EP=4, r=2, T=777, n_mb=2, h=256, hff=192)],
                         ids=["config1-tiny", "ragged-small"])
def test_whole_layer_matches_oracle(cfg):
    ids, gates = routing(cfg)
    counts = rl.relibra_route_hist(torch.from_numpy(ids).to(DEV), cfg.E).cpu().numpy()
    assert np.array_equal(counts, oracle.route_hist(ids, cfg.E)[0])
    p = plan_both(cfg, counts)
    Wg, Wu, Wd = wl.make_weights(cfg)
    Wgd, Wud, Wdd = Wg.to(DEV), Wu.to(DEV), Wd.to(DEV)
    n_slots = cfg.E + cfg.EP * cfg.r
    for mb in range(cfg.n_mb):
        X, dOut = wl.make_tokens(cfg, mb)
        dW = [torch.empty((n_slots, cfg.hff, cfg.h), dtype=torch.float32, device=DEV),
              torch.empty((n_slots, cfg.hff, cfg.h), dtype=torch.float32, device=DEV),
              torch.empty((n_slots, cfg.h, cfg.hff), dtype=torch.float32, device=DEV)]
        Out, dgate, dX = run_layer_gpu(cfg, mb, ids[mb], gates[mb], p, Wgd, Wud, Wdd, X.to(DEV), dOut.to(DEV), dW)
        Out_o, dgate_o, dX_o, dWg_o, dWu_o, dWd_o = run_layer_oracle(cfg, mb, ids[mb], gates[mb], p, Wg, Wu, Wd, X, dOut)
        assert rel_l2(Out, Out_o) <= TOL
        assert rel_l2(dgate, dgate_o) <= TOL
        assert rel_l2(dX, dX_o) <= TOL
        assert rel_l2(dW[0][:cfg.E], dWg_o) <= TOL
        assert rel_l2(dW[1][:cfg.E], dWu_o) <= TOL
        assert rel_l2(dW[2][:cfg.E], dWd_o) <= TOL


# ------------------------------------------------------------------ layer-shared replica buffer
def test_replica_push_fills_slots_and_ffn_reads_them():
    """Section 5.1: the push copies each live replica's home parameters into its slot (bit copy,
    checked against the oracle); the FFN reading replica groups' parameters from those slots must
    give bit-identical results to reading them from the home blocks."""
    cfg = wl.small_config(E=16, k=4, EP=4, r=2, T=777, n_mb=2, h=256, hff=192)
    ids, gates = routing(cfg)
    counts = oracle.route_hist(ids, cfg.E)[0]
    p = plan_both(cfg, counts)
    Wg, Wu, Wd = wl.make_weights(cfg)
    n_slots = cfg.E + cfg.EP * cfg.r
    assert (p["replica_expert"] >= 0).any(), "the case must place replicas"

    def with_slots(W):      # home blocks followed by replica slots holding recognisable junk
        junk = torch.full((cfg.EP * cfg.r, *W.shape[1:]), 7.0, dtype=torch.bfloat16)
        return torch.cat([W, junk]).contiguous()

    big = [with_slots(W) for W in (Wg, Wu, Wd)]
    big_d = [W.to(DEV) for W in big]
    home_d = [W.to(DEV) for W in (Wg, Wu, Wd)]
    for mb in range(cfg.n_mb):
        rep = p["replica_expert"][mb].reshape(-1)
        err = rl.relibra_replica_push(*big_d, dev_i32(rep), cfg.E, cfg.EP, cfg.r, n_workgroups=3)
        assert err.item() == 0
        for W_d, W in zip(big_d, big):
            want = oracle.replica_push(W.view(torch.uint16).numpy(), rep, cfg.E)
            got = W_d.cpu().view(torch.uint16).numpy()
            live = np.concatenate([np.ones(cfg.E, bool), rep >= 0])
            assert np.array_equal(got[live], want[live])
            W.copy_(W_d.cpu())              # slots keep their contents from one micro-batch to the next
        X, dOut = wl.make_tokens(cfg, mb)
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
        tabs = {key: dev_i32(p[key][mb]) for key in ("inst_ptr", "inst_rows", "inst_group", "group_offset",
                                                     "group_expert", "group_dw_slot")}
        row_of, src_of, Xrows = rl.relibra_permute(t(ids[mb]), tabs["inst_ptr"], tabs["inst_rows"], tabs["inst_group"],
                                                   tabs["group_offset"], X.to(DEV), cfg.E, cfg.G)
        outs = []
        for use_slots in (False, True):
            err = rl.new_err_flag()
            W3 = big_d if use_slots else home_d
            ge = tabs["group_dw_slot"] if use_slots else tabs["group_expert"]
            Gt, U, A, Y = rl.relibra_moe_ffn_fwd(Xrows, tabs["group_offset"], ge, *W3, err_flag=err)
            dW = [torch.zeros((n_slots, cfg.hff, cfg.h), dtype=torch.float32, device=DEV),
                  torch.zeros((n_slots, cfg.hff, cfg.h), dtype=torch.float32, device=DEV),
                  torch.zeros((n_slots, cfg.h, cfg.hff), dtype=torch.float32, device=DEV)]
            dY = torch.randn(Y.shape, generator=torch.Generator().manual_seed(mb)).to(torch.bfloat16).to(DEV)
            dXrows = rl.relibra_moe_ffn_bwd(dY, Xrows, Gt, U, A, tabs["group_offset"], tabs["group_expert"],
                                            tabs["group_dw_slot"], *W3, *dW, err_flag=err, E=cfg.E,
                                            flags=rl.BWD_REPLICA_WEIGHTS if use_slots else 0)
            assert err.item() == 0
            outs.append((Y, dXrows, dW[0][:cfg.E], dW[1][:cfg.E], dW[2][:cfg.E]))
        for a, b in zip(*outs):
            assert torch.equal(a, b)
        # the same through the deferred and the gate-fused backward (no dW array: the slot table only
        # selects parameter blocks, and the wrapper must size it by the parameter arrays)
        row_tok = rl.relibra_row_tokens(src_of, cfg.k, cfg.T)
        row_gate = rl.relibra_row_gates(src_of, t(gates[mb]))
        Gt, U, A, Y = rl.relibra_moe_ffn_fwd(Xrows, tabs["group_offset"], tabs["group_expert"], *home_d)
        dY = torch.randn(Y.shape, generator=torch.Generator().manual_seed(100 + mb)).to(torch.bfloat16).to(DEV)
        got = []
        for use_slots in (False, True):
            err = rl.new_err_flag()
            W3 = big_d if use_slots else home_d
            fl = rl.BWD_REPLICA_WEIGHTS if use_slots else 0
            dXd = rl.relibra_moe_ffn_bwd(dY, None, Gt, U, A, tabs["group_offset"], tabs["group_expert"], tabs["group_dw_slot"],
                                         *W3, None, None, None, err_flag=err, E=cfg.E, flags=fl | rl.BWD_DEFER_WGRAD)
            dXg, dgate = rl.relibra_moe_ffn_bwd_gated(dOut.to(DEV), row_tok, row_gate, Gt, U, tabs["group_offset"],
                                                     tabs["group_expert"], tabs["group_dw_slot"], *W3, src_of=src_of,
                                                     err_flag=err, E=cfg.E, flags=fl)
            assert err.item() == 0
            got.append((dXd, dXg, dgate))
        for a, b in zip(*got):
            assert torch.equal(a, b)


def test_replica_pull_equals_the_inline_sum_and_two_layers_share_one_slot_buffer():
    """Section 5.1: one buffer of r slots per rank serves every layer in turn (parameters pushed
    before a layer's expert computation, gradients pulled back after its backward).  Two layers with
    their own weights and routing run through ONE shared slot buffer (parameters and gradients),
    the slots overwritten between layers; every result must equal, bit for bit, the run in which
    each layer has private slots and the backward call sums the replica gradients in line."""
    L = 2
    cfgs = [wl.small_config(E=16, k=4, EP=4, r=2, T=777, n_mb=1, h=256, hff=192, index=70 + l) for l in range(L)]
    E, EP, r, h, hff = cfgs[0].E, cfgs[0].EP, cfgs[0].r, cfgs[0].h, cfgs[0].hff
    n_rep = EP * r
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    layers = []
    for cfg in cfgs:
        ids, gates = routing(cfg)
        p = plan_both(cfg, oracle.route_hist(ids, cfg.E)[0])
        assert (p["replica_expert"] >= 0).any()
        X, dOut = wl.make_tokens(cfg, 0)
        tabs = {key: dev_i32(p[key][0]) for key in ("inst_ptr", "inst_rows", "inst_group", "group_offset",
                                                    "group_expert", "group_dw_slot")}
        row_of, src_of, Xrows = rl.relibra_permute(t(ids[0]), tabs["inst_ptr"], tabs["inst_rows"], tabs["inst_group"],
                                                   tabs["group_offset"], X.to(DEV), E, cfg.G)
        dY = torch.randn((cfg.N, h), generator=torch.Generator().manual_seed(cfg.index)).to(torch.bfloat16).to(DEV)
        layers.append(dict(p=p, tabs=tabs, Xrows=Xrows, dY=dY, W=[W.to(DEV) for W in wl.make_weights(cfg)],
                           rep=dev_i32(p["replica_expert"][0].reshape(-1))))

    def run_layer(ly, Wp, dWp, n_blocks, slot_table, pull):
        """forward + backward of one layer on parameter arrays Wp / gradient arrays dWp of n_blocks blocks whose
        first E are the layer's home blocks and whose last n_rep are the replica slots."""
        err = rl.new_err_flag()
        rl.relibra_replica_push(*Wp, ly["rep"], n_blocks - n_rep, EP, r, n_workgroups=5, err_flag=err)
        Gt, U, A, Y = rl.relibra_moe_ffn_fwd(ly["Xrows"], ly["tabs"]["group_offset"], slot_table, *Wp, err_flag=err)
        flags = rl.BWD_REPLICA_WEIGHTS | (rl.BWD_NO_REPLICA_SUM if pull else 0)
        dXrows = rl.relibra_moe_ffn_bwd(ly["dY"], ly["Xrows"], Gt, U, A, ly["tabs"]["group_offset"], ly["tabs"]["group_expert"],
                                        slot_table, *Wp, *dWp, err_flag=err, E=n_blocks - n_rep, flags=flags)
        if pull:
            rl.relibra_replica_pull(*dWp, ly["rep"], n_blocks - n_rep, EP, r, n_workgroups=3, err_flag=err)
        assert err.item() == 0
        return Y, dXrows

    shapes = [(hff, h), (hff, h), (h, hff)]
    # reference: private slots per layer, replica gradients summed inside the backward call
    want = []
    for ly in layers:
        Wp = [torch.cat([W, torch.zeros((n_rep, *W.shape[1:]), dtype=W.dtype, device=DEV)]) for W in ly["W"]]
        dWp = [torch.zeros((E + n_rep, *s), dtype=torch.float32, device=DEV) for s in shapes]
        Y, dXrows = run_layer(ly, Wp, dWp, E + n_rep, ly["tabs"]["group_dw_slot"], pull=False)
        want.append((Y, dXrows, *[d[:E].clone() for d in dWp]))
    # shared: [layer 0 home | layer 1 home | slots]; layer l sees the tail that starts at its home blocks, so a
    # replica slot's block index is (L - l) * E + s in its view
    W_all = [torch.cat([ly["W"][i] for ly in layers] + [torch.full((n_rep, *shapes[i]), 7.0, dtype=torch.bfloat16, device=DEV)])
             for i in range(3)]
    dW_all = [torch.full((L * E + n_rep, *s), float("nan"), dtype=torch.float32, device=DEV) for s in shapes]
    got = [None] * L
    for l in (0, 1, 1, 0):                                   # forward order, then backward order: slots refilled each time
        ly = layers[l]
        slot = ly["p"]["group_dw_slot"][0].copy()
        slot[slot >= E] += (L - l - 1) * E
        view_W = [W[l * E:] for W in W_all]
        view_dW = [d[l * E:] for d in dW_all]
        Y, dXrows = run_layer(ly, view_W, view_dW, (L - l) * E + n_rep, dev_i32(slot), pull=True)
        got[l] = (Y, dXrows, *[d[l * E:(l + 1) * E].clone() for d in dW_all])
    for l in range(L):
        for a, b in zip(got[l], want[l]):
            assert torch.equal(a, b), l
    # the home parameters were never written
    for i in range(3):
        for l, ly in enumerate(layers):
            assert torch.equal(W_all[i][l * E:(l + 1) * E], ly["W"][i])


def test_replica_push_flags_bad_table_and_leaves_empty_slots():
    E, EP, r, h, hff = 4, 2, 2, 64, 64
    W = [torch.arange((E + EP * r) * h * hff, dtype=torch.float32).reshape(E + EP * r, hff, h).to(torch.bfloat16).to(DEV)
         for _ in range(3)]
    before = [w.clone() for w in W]
    err = rl.relibra_replica_push(*W, dev_i32([2, -1, 99, 0]), E, EP, r, n_workgroups=1)
    assert err.item() == rl.ERR_ID_RANGE
    for w, b in zip(W, before):
        assert torch.equal(w[E + 0], b[2]) and torch.equal(w[E + 3], b[0])
        assert torch.equal(w[E + 1], b[E + 1]) and torch.equal(w[E + 2], b[E + 2])
        assert torch.equal(w[:E], b[:E])


@pytest.mark.parametrize("E,slots,h,hff,n_wg", [
    (1, 1, 8, 8, 1),             # one vector short of a thread's share
    (5, 7, 192, 320, 3),         # chunks that the block does not fill, several slots of one expert
    (3, 1100, 64, 72, 5),        # three lists of slots: an expert's sum goes on across them
    (40, 16, 256, 520, 64),      # more workgroups than chunks of an expert
])
def test_replica_push_and_pull_at_list_and_chunk_edges(E, slots, h, hff, n_wg):
    rng = np.random.default_rng(slots)
    table = rng.integers(-1, E, slots).astype(np.int32)
    table[0] = 0
    gen = torch.Generator().manual_seed(slots)
    W = [torch.randn((E + slots, h * hff), generator=gen).to(torch.bfloat16) for _ in range(3)]
    dW = [torch.randn((E + slots, h * hff), generator=gen) for _ in range(3)]
    Wd, dWd = [w.to(DEV) for w in W], [d.to(DEV) for d in dW]
    shape = lambda ts: [t.view(E + slots, h, hff) for t in ts]
    err = rl.relibra_replica_push(*shape(Wd), dev_i32(table), E, slots, 1, n_workgroups=n_wg)
    rl.relibra_replica_pull(*shape(dWd), dev_i32(table), E, slots, 1, n_workgroups=n_wg, err_flag=err)
    assert err.item() == 0
    for s, e in enumerate(table):
        if e >= 0:
            for w, d in zip(W, dW):
                w[E + s] = w[e]
                d[e] += d[E + s]                 # ascending slots, one fp32 addition each: the defined order
    for got, want in zip(Wd + dWd, W + dW):
        assert torch.equal(got.cpu(), want)


# ------------------------------------------------------------------ batched weight gradients
def test_batched_weight_gradients_match_oracle_and_per_microbatch_path():
    """dW of a whole batch in one pass (Section 2.1: gradients accumulate over micro-batches):
    against the oracle's sum over micro-batches (all instances of an expert), and against the
    per-micro-batch accumulate path of the library, which differs only in fp32 summation order."""
    cfg = wl.small_config(E=16, k=4, EP=4, r=2, T=777, n_mb=3, h=256, hff=192)
    ids, gates = routing(cfg)
    counts = oracle.route_hist(ids, cfg.E)[0]
    p = plan_both(cfg, counts)
    Wg, Wu, Wd = wl.make_weights(cfg)
    W_d = [W.to(DEV) for W in (Wg, Wu, Wd)]
    n_slots = cfg.E + cfg.EP * cfg.r
    shapes = [(cfg.hff, cfg.h), (cfg.hff, cfg.h), (cfg.h, cfg.hff)]
    dW_ref = [np.zeros((cfg.E, *s)) for s in shapes]
    dW_mb = [torch.empty((n_slots, *s), dtype=torch.float32, device=DEV) for s in shapes]
    err = rl.new_err_flag()
    kept, fused_in = [], []
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    for mb in range(cfg.n_mb):
        X, _ = wl.make_tokens(cfg, mb)
        tabs = {key: dev_i32(p[key][mb]) for key in ("inst_ptr", "inst_rows", "inst_group", "group_offset",
                                                     "group_expert", "group_dw_slot")}
        Xd = X.to(DEV)
        row_of, src_of, Xrows = rl.relibra_permute(t(ids[mb]), tabs["inst_ptr"], tabs["inst_rows"], tabs["inst_group"],
                                                   tabs["group_offset"], Xd, cfg.E, cfg.G, err_flag=err)
        fused_in.append((Xd, rl.relibra_row_tokens(src_of, cfg.k, cfg.T, err_flag=err)))
        Gt, U, A, Y = rl.relibra_moe_ffn_fwd(Xrows, tabs["group_offset"], tabs["group_expert"], *W_d, err_flag=err)
        dY = torch.randn(Y.shape, generator=torch.Generator().manual_seed(100 + mb)).to(torch.bfloat16)
        dY_d = dY.to(DEV)
        ws = torch.empty(rl.workspace_bytes(rl.WS_FFN_BWD, cfg.N, 1, cfg.E, cfg.G, cfg.h, cfg.hff), dtype=torch.uint8, device=DEV)
        dX_deferred = rl.relibra_moe_ffn_bwd(dY_d, Xrows, Gt, U, A, tabs["group_offset"], tabs["group_expert"],
                                             tabs["group_dw_slot"], *W_d, None, None, None, err_flag=err, E=cfg.E,
                                             flags=rl.BWD_DEFER_WGRAD, workspace=ws)
        kept.append(dict(dYrows=dY_d, Xrows=Xrows, A=A, bwd_workspace=ws, inst_ptr=tabs["inst_ptr"],
                         inst_group=tabs["inst_group"], group_offset=tabs["group_offset"]))
        dX_full = rl.relibra_moe_ffn_bwd(dY_d, Xrows, Gt, U, A, tabs["group_offset"], tabs["group_expert"],
                                         tabs["group_dw_slot"], *W_d, *dW_mb, err_flag=err,
                                         flags=rl.BWD_ACCUMULATE if mb else 0)
        assert torch.equal(dX_deferred, dX_full)                 # the data gradients do not depend on the flag
        _, dWg_o, dWu_o, dWd_o = oracle.ffn_bwd(Xrows.cpu(), dY, p["group_offset"][mb], p["group_expert"][mb], Wg, Wu, Wd)
        for acc, o in zip(dW_ref, (dWg_o, dWu_o, dWd_o)):
            acc += o
    dW_b = [torch.full((cfg.E, *s), 3.0, dtype=torch.float32, device=DEV) for s in shapes]
    rl.relibra_moe_ffn_wgrad_batched(kept, cfg.E, *dW_b, err_flag=err)
    assert err.item() == 0
    for got, want, per_mb in zip(dW_b, dW_ref, dW_mb):
        assert rel_l2(got, want) <= TOL
        assert rel_l2(got, per_mb[:cfg.E].double().cpu().numpy()) <= 1e-5
    # the row gather fused in (token tensor + row -> token table instead of gathered rows): same operands,
    # same order, bit-identical weight gradients
    fused = [dict(m, Xrows=None, X=xd, row_tok=rt) for m, (xd, rt) in zip(kept, fused_in)]
    dW_f = [torch.empty((cfg.E, *s), dtype=torch.float32, device=DEV) for s in shapes]
    rl.relibra_moe_ffn_wgrad_batched(fused, cfg.E, *dW_f, err_flag=err)
    assert err.item() == 0
    for a_, b_ in zip(dW_f, dW_b):
        assert torch.equal(a_, b_)
    # both output tile shapes, forced (the default picks by contraction length): same sums, same order
    for tile in ("narrow", "wide"):
        for inputs in (kept, fused):
            dW_t = [torch.full((cfg.E, *s), float("nan"), dtype=torch.float32, device=DEV) for s in shapes]
            rl.relibra_moe_ffn_wgrad_batched(inputs, cfg.E, *dW_t, err_flag=err, tile=tile)
            assert err.item() == 0
            for a_, b_ in zip(dW_t, dW_b):
                assert torch.equal(a_, b_), tile
    once = [w.clone() for w in dW_b]
    rl.relibra_moe_ffn_wgrad_batched(kept, cfg.E, *dW_b, accumulate=True, err_flag=err)
    for got, one in zip(dW_b, once):
        assert torch.allclose(got, 2 * one, rtol=1e-6, atol=0)
    # a corrupted table is skipped and flagged, never dereferenced
    bad = dict(kept[1])
    bad["inst_group"] = kept[1]["inst_group"].clone()
    bad["inst_group"][0] = cfg.G + 5
    err2 = rl.relibra_moe_ffn_wgrad_batched([kept[0], bad, kept[2]], cfg.E, *dW_b)
    assert err2.item() == rl.ERR_GROUP_TABLE
    # an instance table that is not monotone (ranges of different experts overlap) lists more pieces than
    # a well-formed one can: the surplus is dropped and flagged, nothing is written past the piece arrays
    cap = kept[0]["inst_group"].shape[0]
    zig = dict(kept[0])
    zig["inst_ptr"] = dev_i32([0 if e % 2 == 0 else cap for e in range(cfg.E + 1)])
    err3 = rl.relibra_moe_ffn_wgrad_batched([zig] * rl.MAX_WGRAD_MB, cfg.E, *dW_b)
    torch.cuda.synchronize()
    assert err3.item() == rl.ERR_GROUP_TABLE


# ------------------------------------------------------------------ transposed weights for the data gradients
@pytest.mark.parametrize("n,a,b", [(3, 64, 64), (2, 192, 256), (5, 72, 136), (1, 8, 8)])
def test_transpose_experts_is_exact(n, a, b):
    W = torch.randn((n, a, b), generator=torch.Generator().manual_seed(a + b)).to(torch.bfloat16).to(DEV)
    got = rl.relibra_transpose_experts(W)
    assert torch.equal(got, W.transpose(1, 2).contiguous())


@pytest.mark.parametrize("a,b", [(128, 128), (120, 136), (264, 8), (8, 248), (136, 392)])
def test_transpose_experts_at_tile_edges(a, b):
    W = torch.randn((3, a, b), generator=torch.Generator().manual_seed(a * b)).to(torch.bfloat16).to(DEV)
    out = torch.full((4, b, a), 7.0, dtype=torch.bfloat16, device=DEV)
    rl.relibra_transpose_experts(W, out[:3])
    assert torch.equal(out[:3], W.transpose(1, 2).contiguous()) and (out[3] == 7.0).all()


@pytest.mark.parametrize("case", [FFN_CASES[0], FFN_CASES[3], FFN_CASES[4]])
def test_backward_with_transposed_weights_matches_oracle_and_the_plain_layout(case):
    """The data gradients read their weights from transposed copies: same mathematics, so the
    result must meet the oracle's bar and agree with the plain-layout kernels."""
    go, ge, X, dY, Wg, Wu, Wd = ffn_case(**case)
    E = case["E"]
    slots, n_slots = dw_slots(ge, E)
    dev = lambda a: a.to(DEV)
    Xd, dYd, W_d = dev(X), dev(dY), [dev(W) for W in (Wg, Wu, Wd)]
    W_t = [rl.relibra_transpose_experts(W) for W in W_d]
    go_d, ge_d, sl_d = dev_i32(go), dev_i32(ge), dev_i32(slots)
    err = rl.new_err_flag()
    Gt, U, A, Y = rl.relibra_moe_ffn_fwd(Xd, go_d, ge_d, *W_d, err_flag=err)
    outs = []
    for W3, flags in ((W_d, 0), (W_t, rl.BWD_TRANSPOSED_WEIGHTS)):
        dW = [torch.zeros((n_slots, *s), dtype=torch.float32, device=DEV)
              for s in ((case["hff"], case["h"]), (case["hff"], case["h"]), (case["h"], case["hff"]))]
        dX = rl.relibra_moe_ffn_bwd(dYd, Xd, Gt, U, A, go_d, ge_d, sl_d, *W3, *dW, flags=flags, err_flag=err, E=E)
        outs.append((dX, *dW))
    assert err.item() == 0
    live = np.concatenate([np.arange(go[g], go[g + 1]) for g in range(len(ge)) if ge[g] >= 0 and go[g + 1] > go[g]])
    lv = torch.from_numpy(live).to(DEV)
    assert rel_l2(outs[1][0][lv], outs[0][0][lv].double().cpu().numpy()) <= 1e-6      # data gradients: same sums
    for a_, b_ in zip(outs[0][1:], outs[1][1:]):
        assert torch.equal(a_, b_)                                                    # weight gradients do not read W
    dX_o, _, _, _ = oracle.ffn_bwd(X, dY, go, ge, Wg, Wu, Wd)
    assert rel_l2(outs[1][0][lv], dX_o[live]) <= TOL


@pytest.mark.parametrize("case", [FFN_CASES[0], FFN_CASES[3], FFN_CASES[4]])
def test_forward_with_transposed_weights_is_bit_identical(case):
    """Forward GEMMs reading transposed weight copies multiply the same operands in the same
    order: every stored tensor must equal the plain-layout result bit for bit (which the other
    tests hold against the oracle)."""
    go, ge, X, dY, Wg, Wu, Wd = ffn_case(**case)
    Xd, W_d = X.to(DEV), [W.to(DEV) for W in (Wg, Wu, Wd)]
    W_t = [rl.relibra_transpose_experts(W) for W in W_d]
    go_d, ge_d = dev_i32(go), dev_i32(ge)
    err = rl.new_err_flag()
    plain = rl.relibra_moe_ffn_fwd(Xd, go_d, ge_d, *W_d, err_flag=err)
    mk = lambda t: torch.zeros_like(t)
    swapped = rl.relibra_moe_ffn_fwd(Xd, go_d, ge_d, *W_t, Gt=mk(plain[0]), U=mk(plain[1]), A=mk(plain[2]), Yrows=mk(plain[3]),
                                     err_flag=err, flags=rl.FWD_TRANSPOSED_WEIGHTS)
    assert err.item() == 0
    live = np.concatenate([np.arange(go[g], go[g + 1]) for g in range(len(ge)) if ge[g] >= 0 and go[g + 1] > go[g]])
    lv = torch.from_numpy(live).to(DEV)
    for a_, b_ in zip(plain, swapped):
        assert torch.equal(a_[lv], b_[lv])
    Y_o = oracle.ffn_fwd(X, go, ge, Wg, Wu, Wd)[3]
    assert rel_l2(swapped[3][lv], Y_o[live]) <= TOL


def many_group_case(seed, h, hff):
    """Rows of every kind of tile in the first groups, then enough short groups that the wide tiles are taken."""
    rng = np.random.default_rng(seed)
    first = (300, 64, 65, 1, 0, 130)
    rows = (*first, *rng.integers(1, 9, 160).tolist())
    case = ffn_case(seed=seed, E=3, h=h, hff=hff, rows=rows, experts=(1, 0, 2, 1, -1, 0, *rng.integers(0, 3, 160).tolist()))
    return len(first), case


@pytest.mark.parametrize("h,hff", [(k, 512) for k in (64, 256, 320, 384, 448, 512, 576, 640, 704, 768, 832, 896)]
                         + [(1024, k) for k in (256, 320, 384, 512, 576, 640, 704, 768, 832)] + [(960, 1472), (1472, 704), (512, 960)])
def test_wide_tiles_on_weights_as_stored(h, hff):
    """The wide tiles take k-contiguous weights 64 k-values of one half of their columns at a time.  Contractions
    of every remainder of a trip through the LDS rings, row tiles of both heights, output widths that the tiles
    do not divide: bit for bit what the same products on transposed copies give, and within the bar of the oracle."""
    n_first, (go, ge, X, dY, Wg, Wu, Wd) = many_group_case(h + hff, h, hff)
    Xd, dYd, W_d = X.to(DEV), dY.to(DEV), [W.to(DEV) for W in (Wg, Wu, Wd)]
    W_t = [rl.relibra_transpose_experts(W) for W in W_d]
    go_d, ge_d, sl_d = dev_i32(go), dev_i32(ge), dev_i32(np.maximum(ge, 0))
    err = rl.new_err_flag()
    mk = lambda cols: torch.zeros((X.shape[0], cols), dtype=torch.bfloat16, device=DEV)
    outs = []
    for W3, ffl, bfl in ((W_d, 0, 0), (W_t, rl.FWD_TRANSPOSED_WEIGHTS, rl.BWD_TRANSPOSED_WEIGHTS)):
        out = rl.relibra_moe_ffn_fwd(Xd, go_d, ge_d, *W3, Gt=mk(hff), U=mk(hff), A=mk(hff), Yrows=mk(h), err_flag=err, flags=ffl)
        dX = rl.relibra_moe_ffn_bwd(dYd, None, *out[:3], go_d, ge_d, sl_d, *W3, None, None, None, dXrows=mk(h), err_flag=err, E=3,
                                    flags=bfl | rl.BWD_DEFER_WGRAD)
        outs.append((*out, dX))
    assert err.item() == 0
    for plain, swapped in zip(*outs):
        assert torch.equal(plain, swapped)
    # the short groups are checked through the transposed copies' kernels, the first ones against the oracle
    n = go[n_first]
    go_o, ge_o = go[:n_first + 1], ge[:n_first]
    for got, want in zip(outs[0], (*oracle.ffn_fwd(X[:n], go_o, ge_o, Wg, Wu, Wd), oracle.ffn_bwd(X[:n], dY[:n], go_o, ge_o, Wg, Wu, Wd)[0])):
        assert rel_l2(got[:n], want) <= TOL


@pytest.mark.parametrize("groups", [20, 166], ids=["few-tiles", "many-tiles"])
def test_weight_gradients_of_short_groups(groups):
    """Both rings of the small weight-gradient tile: calls of few tiles, and of more than two per compute unit."""
    _, (go, ge, X, dY, Wg, Wu, Wd) = many_group_case(groups, 256, 320)
    go, ge = go[:groups + 1], ge[:groups]
    N = int(go[-1])
    X, dY = X[:N], dY[:N]
    slots, n_slots = dw_slots(ge, 3)
    go_d, ge_d, W_d, err = dev_i32(go), dev_i32(ge), [W.to(DEV) for W in (Wg, Wu, Wd)], rl.new_err_flag()
    Gt, U, A, _ = rl.relibra_moe_ffn_fwd(X.to(DEV), go_d, ge_d, *W_d, err_flag=err)
    dW = [torch.full((n_slots, *W.shape[1:]), 3.0, dtype=torch.float32, device=DEV) for W in (Wg, Wu, Wd)]
    rl.prof_start(level=1, max_records=16)
    rl.relibra_moe_ffn_bwd(dY.to(DEV), X.to(DEV), Gt, U, A, go_d, ge_d, dev_i32(slots), *W_d, *dW, err_flag=err, E=3)
    timed = set(rl.prof_stop())
    assert err.item() == 0
    assert timed == {"bwd_act", "bwd_dx"} | ({"wgrad_pair"} if groups == 20 else {"wgrad_down", "wgrad_gate_up"})
    for got, want in zip(dW, oracle.ffn_bwd(X, dY, go, ge, Wg, Wu, Wd)[1:]):
        for e in range(3):
            assert rel_l2(got[e], want[e]) <= TOL


@pytest.mark.parametrize("E,h,hff,bounds", [
    (66, 320, 448, ((129, 290), (380, 580))),              # a last round that is nearly empty: the smaller tiles
    (64, 448, 448, ((129, 290), (380, 580))),              # 256 x 256 tiles where written, ragged rows and outputs
    (64, 448, 512, ((1520, 1640),)),                       # 256 x 256 tiles where written and where added to
])
def test_weight_gradients_of_many_rows_per_group(E, h, hff, bounds):
    """The 256 x 256 tiles of the per-micro-batch weight gradients and the smaller ones beside them."""
    err = rl.new_err_flag()
    rng = np.random.default_rng(5)
    for lo, hi in bounds:
        rows = rng.integers(lo, hi, E)
        go, ge, X, dY, Wg, Wu, Wd = ffn_case(seed=lo, E=E, h=h, hff=hff, rows=rows, experts=range(E))
        go_d, ge_d, W_d = dev_i32(go), dev_i32(ge), [W.to(DEV) for W in (Wg, Wu, Wd)]
        Xd, dYd = X.to(DEV), dY.to(DEV)
        Gt, U, A, _ = rl.relibra_moe_ffn_fwd(Xd, go_d, ge_d, *W_d, err_flag=err)
        dW = [torch.full(W.shape, 3.0, dtype=torch.float32, device=DEV) for W in (Wg, Wu, Wd)]
        run = lambda flags: rl.relibra_moe_ffn_bwd(dYd, Xd, Gt, U, A, go_d, ge_d, ge_d, *W_d, *dW, err_flag=err, flags=flags)
        run(0)
        once = [w.double() for w in dW]
        run(rl.BWD_ACCUMULATE)
        assert err.item() == 0
        g, u, dA = Gt.double(), U.double(), torch.cat([dYd[go[e]:go[e + 1]].double() @ W_d[2][e].double() for e in range(E)])
        sg = torch.sigmoid(g)
        dG, dU = dA * u * sg * (1 + g * (1 - sg)), dA * g * sg
        for e in range(E):
            at = slice(go[e], go[e + 1])
            for got, twice, want in zip(once, dW, (dG[at].T @ Xd[at].double(), dU[at].T @ Xd[at].double(), dYd[at].double().T @ A[at].double())):
                assert rel_l2(got[e], want.cpu().numpy()) <= TOL
                assert rel_l2(twice[e], 2 * got[e].cpu().numpy()) <= 1e-6


@pytest.mark.parametrize("weights_t", [False, True], ids=["stored-layout", "transposed-copies"])
@pytest.mark.parametrize("h,hff", [(512, 1024), (960, 1472), (512, 960), (576, 1024), (704, 1536)])
def test_gate_fused_backward_on_wide_tiles(h, hff, weights_t):
    """Gates that are powers of two scale without rounding: the gate-fused data gradients then equal, bit for bit,
    the unfused ones on the scaled rows; dgate = <dOut, Y> within the bar.  Wide tiles, also where they reach
    beyond the columns."""
    _, (go, ge, X, dY, Wg, Wu, Wd) = many_group_case(7 * h + hff, h, hff)
    N = X.shape[0]
    gate = torch.from_numpy(np.random.default_rng(h).choice([0.25, 0.5, 1.0, 2.0], N).astype(np.float32)).to(DEV)
    tok = torch.arange(N, dtype=torch.int32, device=DEV)
    Xd, dO, W_d = X.to(DEV), dY.to(DEV), [W.to(DEV) for W in (Wg, Wu, Wd)]
    go_d, ge_d, sl_d = dev_i32(go), dev_i32(ge), dev_i32(np.maximum(ge, 0))
    err = rl.new_err_flag()
    Gt, U, A, Y = rl.relibra_moe_ffn_fwd(Xd, go_d, ge_d, *W_d, err_flag=err)
    guard = 1 << 16
    need = rl.workspace_bytes(rl.WS_DGATE, N, 1, 3, len(ge), h, hff)
    scratch = torch.full((need + guard,), 99, dtype=torch.uint8, device=DEV)
    W_b, flags = ([rl.relibra_transpose_experts(W) for W in W_d], rl.BWD_TRANSPOSED_WEIGHTS) if weights_t else (W_d, 0)
    got, dgate = rl.relibra_moe_ffn_bwd_gated(dO, tok, gate, Gt, U, go_d, ge_d, sl_d, *W_b, E=3, dgate_scratch=scratch, err_flag=err,
                                              flags=flags)
    want = rl.relibra_moe_ffn_bwd((gate[:, None] * dO.float()).to(torch.bfloat16), None, Gt, U, A, go_d, ge_d, sl_d, *W_d, None, None, None,
                                  E=3, flags=rl.BWD_DEFER_WGRAD, err_flag=err)
    assert err.item() == 0
    live = torch.from_numpy(np.concatenate([np.arange(go[g], go[g + 1]) for g in range(len(ge)) if ge[g] >= 0])).to(DEV)
    assert torch.equal(got[live], want[live])
    assert rel_l2(dgate[live], (dO.double() * Y.double()).sum(1)[live].cpu().numpy()) <= TOL
    assert (scratch[need:] == 99).all()


# ------------------------------------------------------------------ row gather fused into the GEMMs
def test_forward_with_fused_row_gather_is_bit_identical():
    """relibra_moe_ffn_fwd_gather reads row `row` as X[row_tok[row]]: the same operands in the same
    order as the two-step form (gather, then forward), so every output must match bit for bit;
    row_tok itself is checked against the oracle's permutation."""
    cfg = wl.small_config(E=16, k=4, EP=4, r=2, T=777, n_mb=2, h=256, hff=192)
    ids, gates = routing(cfg)
    counts = oracle.route_hist(ids, cfg.E)[0]
    p = plan_both(cfg, counts)
    Wg, Wu, Wd = [W.to(DEV) for W in wl.make_weights(cfg)]
    for mb in range(cfg.n_mb):
        X, _ = wl.make_tokens(cfg, mb)
        Xd = X.to(DEV)
        tabs = {key: dev_i32(p[key][mb]) for key in ("inst_ptr", "inst_rows", "inst_group", "group_offset", "group_expert")}
        ids_d = torch.from_numpy(ids[mb]).to(DEV)
        err = rl.new_err_flag()
        row_of, src_of, Xrows = rl.relibra_permute(ids_d, tabs["inst_ptr"], tabs["inst_rows"], tabs["inst_group"],
                                                   tabs["group_offset"], Xd, cfg.E, cfg.G, err_flag=err)
        row_tok = rl.relibra_row_tokens(src_of, cfg.k, cfg.T, err_flag=err)
        _, src_o = oracle.permute(ids[mb], cfg.E, p["inst_ptr"][mb], p["inst_rows"][mb], p["inst_group"][mb], p["group_offset"][mb])
        assert np.array_equal(row_tok.cpu().numpy(), src_o // cfg.k)
        two_step = rl.relibra_moe_ffn_fwd(Xrows, tabs["group_offset"], tabs["group_expert"], Wg, Wu, Wd, err_flag=err)
        fused = rl.relibra_moe_ffn_fwd_gather(Xd, row_tok, tabs["group_offset"], tabs["group_expert"], Wg, Wu, Wd, err_flag=err)
        assert err.item() == 0
        for a, b in zip(two_step, fused):
            assert torch.equal(a, b)
        # and together with transposed weight copies (the benchmark's default forward)
        W_t = [rl.relibra_transpose_experts(W) for W in (Wg, Wu, Wd)]
        both = rl.relibra_moe_ffn_fwd_gather(Xd, row_tok, tabs["group_offset"], tabs["group_expert"], *W_t, err_flag=err,
                                             flags=rl.FWD_TRANSPOSED_WEIGHTS)
        assert err.item() == 0
        for a, b in zip(two_step, both):
            assert torch.equal(a, b)
    bad = src_of.clone()
    bad[3] = cfg.T * cfg.k + 7
    err = rl.new_err_flag()
    rt = rl.relibra_row_tokens(bad, cfg.k, cfg.T, err_flag=err)
    assert err.item() == rl.ERR_PLAN_COVER and rt[3].item() == 0


# ------------------------------------------------------------------ gate-side fusion of the backward
@pytest.mark.parametrize("hff", [320, 512], ids=["ragged-dA-tiles", "whole-dA-tiles"])
@pytest.mark.parametrize("weights_t", [False, True], ids=["stored-layout", "transposed-copies"])
def test_gate_fused_backward_matches_the_unfused_definition(weights_t, hff):
    """The combine (Section 2.1: gate-weighted sum of the selected experts' outputs) is linear, so its
    backward may move into the expert backward: dOut rows read straight from the token tensor, the gate
    applied to dA, dgate as a row reduction of dA' against A, dWd from dOut rows against gate * A.  The
    oracle computes the unfused definition (combine backward, then expert backward); the fused path must
    agree within the floating-point tolerance on dX, dgate and all three weight gradients, its forward
    outputs must equal the unfused forward's bit for bit, and two runs must agree bit for bit."""
    cfg = wl.small_config(E=16, k=4, EP=4, r=2, T=777, n_mb=2, h=512, hff=hff)
    ids, gates = routing(cfg)
    counts = oracle.route_hist(ids, cfg.E)[0]
    p = plan_both(cfg, counts)
    Wg, Wu, Wd = wl.make_weights(cfg)
    W_d = [W.to(DEV) for W in (Wg, Wu, Wd)]
    W_f = [rl.relibra_transpose_experts(W) for W in W_d] if weights_t else W_d       # forward operands
    f_flags = rl.FWD_TRANSPOSED_WEIGHTS if weights_t else 0
    shapes = [(cfg.hff, cfg.h), (cfg.hff, cfg.h), (cfg.h, cfg.hff)]
    dW_ref = [np.zeros((cfg.E, *s)) for s in shapes]
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    err = rl.new_err_flag()
    kept = []
    for mb in range(cfg.n_mb):
        X, dOut = wl.make_tokens(cfg, mb)
        Xd, dOut_d, gates_d = X.to(DEV), dOut.to(DEV), t(gates[mb])
        tabs = {key: dev_i32(p[key][mb]) for key in ("inst_ptr", "inst_rows", "inst_group", "group_offset",
                                                     "group_expert", "group_dw_slot")}
        row_of, src_of, _ = rl.relibra_permute(t(ids[mb]), tabs["inst_ptr"], tabs["inst_rows"], tabs["inst_group"],
                                               tabs["group_offset"], Xd, cfg.E, cfg.G, err_flag=err)
        row_tok = rl.relibra_row_tokens(src_of, cfg.k, cfg.T, err_flag=err)
        row_gate = rl.relibra_row_gates(src_of, gates_d, err_flag=err)
        row_of_o, src_o = oracle.permute(ids[mb], cfg.E, p["inst_ptr"][mb], p["inst_rows"][mb], p["inst_group"][mb],
                                         p["group_offset"][mb])
        assert np.array_equal(row_gate.cpu().numpy(), gates[mb].reshape(-1)[src_o])
        # forward: everything the ungated call writes, bit for bit, plus Ag = gate * A
        plain = rl.relibra_moe_ffn_fwd_gather(Xd, row_tok, tabs["group_offset"], tabs["group_expert"], *W_f, err_flag=err, flags=f_flags)
        Gt, U, A, Ag, Y = rl.relibra_moe_ffn_fwd_gated(Xd, row_tok, row_gate, tabs["group_offset"], tabs["group_expert"], *W_f,
                                                       err_flag=err, flags=f_flags)
        for a_, b_ in zip(plain, (Gt, U, A, Y)):
            assert torch.equal(a_, b_)
        Xrows_o = oracle.gather_rows(X, src_o, cfg.k)
        go, ge = p["group_offset"][mb], p["group_expert"][mb]
        _, _, A_o, Y_o = oracle.ffn_fwd(Xrows_o, go, ge, Wg, Wu, Wd)
        assert rel_l2(Ag, gates[mb].reshape(-1)[src_o][:, None].astype(np.float64) * A_o) <= TOL
        # gated in place (A and Ag the same tensor): same Gt, U and Ag; rows come out gate-scaled, the combine is a sum
        A_ip = torch.empty_like(A)
        Gt_p, U_p, _, Ag_p, Y_p = rl.relibra_moe_ffn_fwd_gated(Xd, row_tok, row_gate, tabs["group_offset"], tabs["group_expert"],
                                                               *W_f, A=A_ip, Ag=A_ip, err_flag=err, flags=f_flags)
        assert torch.equal(Gt_p, Gt) and torch.equal(U_p, U) and torch.equal(Ag_p, Ag)
        Out_p = rl.relibra_unpermute_combine(rl.COMBINE_SUM, Y_p, row_of, cfg.T, cfg.k, err_flag=err)
        assert rel_l2(Out_p, oracle.combine_fwd(Y_o, gates[mb], row_of_o, cfg.T, cfg.k)) <= TOL
        # backward
        ws = torch.empty(rl.workspace_bytes(rl.WS_FFN_BWD, cfg.N, 1, cfg.E, cfg.G, cfg.h, cfg.hff), dtype=torch.uint8, device=DEV)
        b_flags = rl.BWD_TRANSPOSED_WEIGHTS if weights_t else 0
        W_b = W_f if weights_t else W_d
        dgate = torch.full((cfg.T, cfg.k), float("nan"), dtype=torch.float32, device=DEV)
        dXrows, _ = rl.relibra_moe_ffn_bwd_gated(dOut_d, row_tok, row_gate, Gt, U, tabs["group_offset"], tabs["group_expert"],
                                                 tabs["group_dw_slot"], *W_b, src_of=src_of, flags=b_flags, dgate=dgate,
                                                 workspace=ws, err_flag=err, E=cfg.E)
        dXrows2, dgate_rows = rl.relibra_moe_ffn_bwd_gated(dOut_d, row_tok, row_gate, Gt, U, tabs["group_offset"],
                                                           tabs["group_expert"], tabs["group_dw_slot"], *W_b, flags=b_flags,
                                                           err_flag=err, E=cfg.E)
        assert torch.equal(dXrows, dXrows2)                                       # reproducible
        assert torch.equal(dgate.reshape(-1)[src_of.long()], dgate_rows)          # the two dgate layouts
        dX = rl.relibra_unpermute_combine(rl.COMBINE_SUM, dXrows, row_of, cfg.T, cfg.k, err_flag=err)
        # oracle: the unfused definition
        dY_o, dgate_o = oracle.combine_bwd(dOut.double().numpy(), Y_o, gates[mb], row_of_o, cfg.T, cfg.k)
        dY16 = torch.from_numpy(dY_o).to(torch.bfloat16)
        dXrows_o, dWg_o, dWu_o, dWd_o = oracle.ffn_bwd(Xrows_o, dY16, go, ge, Wg, Wu, Wd)
        dX_o = oracle.combine_fwd(dXrows_o, None, row_of_o, cfg.T, cfg.k)
        assert rel_l2(dX, dX_o) <= TOL
        assert rel_l2(dgate, dgate_o) <= TOL
        for acc, o in zip(dW_ref, (dWg_o, dWu_o, dWd_o)):
            acc += o
        kept.append(dict(dOut=dOut_d, X=Xd, row_tok=row_tok, A=Ag, bwd_workspace=ws, inst_ptr=tabs["inst_ptr"],
                         inst_group=tabs["inst_group"], group_offset=tabs["group_offset"]))
    assert err.item() == 0
    for tile in (None, "narrow", "wide"):
        dW = [torch.full((cfg.E, *s), float("nan"), dtype=torch.float32, device=DEV) for s in shapes]
        rl.relibra_moe_ffn_wgrad_batched(kept, cfg.E, *dW, err_flag=err, tile=tile)
        assert err.item() == 0
        for got, want in zip(dW, dW_ref):
            assert rel_l2(got, want) <= TOL, tile
        if tile is None:
            first = dW
        else:
            for a_, b_ in zip(dW, first):
                assert torch.equal(a_, b_), tile
    # argument checks: the fused backward needs its scratch, and a bad src_of entry is flagged, not followed
    with pytest.raises(rl.RelibraError):
        rl.relibra_moe_ffn_bwd_gated(dOut_d, row_tok, row_gate, Gt, U, tabs["group_offset"], tabs["group_expert"],
                                     tabs["group_dw_slot"], *W_b, flags=b_flags, E=cfg.E,
                                     dgate_scratch=torch.empty(256, dtype=torch.uint8, device=DEV))
    bad = src_of.clone()
    bad[5] = cfg.N + 3
    err2 = rl.new_err_flag()
    rl.relibra_moe_ffn_bwd_gated(dOut_d, row_tok, row_gate, Gt, U, tabs["group_offset"], tabs["group_expert"],
                                 tabs["group_dw_slot"], *W_b, src_of=bad, flags=b_flags, err_flag=err2, E=cfg.E,
                                 dgate=torch.zeros(cfg.N, dtype=torch.float32, device=DEV))
    assert err2.item() == rl.ERR_PLAN_COVER
