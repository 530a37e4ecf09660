"""Parity of the HIP search (through the C ABI) with the CPU oracle.

Bar: bit-exact per-node fronts and goal fronts (the label vectors are unique,
see the oracle's header); witnesses may differ and are checked by re-walking
their paths.
"""
import dataclasses

import numpy as np
import pytest

from oracle import checks, graph as ograph, search as osearch
from paper_1705_02408_amd import synth
from tests.graphs import as_vecs, from_edges, load_golden

pytestmark = pytest.mark.gpu

mpap = pytest.importorskip("paper_1705_02408_amd.mpap")


def bits(a):
    return np.ascontiguousarray(a, dtype=np.float32).view(np.uint32)


def sort_lex(v):
    v = np.asarray(v, dtype=np.float32).reshape(-1, 3)
    if v.shape[0] == 0:
        return v
    return v[np.lexsort((v[:, 2], v[:, 1], v[:, 0]))]


def upload(g):
    return mpap.mpap_graph_from_csr(g["row_ptr"], g["col"], g["cost"], g["drift"], g["reset"],
                                    g["goal"])


def run(g, beta, n_obj, radius=1.0, lam=0.5, **kw):
    dg = upload(g)
    res = mpap.mpap_search(dg, beta, n_obj, radius, lam, **kw)
    return dg, res


def check_against_oracle(g, res, ref, beta, n_obj, all_nodes=True, node_stride=1):
    n = g["row_ptr"].shape[0] - 1
    st = res.stats()
    assert st["front_labels"] == ref.X
    nodes = range(n) if all_nodes else range(0, n, node_stride)
    for v in nodes:
        a = sort_lex(res.node_front(v))
        b = ref.node_front(v)
        assert a.shape == b.shape, (v, a.shape, b.shape)
        assert np.array_equal(bits(a), bits(b)), v
    fr = res.goal_front()
    rv, _, _ = osearch.goal_front(ref, g["goal"])
    assert fr.vecs.shape == rv.shape
    assert np.array_equal(bits(fr.vecs), bits(rv))
    # witnesses: each path re-walks to its vector, feasibly, ending in a goal node
    for k in range(fr.vecs.shape[0]):
        path = res.path(int(fr.label[k]))
        assert path[0] == 0 and path[-1] == fr.goal_node[k] and g["goal"][path[-1]]
        c, d, m, ok = osearch.rewalk(g, path, beta, n_obj)
        assert ok
        assert bits([c, d, m if n_obj == 3 else 0.0]).tolist() == bits(fr.vecs[k]).tolist()
    return st


# ------------------------------------------------------------ tiny graphs
@pytest.mark.parametrize("seed,n,p_reset,n_obj,ints,beta", [
    (0, 30, 0.0, 2, False, 0.9), (1, 30, 0.0, 3, False, 0.9), (2, 30, 0.0, 2, True, 1.0),
    (5, 14, 0.3, 3, False, 0.6), (6, 14, 0.3, 2, True, 0.75), (10, 12, 0.25, 3, True, 0.5),
    (12, 200, 0.2, 2, False, 0.8), (13, 200, 0.2, 3, True, 1.0),
])
def test_tiny_graphs(seed, n, p_reset, n_obj, ints, beta):
    g = synth.tiny_random_graph(seed, n=n, p_reset=p_reset, mean_degree=3.0, integer_costs=ints)
    ref = osearch.search(g, beta, n_obj)
    dg, res = run(g, beta, n_obj, radius=0.25)
    check_against_oracle(g, res, ref, beta, n_obj)
    res.close()
    dg.close()


@pytest.mark.parametrize("name,n_obj", [("narrow_passage.json", 2), ("diamond_reset.json", 2),
                                        ("diamond_reset.json", 3)])
def test_golden(name, n_obj):
    spec, g = load_golden(name)
    dg, res = run(g, spec["beta"], n_obj)
    fr = res.goal_front()
    want = spec.get("expected_goal_front") or spec["cases"][str(n_obj)]["goal_front"]
    assert np.array_equal(bits(fr.vecs), bits(as_vecs(want)))
    res.close()
    dg.close()


# ------------------------------------------------------------ roadmaps
@pytest.fixture(scope="module")
def road2d():
    out = {}
    for seed in (0, 1, 2):
        env = synth.plain2d(seed)
        out[seed] = (env, ograph.build_graph(env))
    return out


@pytest.mark.parametrize("seed", [0, 1, 2])
def test_plain2d_full_parity(road2d, seed):
    env, g = road2d[seed]
    ref = osearch.search(g, env.beta, 2)
    dg, res = run(g, env.beta, 2, radius=env.radius, lam=env.lam)
    st = check_against_oracle(g, res, ref, env.beta, 2)
    assert st["labels_expanded"] >= ref.X
    res.close()
    dg.close()


@pytest.mark.parametrize("lam", [0.125, 0.5, 1.0, 4.0, 1e6])
def test_group_factor_does_not_change_fronts(road2d, lam):
    env, g = road2d[0]
    ref = osearch.search(g, env.beta, 2)
    dg, res = run(g, env.beta, 2, radius=env.radius, lam=lam)
    check_against_oracle(g, res, ref, env.beta, 2, all_nodes=False, node_stride=7)
    res.close()
    dg.close()


@pytest.mark.parametrize("beta", [0.0, 0.05, np.inf])
def test_bound_edge_cases(road2d, beta):
    env, g = road2d[1]
    ref = osearch.search(g, beta, 2)
    dg, res = run(g, beta, 2, radius=env.radius)
    check_against_oracle(g, res, ref, beta, 2, all_nodes=False, node_stride=3)
    res.close()
    dg.close()


def test_plain3d_small_three_objectives():
    env = synth.plain3d(0, n=3000)
    g = ograph.build_graph(env)
    ref = osearch.search(g, env.beta, 3)
    dg, res = run(g, env.beta, 3, radius=env.radius)
    check_against_oracle(g, res, ref, env.beta, 3)
    res.close()
    dg.close()


@pytest.mark.parametrize("threads", [256, 512])
@pytest.mark.parametrize("dim", [2, 3])
def test_workgroup_size_does_not_change_fronts(threads, dim):
    """Two or four workgroups per CU (smaller LDS stages, more spills) give the
    oracle's fronts bit for bit."""
    env = synth.plain2d(5, n=2000) if dim == 2 else synth.plain3d(2, n=3000)
    g = ograph.build_graph(env)
    ref = osearch.search(g, env.beta, env.n_obj)
    dg, res = run(g, env.beta, env.n_obj, radius=env.radius, block_threads=threads)
    assert res.stats()["blocks"] == 256 * (1024 // threads)
    assert res.stats()["wave_build"] == 0
    check_against_oracle(g, res, ref, env.beta, env.n_obj, all_nodes=False, node_stride=2)
    res.close()
    dg.close()


@pytest.mark.parametrize("case,stage_cap", [("tiny3", 0), ("2d", 0), ("3d", 0), ("3d", 64),
                                             ("2d", 128)])
def test_single_wave_merges(case, stage_cap):
    """Every iteration merged by single waves (small fronts) and workgroups
    (large ones, and fronts that outgrow a wave's slice: stage_cap shrinks the
    slice so that many do) gives the oracle's fronts bit for bit."""
    if case == "tiny3":
        g = synth.tiny_random_graph(13, n=200, p_reset=0.2, mean_degree=3.0, integer_costs=True)
        beta, n_obj, radius = 1.0, 3, 0.25
    else:
        env = synth.plain2d(6, n=2000) if case == "2d" else synth.plain3d(3, n=3000)
        g = ograph.build_graph(env)
        beta, n_obj, radius = env.beta, env.n_obj, env.radius
    ref = osearch.search(g, beta, n_obj)
    dg, res = run(g, beta, n_obj, radius=radius, wave_min_targets=1, stage_cap=stage_cap)
    assert res.stats()["wave_build"] == 1
    check_against_oracle(g, res, ref, beta, n_obj, all_nodes=False, node_stride=2)
    res.close()
    dg.close()


def test_deterministic(road2d):
    env, g = road2d[2]
    dg = upload(g)
    out = []
    for _ in range(2):
        res = mpap.mpap_search(dg, env.beta, 2, env.radius, env.lam)
        fr = res.goal_front()
        st = res.stats()
        out.append((bits(fr.vecs).tobytes(), fr.label.tobytes(), fr.goal_node.tobytes(),
                    st["labels_expanded"], st["waves"], st["merges"], st["candidates"]))
        res.close()
    assert out[0] == out[1]
    dg.close()


# ------------------------------------------------------------ edge cases
def test_no_goal_gives_empty_front(road2d):
    env, g = road2d[0]
    g2 = dict(g)
    g2["goal"] = np.zeros_like(g["goal"])
    dg, res = run(g2, env.beta, 2, radius=env.radius)
    assert res.goal_front().vecs.shape == (0, 3)
    res.close()
    dg.close()


def test_isolated_root():
    g = dict(row_ptr=np.array([0, 0, 1, 2], np.int32), col=np.array([2, 1], np.int32),
             cost=np.array([1.0, 1.0], np.float32), drift=np.array([0.0, 0.0], np.float32),
             reset=np.zeros(3, np.uint8), goal=np.array([0, 0, 1], np.uint8))
    dg, res = run(g, 1.0, 2)
    assert res.goal_front().vecs.shape == (0, 3)
    assert sort_lex(res.node_front(0)).tolist() == [[0.0, 0.0, 0.0]]
    assert res.stats()["labels_expanded"] == 1
    res.close()
    dg.close()


def test_root_in_goal_and_nonzero_init_node():
    spec, g = load_golden("diamond_reset.json")
    g2 = dict(g)
    g2["goal"] = np.array([1, 0, 0, 0, 0], np.uint8)
    dg, res = run(g2, 1.0, 2)
    assert res.goal_front().vecs.tolist() == [[0.0, 0.0, 0.0]]
    res.close()
    res = mpap.mpap_search(dg, 1.0, 2, 1.0, 0.5, init_node=1)
    assert sort_lex(res.node_front(1)).tolist() == [[0.0, 0.0, 0.0]]
    res.close()
    dg.close()


def test_invalid_arguments_are_rejected():
    g = dict(row_ptr=np.array([0, 1, 1], np.int32), col=np.array([1], np.int32),
             cost=np.array([0.0], np.float32), drift=np.array([0.0], np.float32),
             reset=np.zeros(2, np.uint8), goal=np.array([0, 1], np.uint8))
    with pytest.raises(mpap.MpapError) as ei:
        upload(g)
    assert ei.value.status == mpap.MPAP_ERR_INVAL
    g["cost"][0] = 1.0
    g["col"][0] = 5
    with pytest.raises(mpap.MpapError):
        upload(g)
    g["col"][0] = 1
    dg = upload(g)
    for kw in (dict(n_obj=4), dict(init_node=7), dict(lam=0.0), dict(beta=np.nan)):
        args = dict(beta=1.0, n_obj=2, radius=1.0, lam=0.5)
        args.update(kw)
        with pytest.raises(mpap.MpapError) as ei:
            mpap.mpap_search(dg, **args)
        assert ei.value.status == mpap.MPAP_ERR_INVAL
    dg.close()


def test_wave_cap_reports_noconverge(road2d):
    env, g = road2d[0]
    dg = upload(g)
    with pytest.raises(mpap.MpapError) as ei:
        mpap.mpap_search(dg, env.beta, 2, env.radius, env.lam, max_waves=3)
    assert ei.value.status == mpap.MPAP_ERR_NOCONVERGE
    dg.close()


# ------------------------------------------------------------ graph build
@pytest.mark.parametrize("dim,n,seed", [(2, 2000, 0), (2, 2000, 3), (3, 3000, 1)])
def test_build_graph_matches_oracle(dim, n, seed):
    env = synth.plain2d(seed, n=n) if dim == 2 else synth.plain3d(seed, n=n)
    ref = ograph.build_graph(env)
    dg = mpap.mpap_build_graph(env)
    got = dg.export()
    dg.close()
    # neighbour sets (Near + Collision) and lengths: exact
    assert np.array_equal(got["row_ptr"], ref["row_ptr"])
    assert np.array_equal(got["col"], ref["col"])
    assert np.array_equal(bits(got["cost"]), bits(ref["cost"]))
    assert np.array_equal(got["goal"], ref["goal"])
    # drift and relocalisation flags: the same float64 evaluation of q
    # (summed in the same order, rounded once to float32) as the oracle, so
    # the same bits
    bad = np.nonzero(bits(got["drift"]) != bits(ref["drift"]))[0]
    assert bad.size == 0, (bad.size, bad[:8])
    assert np.array_equal(got["reset"], ref["reset"])


@pytest.mark.parametrize("n", [14, 15, 16, 17, 16383, 16384])
def test_goal_list_of_built_roadmaps(n):
    """The goal front of roadmaps whose node count (n + 1) lies around the 16
    flags a thread reads and the 16,384 of a round: the minimum over the nodes
    that the goal mask names, the last sample among them."""
    env = synth.plain2d(23, n=n)
    env = dataclasses.replace(env, goal=env.pos[-1].copy(), goal_radius=0.2 if n < 100 else 0.06,
                              box_lo=env.box_lo[:0], box_hi=env.box_hi[:0])
    dg = mpap.mpap_build_graph(env)
    goal = np.flatnonzero(dg.export()["goal"])
    assert goal[-1] == n and dg.info()["n_goal"] == goal.size
    res = mpap.mpap_search(dg, np.inf, 2, env.radius, 4.0)
    vecs = np.concatenate([res.node_front(int(v)) for v in goal])
    vecs = sort_lex(vecs)
    want, best = [], np.inf
    for row in vecs:
        if row[1] < best:
            want.append(row)
            best = row[1]
    assert np.array_equal(bits(res.goal_front().vecs), bits(np.array(want).reshape(-1, 3)))
    res.close()
    dg.close()


@pytest.mark.parametrize("dim,n,boxes", [(2, 300, 0), (2, 300, 1), (2, 700, 64), (3, 700, 65),
                                         (3, 40, 129), (3, 1500, 200)])
def test_obstacles_by_the_wave(dim, n, boxes):
    """Edges against 0 to 200 boxes (none, one word of 64, one more, several;
    waves with one source, with many and partly filled), some of them thin,
    some touching samples: the oracle's edges."""
    env = synth.plain2d(17, n=n) if dim == 2 else synth.plain3d(17, n=n)
    rng = np.random.default_rng(boxes)
    lo = rng.uniform(0.0, 0.95, (boxes, dim)).astype(np.float32)
    hi = lo + rng.choice([0.0, 0.002, 0.03, 0.08], (boxes, dim)).astype(np.float32)
    if boxes > 1:
        lo[1] = hi[1] = env.pos[5]
    env = dataclasses.replace(env, box_lo=lo, box_hi=hi, goal=env.pos[-1].copy(),
                              goal_radius=0.3)
    ref = ograph.build_graph(env)
    dg = mpap.mpap_build_graph(env)
    got = dg.export()
    for k in ("row_ptr", "col"):
        assert np.array_equal(got[k], ref[k]), k
    assert np.array_equal(bits(got["cost"]), bits(ref["cost"]))
    dg.close()


@pytest.mark.parametrize("dim,n,what", [
    (2, 400, "many points"), (3, 300, "many points"), (2, 400, "narrow blobs"),
    (3, 300, "narrow blobs"), (2, 400, "far blobs"), (3, 300, "no blobs"),
    (2, 6000, "few blobs"), (2, 14000, "few blobs"), (3, 9000, "few blobs")])
def test_drift_along_segments(dim, n, what):
    """The drift by products along each segment against the oracle's
    exponential per midpoint: segments of more midpoints than one run, blobs
    so narrow that their first value would underflow, blobs out of reach, and
    roadmaps large enough for two lanes and one lane per pair.  The float64
    sums agree to 2e-13 relative, so the float32 values differ at most by one
    rounding, and by that in less than 1e-4 of the edges (2e-13 / 2^-24 is
    3e-6)."""
    env = synth.plain2d(8, n=n) if dim == 2 else synth.plain3d(8, n=n)
    kw = dict(goal=env.pos[-1].copy())
    if what == "many points":
        kw["check_step"] = float(np.float32(0.0015))
    elif what == "narrow blobs":
        sigma = env.blob_sigma.copy()
        sigma[::2] = np.float32(0.003)
        kw["blob_sigma"] = sigma
    elif what == "far blobs":
        for k in ("pos", "box_lo", "box_hi", "blob_mu"):
            kw[k] = getattr(env, k) * np.float32(40.0)
        kw.update(goal=kw["pos"][-1].copy(), radius=env.radius * 40.0,
                  check_step=env.check_step * 40.0)
    elif what == "no blobs":
        kw.update(blob_mu=env.blob_mu[:0], blob_sigma=env.blob_sigma[:0], blob_amp=env.blob_amp[:0])
    elif what == "few blobs":
        kw.update(blob_mu=env.blob_mu[:5], blob_sigma=env.blob_sigma[:5], blob_amp=env.blob_amp[:5])
    env = dataclasses.replace(env, **kw)
    ref = ograph.build_graph(env)
    dg = mpap.mpap_build_graph(env)
    got = dg.export()
    dg.close()
    assert np.array_equal(got["col"], ref["col"])
    ulps = np.abs(bits(got["drift"]).astype(np.int64) - bits(ref["drift"]).astype(np.int64))
    print(what, ref["col"].size, "edges,", int((ulps > 0).sum()), "differ", flush=True)
    assert ulps.max() <= 1
    assert (ulps > 0).sum() <= 1e-4 * ulps.size


def near_env(pos, radius, boxes=False, blobs=True):
    """An environment with the given float32 positions: its last node is the
    goal (a build needs one); no boxes unless asked, so its edges are the Near
    pairs themselves."""
    pos = np.ascontiguousarray(pos, np.float32)
    dim = pos.shape[1]
    env = synth.plain2d(0, n=200) if dim == 2 else synth.plain3d(0, n=200)
    kw = dict(pos=pos, radius=float(np.float32(radius)), goal=pos[-1].copy(),
              goal_radius=float(np.float32(1e-3)))
    if not boxes:
        kw.update(box_lo=np.zeros((0, dim), np.float32), box_hi=np.zeros((0, dim), np.float32))
    if not blobs:
        kw.update(blob_mu=np.zeros((0, dim), np.float32), blob_sigma=np.zeros(0, np.float32),
                  blob_amp=np.zeros(0, np.float32))
    return dataclasses.replace(env, **kw)


def assert_same_roadmap(env, near_grid):
    ref = ograph.build_graph(env)
    dg = mpap.mpap_build_graph(env, near_grid=near_grid)
    got = dg.export()
    dg.close()
    assert np.array_equal(got["row_ptr"], ref["row_ptr"]), near_grid
    assert np.array_equal(got["col"], ref["col"]), near_grid
    assert np.array_equal(bits(got["cost"]), bits(ref["cost"])), near_grid
    assert np.array_equal(bits(got["drift"]), bits(ref["drift"])), near_grid
    assert np.array_equal(got["goal"], ref["goal"]), near_grid
    return ref


@pytest.mark.parametrize("near_grid", [1, -1])
@pytest.mark.parametrize("dim,n,seed", [(2, 2000, 0), (3, 3000, 1)])
def test_near_by_grid_and_by_all_pairs_match_oracle(dim, n, seed, near_grid):
    env = synth.plain2d(seed, n=n) if dim == 2 else synth.plain3d(seed, n=n)
    assert_same_roadmap(env, near_grid)


@pytest.mark.parametrize("near_grid", [0, 1])
def test_near_grid_on_clustered_samples(near_grid):
    """Dense clusters among sparse samples: cells of very different fill,
    rows of the cluster beyond the in-place sort's 256 entries (then the
    fill compares all pairs), and a second, milder cluster."""
    rng = np.random.default_rng(7)
    a = rng.uniform(0.0, 1.0, (1500, 3))
    b = 0.5 + 0.03 * rng.standard_normal((900, 3))
    c = 0.2 + 0.08 * rng.uniform(0.0, 1.0, (400, 3))
    pos = np.concatenate([a, b, c])
    ref = assert_same_roadmap(near_env(pos, 0.07), near_grid)
    assert np.diff(ref["row_ptr"]).max() > 256


def test_near_grid_rows_at_the_sort_limit():
    """Every row below 256 candidates: the grid fill sorts all of them."""
    rng = np.random.default_rng(11)
    a = rng.uniform(0.0, 1.0, (3000, 3))
    b = 0.5 + 0.04 * rng.standard_normal((300, 3))
    ref = assert_same_roadmap(near_env(np.concatenate([a, b]), 0.06), 1)
    deg = np.diff(ref["row_ptr"])
    assert 100 < deg.max() <= 256


def test_near_grid_with_one_cell():
    """A radius wider than the sample box: one cell, every pair a neighbour,
    rows beyond the sort limit."""
    rng = np.random.default_rng(3)
    pos = rng.uniform(0.0, 1.0, (300, 2))
    ref = assert_same_roadmap(near_env(pos, 2.0, blobs=False), 1)
    assert ref["row_ptr"][-1] == 300 * 299


@pytest.mark.parametrize("dim", [2, 3])
def test_near_grid_on_chains_just_under_the_radius(dim):
    """Samples along a diagonal, consecutive ones about r apart (some just
    below, some just above in float32), far from the origin: pairs straddle
    cell boundaries wherever the cells fall."""
    r = np.float32(0.05)
    k = np.arange(2000, dtype=np.float64)
    step = float(r) * (1.0 - 3e-7 * ((k % 7) - 3)) / np.sqrt(dim)
    t = np.cumsum(step)
    pos = 100.0 + np.repeat(t[:, None], dim, axis=1)
    pos[:, 0] += 1e-4 * (k % 3)
    ref = assert_same_roadmap(near_env(pos, r, blobs=False), 1)
    assert 0 < ref["row_ptr"][-1] < 4 * 2000


@pytest.mark.parametrize("dim,offset,length,n,r", [(2, 1e3, 1.0, 4000, 0.02),
                                                   (3, 1e4, 1.0, 3000, 0.06),
                                                   (2, 1e4, 1000.0, 4000, 0.5)])
def test_near_grid_far_from_the_origin(dim, offset, length, n, r):
    """Samples offset far from the origin, where float32 coordinates are
    coarse (spacing 6e-5 at 1e3, 1e-3 at 1e4), in a square or cube of side
    1, or along a strip 1000 long and 0.3 wide (about 2,000 cells on its
    axis): the grid keeps every pair of the all-pairs set."""
    rng = np.random.default_rng(int(offset) + dim + n)
    u = rng.uniform(0.0, 1.0, (n, dim))
    if length > 1.0:
        u[:, 0] *= length
        u[:, 1:] *= 0.3
    ref = assert_same_roadmap(near_env(offset + u, r, blobs=False), 1)
    assert ref["row_ptr"][-1] > 0


def test_near_grid_on_collinear_samples():
    """Every sample on one line: one cell across, many along."""
    rng = np.random.default_rng(5)
    x = rng.uniform(0.0, 1.0, 2000)
    pos = np.stack([x, np.full_like(x, 0.5)], axis=1)
    assert_same_roadmap(near_env(pos, 0.004), 1)


@pytest.mark.parametrize("n", [1, 2])
def test_near_grid_on_one_or_two_nodes(n):
    pos = np.array([[0.1, 0.2, 0.3], [0.11, 0.2, 0.3]])[:n]
    assert_same_roadmap(near_env(pos, 0.05), 1)


def test_build_graph_rejects_a_bad_near_grid_mode():
    env = synth.plain2d(0, n=300)
    with pytest.raises(mpap.MpapError) as ei:
        mpap.mpap_build_graph(env, near_grid=2)
    assert ei.value.status == mpap.MPAP_ERR_INVAL


def test_build_graph_without_goal_sample_fails():
    env = synth.plain2d(0, n=300)
    env.goal = np.array([5.0, 5.0], np.float32)
    with pytest.raises(mpap.MpapError) as ei:
        mpap.mpap_build_graph(env)
    assert ei.value.status == mpap.MPAP_ERR_NOGOAL


def test_search_on_device_built_graph_matches_oracle():
    """The library's roadmap is the oracle's (same bits); the search on it
    gives the oracle's fronts."""
    env = synth.plain2d(4)
    dg = mpap.mpap_build_graph(env)
    g = ograph.build_graph(env)
    got = dg.export()
    for k in ("row_ptr", "col", "cost", "drift", "reset", "goal"):
        assert np.array_equal(np.asarray(got[k]).view(np.uint8), np.asarray(g[k]).view(np.uint8)), k
    ref = osearch.search(g, env.beta, 2)
    res = mpap.mpap_search(dg, env.beta, 2, env.radius, env.lam)
    check_against_oracle(g, res, ref, env.beta, 2, all_nodes=False, node_stride=5)
    res.close()
    dg.close()
    _ = checks


@pytest.mark.parametrize("stage_cap", [64, 256])
def test_fronts_beyond_the_lds_stage_spill_exactly(road2d, stage_cap):
    """Fronts larger than the LDS staging capacity are merged in device
    memory; forcing a tiny capacity must not change any front."""
    env, g = road2d[0]
    ref = osearch.search(g, env.beta, 2)
    dg = upload(g)
    res = mpap.mpap_search(dg, env.beta, 2, env.radius, env.lam, stage_cap=stage_cap)
    assert res.stats()["max_front"] > stage_cap
    check_against_oracle(g, res, ref, env.beta, 2, all_nodes=False, node_stride=2)
    res.close()
    dg.close()


# ------------------------------------------------------------ high in-degree
def hub_graph(seed, n_b=10, n_a=40, n_spoke=1500, fan=6, p_reset=0.1):
    """root -> B layer -> A layer (all pairs) -> spokes (fan random A parents
    each) -> one hub -> goal.  The hub's in-degree (n_spoke) spans several
    in-edge tiles; with a huge group factor every spoke label reaches the hub
    in one iteration (thousands of children: many candidate rounds and
    chunks in one merge)."""
    rng = np.random.default_rng(seed)
    B = list(range(1, 1 + n_b))
    A = list(range(1 + n_b, 1 + n_b + n_a))
    S = list(range(1 + n_b + n_a, 1 + n_b + n_a + n_spoke))
    hub = S[-1] + 1
    goal = hub + 1
    n = goal + 1
    edges = []

    def edge(u, v):
        edges.append((u, v, float(rng.uniform(0.01, 1.0)), float(rng.uniform(0.0, 0.2))))

    for b in B:
        edge(0, b)
    for b in B:
        for a in A:
            edge(b, a)
    for s in S:
        for a in rng.choice(A, fan, replace=False):
            edge(int(a), s)
    for s in S:
        edge(s, hub)
    edge(hub, goal)
    reset = rng.random(n) < p_reset
    reset[0] = False
    goal_mask = np.zeros(n, dtype=np.uint8)
    goal_mask[goal] = 1
    return from_edges(n, edges, reset, goal_mask), hub


@pytest.mark.parametrize("n_obj,threads,lam,halves", [
    (3, 256, 1e6, 0), (3, 1024, 1e6, 0), (2, 256, 1e6, 0), (3, 1024, 0.5, 0),
    (3, 1024, 1e6, 1 << 20), (2, 1024, 1e6, 1 << 20)])
def test_hub_with_many_in_edge_tiles(n_obj, threads, lam, halves):
    """halves > 0 forces merges by halves with no children limit: the 1,500
    spokes are merged two at a time per workgroup and the hub (thousands of
    children in several in-edge tiles) by one half."""
    g, hub = hub_graph(7)
    assert g["col"].tolist().count(hub) > 1024
    beta = 0.5
    ref = osearch.search(g, beta, n_obj)
    dg, res = run(g, beta, n_obj, radius=0.5, lam=lam, block_threads=threads,
                  merge_halves=halves)
    st = check_against_oracle(g, res, ref, beta, n_obj)
    print(f"hub n_obj {n_obj} threads {threads}: X {st['front_labels']}, hub front "
          f"{res.node_front(hub).shape[0]}, candidates {st['candidates']}, half merges "
          f"{st['half_merges']}", flush=True)
    if halves:
        assert st["half_merges"] > 0
    res.close()
    dg.close()


@pytest.mark.parametrize("n_obj", [2, 3])
def test_single_wave_and_workgroup_merges_in_one_iteration(n_obj):
    """Spokes with a few children each go to single waves, the hub (thousands)
    and, with a slice of 64 labels, the layers before it to workgroups, in the
    same iterations."""
    g, hub = hub_graph(11)
    ref = osearch.search(g, 0.5, n_obj)
    for stage in (0, 64):
        dg, res = run(g, 0.5, n_obj, radius=0.5, lam=2.0, wave_min_targets=1, stage_cap=stage)
        assert res.stats()["wave_build"] == 1
        check_against_oracle(g, res, ref, 0.5, n_obj)
        res.close()
        dg.close()


@pytest.mark.parametrize("threads,stage_cap,n_obj,goals", [
    (1024, 0, 3, 1499), (256, 0, 2, 1499), (256, 64, 3, 600), (1024, 0, 2, 1024), (512, 0, 3, 1)])
def test_goal_front_over_many_goal_nodes(threads, stage_cap, n_obj, goals):
    """Goal nodes by the hundred (more than a workgroup's threads, exactly as
    many, one), on integer costs, so that equal vectors stand at several: the
    oracle's front, each vector at the smallest goal node that has it."""
    g = synth.tiny_random_graph(21, n=1500, p_reset=0.1, mean_degree=3.0, integer_costs=True)
    mask = np.zeros(1500, dtype=np.uint8)
    mask[1500 - goals:] = 1
    g = dict(g, goal=mask)
    ref = osearch.search(g, 1.0, n_obj)
    dg, res = run(g, 1.0, n_obj, radius=1.0, lam=2.0, block_threads=threads, stage_cap=stage_cap)
    check_against_oracle(g, res, ref, 1.0, n_obj, all_nodes=False, node_stride=5)
    first = {}
    for v in np.flatnonzero(mask):
        for row in bits(res.node_front(int(v))):
            first.setdefault(tuple(row), int(v))
    fr = res.goal_front()
    assert fr.goal_node.tolist() == [first[tuple(row)] for row in bits(fr.vecs)]
    res.close()
    dg.close()


@pytest.mark.parametrize("n,n_obj,share", [(150, 2, 5), (150, 3, 5), (1022, 3, 5), (1023, 3, 8),
                                            (1300, 2, 5)])
def test_workgroups_by_size(n, n_obj, share):
    """Five eighths of the workgroups for two objectives and for small
    roadmaps of three, all of them else (the root is one more node): iterations
    with fewer and with more targets than workgroups, by single waves with two
    objectives."""
    env = synth.plain3d(4, n=n)
    g = ograph.build_graph(env)
    ref = osearch.search(g, env.beta, n_obj)
    for lam in (env.lam, 3.0):
        dg, res = run(g, env.beta, n_obj, radius=env.radius, lam=lam)
        st = res.stats()
        assert (st["blocks"], st["wave_build"]) == (256 * share // 8, 1 if n_obj == 2 else 0)
        check_against_oracle(g, res, ref, env.beta, n_obj)
        res.close()
        dg.close()


@pytest.mark.parametrize("dim,n,share", [(2, 2558, 5), (2, 2559, 8), (3, 16382, 5), (3, 16383, 8),
                                            (6, 16383, 5)])
def test_workgroups_of_built_roadmaps(dim, n, share):
    """Two objectives: the number of nodes from which all workgroups run, by
    the roadmap's dimension (the root is one more node); the same fronts as
    with merges by halves on all of them."""
    env = (synth.plain2d if dim == 2 else synth.plain3d if dim == 3 else synth.plain6d)(4, n=n)
    env = dataclasses.replace(env, goal=env.pos[-1][:min(dim, 3)].copy(), goal_radius=0.1)
    dg = mpap.mpap_build_graph(env)
    res = mpap.mpap_search(dg, env.beta, 2, env.radius, env.lam)
    ref = mpap.mpap_search(dg, env.beta, 2, env.radius, env.lam, merge_halves=8192)
    assert (res.stats()["blocks"], ref.stats()["blocks"]) == (256 * share // 8, 256)
    assert (res.stats()["wave_build"], ref.stats()["wave_build"]) == (1, 0)
    assert res.goal_front().vecs.shape[0] > 0
    assert np.array_equal(bits(res.goal_front().vecs), bits(ref.goal_front().vecs))
    for v in range(0, n + 1, 11):
        assert np.array_equal(bits(res.node_front(v)), bits(ref.node_front(v))), v
    for x in (res, ref, dg):
        x.close()


@pytest.mark.parametrize("n_obj,wave", [(2, 1), (3, 0)])
def test_default_build_by_objectives(n_obj, wave):
    """Two-objective searches merge by single waves where an iteration has
    enough targets; three-objective ones of this size don't."""
    env = synth.plain3d(8, n=4500)
    g = ograph.build_graph(env)
    ref = osearch.search(g, env.beta, n_obj)
    dg, res = run(g, env.beta, n_obj, radius=env.radius, lam=2.0)
    assert res.stats()["wave_build"] == wave
    check_against_oracle(g, res, ref, env.beta, n_obj, all_nodes=False, node_stride=3)
    res.close()
    dg.close()


@pytest.mark.parametrize("threads,wmin", [(256, -1), (512, -1), (1024, -1), (1024, 1)])
def test_node_with_many_out_edges(threads, wmin):
    """A row of 12,000 out-edges: the new targets of one wave outgrow its part
    of the LDS (about 2,400) and go out in several pieces; the next layer's
    edges share 400 targets, each queued once.  Merges by workgroups of every
    size and by single waves."""
    rng = np.random.default_rng(5)
    wide = 12000
    edges = [(0, 1, 0.5, 0.1)]
    edges += [(1, 2 + i, float(c), float(d)) for i, (c, d) in
              enumerate(zip(rng.uniform(0.5, 1.0, wide), rng.uniform(0.0, 0.3, wide)))]
    sink = 2 + wide
    edges += [(2 + i, sink + (i % 400), float(c), 0.05) for i, c in
              enumerate(rng.uniform(0.5, 1.0, wide))]
    goal = sink + 400
    edges += [(sink + i, goal, 0.25, 0.01) for i in range(400)]
    mask = np.zeros(goal + 1, dtype=np.uint8)
    mask[goal] = 1
    g = from_edges(goal + 1, edges, np.zeros(goal + 1, dtype=np.uint8), mask)
    ref = osearch.search(g, 0.6, 2)
    dg, res = run(g, 0.6, 2, radius=1.0, lam=4.0, block_threads=threads, wave_min_targets=wmin)
    check_against_oracle(g, res, ref, 0.6, 2, all_nodes=False, node_stride=7)
    res.close()
    dg.close()


@pytest.mark.parametrize("seed", [0, 1, 2])
def test_merges_by_halves_match_the_oracle(road2d, seed):
    """The build with merges by halves forced on the 2,000-sample roadmaps
    (which default to whole workgroups): every front against the oracle.  A
    group factor of 4 (the fronts do not depend on it) gives iterations with
    the 512 targets that merging by halves needs."""
    env, g = road2d[seed]
    ref = osearch.search(g, env.beta, 2)
    dg = upload(g)
    res = mpap.mpap_search(dg, env.beta, 2, env.radius, 4.0, merge_halves=8192)
    st = res.stats()
    assert st["half_front_cap"] > 0 and st["half_merges"] > 0, st
    check_against_oracle(g, res, ref, env.beta, 2)
    r0 = mpap.mpap_search(dg, env.beta, 2, env.radius, env.lam)
    assert r0.stats()["half_merges"] == 0 and r0.stats()["half_front_cap"] == 0
    r0.close()
    res.close()
    dg.close()


# ------------------------------------------------------------ closed forms
# The device search checked directly against closed forms (no oracle search):
# Dijkstra on float32 sums is exact for the additive objectives.
@pytest.fixture(scope="module")
def road2d_small():
    env = synth.plain2d(4, n=2000)
    return env, ograph.build_graph(env)


@pytest.mark.parametrize("n_obj", [2, 3])
def test_relocalising_everywhere_leaves_one_label_per_node(road2d_small, n_obj):
    """Zero drift and a reset at every node: each front is the single vector
    (shortest-path cost, 0[, 0])."""
    _, g = road2d_small
    g1 = dict(g)
    g1["drift"] = np.zeros_like(g["drift"])
    g1["reset"] = np.ones_like(g["reset"])
    dist = checks.dijkstra(g1, g1["cost"])
    dg, res = run(g1, 0.3, n_obj, radius=0.05)
    for v in range(0, g1["goal"].shape[0], 3):
        f = res.node_front(v)
        if not np.isfinite(dist[v]):
            assert f.shape[0] == 0
            continue
        assert f.shape[0] == 1, v
        assert bits(f[0]).tolist() == bits([dist[v], 0.0, 0.0]).tolist(), v
    res.close()
    dg.close()


def test_drift_equal_to_cost_gives_diagonal_fronts(road2d_small):
    """Drift = cost on every edge, no reset: each front is (dist, dist)."""
    _, g = road2d_small
    g1 = dict(g)
    g1["drift"] = g["cost"].copy()
    g1["reset"] = np.zeros_like(g["reset"])
    dist = checks.dijkstra(g1, g1["cost"])
    dg, res = run(g1, np.inf, 2, radius=0.05)
    for v in range(0, g1["goal"].shape[0], 3):
        f = res.node_front(v)
        if np.isfinite(dist[v]):
            assert f.shape[0] == 1, v
            assert bits(f[0, :2]).tolist() == bits([dist[v], dist[v]]).tolist(), v
    res.close()
    dg.close()


def test_front_ends_are_shortest_paths(road2d_small):
    """With no bound and no resets, each front's least cost is the Dijkstra
    distance on cost and its least drift the Dijkstra distance on drift."""
    _, g = road2d_small
    g0 = dict(g)
    g0["reset"] = np.zeros_like(g["reset"])
    dc = checks.dijkstra(g0, g0["cost"])
    dd = checks.dijkstra(g0, g0["drift"])
    dg, res = run(g0, np.inf, 2, radius=0.05)
    for v in range(0, g0["goal"].shape[0], 3):
        f = res.node_front(v)
        if np.isfinite(dc[v]):
            assert f.shape[0] >= 1
            assert bits([f[:, 0].min()]).tolist() == bits([dc[v]]).tolist(), v
            assert bits([f[:, 1].min()]).tolist() == bits([dd[v]]).tolist(), v
    res.close()
    dg.close()
