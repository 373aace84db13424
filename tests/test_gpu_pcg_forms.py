"""The forms of the block-Jacobi PCG (one launch per linear solve by several workgroups or
by one, asked for by flag or chosen by size, alone or in a served batch) against one launch
per PCG iteration, which ba_set_pcg_form selects.  Needs an MI355X."""
import time

import numpy as np
import pytest

from synth import make_arc_scene, make_pose_graph, make_rig_drive, make_small_drive

pytestmark = pytest.mark.gpu

WIDE, RESIDENT, COOP = 8, 16, 64  # BA_FLAG_PCG_*


def _say(*a):
    print(*a, flush=True)


def _same(a, b):
    assert np.array_equal(a["iter_cost"], b["iter_cost"])
    assert list(a["pcg_iters"]) == list(b["pcg_iters"])
    assert np.array_equal(a["q"], b["q"]) and np.array_equal(a["t"], b["t"])
    assert np.array_equal(a["X"], b["X"])
    assert a["status"] == b["status"]


KW = dict(max_iters=3, pcg_max_iters=30, pcg_rel_tol=1e-10)
SCENES = {  # case: scene, flags beside the default's
    "one tile": (lambda: make_arc_scene(5, 300, seed=4), 0),
    "20 cameras": (lambda: make_arc_scene(21, 600, seed=20), 0),
    "40 cameras": (lambda: make_arc_scene(41, 700, seed=40), 0),
    "41 cameras": (lambda: make_arc_scene(42, 700, seed=41), 0),
    "drive": (lambda: make_small_drive(40, 3000, seed=5), 0),
    "wide": (lambda: make_small_drive(40, 3000, seed=5), WIDE),
    "columns": (lambda: make_arc_scene(168, 1200, seed=9), 0),
    "175 tiles": (lambda: make_small_drive(700, 14000, seed=8), 0),
    "16 rows, columns": (lambda: make_small_drive(1100, 22000, seed=9, mean_track=16.0), 0),
}


def _problem(balib, case, prec, extra=0, **kw):
    kw = {**KW, "precision": prec, **kw}
    if case == "graph 16 rows":
        return balib.Problem.from_pose_graph(make_pose_graph(180), flags=extra, **kw)
    if case == "graph pairs":  # 282 tiles of 32 rows
        return balib.Problem.from_pose_graph(make_pose_graph(1500), flags=extra, **kw)
    if case == "rig":
        return balib.Problem.from_rig(make_rig_drive(40, 1500, seed=3), prior_ext=100.0, prior_rig=100.0,
                                      rig_pairs=np.array([[0, 1], [0, 2]]), **kw)
    make, flags = SCENES[case]
    return balib.Problem.from_scene(make(), flags=flags | extra, **kw)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("case", list(SCENES) + ["graph 16 rows", "graph pairs", "rig"])
def test_one_launch_pcg_equals_a_launch_per_iteration(balib, prec, case):
    """4-, 16- and 32-row tiles, one column set and two, one workgroup and two tiles to a
    workgroup, with and without the resident flag (where it applies): the same solve as with
    a launch per PCG iteration, bit for bit, and back again on the same problem."""
    _say("device solves:", case, prec)
    p = _problem(balib, case, prec).set_pcg_form(balib.PCG_PER_LAUNCH)
    ref = p.solve().result()
    assert p.pcg_form() == balib.PCG_PER_LAUNCH
    a = p.set_pcg_form(balib.PCG_AUTO).reset().solve().result()
    assert p.pcg_form() == balib.PCG_AUTO
    b = p.set_pcg_form(balib.PCG_PER_LAUNCH).reset().solve().result()
    p.close()
    assert ref["status"] in (0, 1) and ref["iters"] == 3
    _same(ref, a)
    _same(ref, b)
    if case in ("rig", "graph pairs"):
        return
    for extra in (RESIDENT, RESIDENT | COOP):
        p = _problem(balib, case, prec, extra)
        info = p.info()
        if info["pcg_resident"]:
            _same(ref, p.solve().result())
            assert p.pcg_form() == balib.PCG_AUTO
            _same(ref, p.set_pcg_form(balib.PCG_PER_LAUNCH).reset().solve().result())
            assert p.pcg_form() == balib.PCG_PER_LAUNCH
        else:
            assert case == "16 rows, columns"  # a tile there reads more than 170 columns
        p.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("case", ["41 cameras", "175 tiles", "graph 16 rows", "graph pairs", "rig"])
def test_a_wait_that_runs_out_falls_back_at_any_iteration(balib, prec, case):
    """Waits that give up at the first, second, a later and the last iteration that has one:
    without the flag the solve is the launch-per-iteration one with its ordinary status;
    with the flag it stops with BA_STATUS_PCG_SYNC where an iteration gets that far."""
    p = _problem(balib, case, prec).set_pcg_form(balib.PCG_PER_LAUNCH)
    ref = p.solve().result()
    p.set_pcg_form(balib.PCG_AUTO)
    last = KW["pcg_max_iters"] - 1
    for it in (1, 2, 7, last):
        _say("device solves:", case, prec, "waits give up from iteration", it)
        p.set_barrier_polls(0, it).set_pcg_form(balib.PCG_AUTO)
        _same(ref, p.reset().solve().result())
        assert p.pcg_form() == balib.PCG_AUTO
        assert p.pcg_fell_back() == sum(n >= it for n in ref["pcg_iters"])
    p.close()
    if case in ("rig", "graph pairs"):
        return
    p = _problem(balib, case, prec, RESIDENT)
    for it in (1, 2, 7, last):
        r = p.set_barrier_polls(0, it).reset().solve().result()
        if ref["pcg_iters"][0] >= it:
            assert r["status"] == balib.STATUS_PCG_SYNC and r["iters"] == 1 and r["accepted"] == 0
        else:
            assert max(ref["pcg_iters"]) >= it or r["status"] == ref["status"]
    p.close()


@pytest.mark.parametrize("first", [1, 2])
def test_a_fall_back_is_remembered(balib, first):
    """After a solve that fell back (one workgroup runs the steps, or all share them) the
    next 16 launch their PCG per iteration, then one launch is tried again; asking for the
    default form tries it at once.  A flagged solve and one that did not fall back hold
    nothing back."""
    p = _problem(balib, "41 cameras", "f32").set_barrier_polls(0, first)
    ref = p.solve().result()
    assert p.pcg_form() == balib.PCG_AUTO and p.pcg_fell_back() == 3
    p.set_barrier_polls(1 << 20)
    for _ in range(16):
        _same(ref, p.reset().solve().result())
        assert p.pcg_form() == balib.PCG_PER_LAUNCH and p.pcg_fell_back() == 0
    for _ in range(2):
        _same(ref, p.reset().solve().result())
        assert p.pcg_form() == balib.PCG_AUTO and p.pcg_fell_back() == 0
    p.set_barrier_polls(0, first).reset().solve()
    assert p.pcg_fell_back() == 3
    p.set_barrier_polls(1 << 20).set_pcg_form(balib.PCG_AUTO)
    _same(ref, p.reset().solve().result())
    assert p.pcg_form() == balib.PCG_AUTO and p.pcg_fell_back() == 0
    p.close()


def test_early_stop_and_cap(balib):
    """A loose tolerance (a few iterations) and a cap of 1 and 3 iterations, for one
    workgroup and several: every form stops where the launch-per-iteration one does."""
    for case in ("20 cameras", "41 cameras"):
        for kw in (dict(pcg_rel_tol=1e-2), dict(pcg_rel_tol=1e-12, pcg_max_iters=1),
                   dict(pcg_rel_tol=1e-12, pcg_max_iters=3)):
            p = _problem(balib, case, "f32", **kw).set_pcg_form(balib.PCG_PER_LAUNCH)
            ref = p.solve().result()
            a = p.set_pcg_form(balib.PCG_AUTO).reset().solve().result()
            p.close()
            p = _problem(balib, case, "f32", RESIDENT, **kw)
            b = p.solve().result()
            p.close()
            _say(case, kw, "pcg", ref["pcg_iters"])
            _same(ref, a)
            _same(ref, b)


def test_refine_per_launch(balib):
    """The two-stage refinement with culling on a drive of 59 free cameras: the default
    form's rounds, activity mask, poses and points are those of a launch per iteration."""
    s = make_small_drive(60, 6000, seed=62, outlier_frac=0.1, huber_delta=1.0)
    out = []
    for form in (balib.PCG_PER_LAUNCH, balib.PCG_AUTO):
        p = balib.Problem.from_scene(s, max_iters=8, precision="f32").set_pcg_form(form)
        hist = p.refine([(1.0, 8.0), (0.0, 3.0)], 2)
        assert p.pcg_form() == form
        out.append((hist, p.active().copy(), p.result()))
        p.close()
    (ha, aa, ra), (hb, ab, rb) = out
    assert ha == hb and np.array_equal(aa, ab)
    assert np.array_equal(ra["q"], rb["q"]) and np.array_equal(ra["X"], rb["X"])


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_served_batches_of_both_forms(balib, prec):
    """Requests of 41 to 700 cameras through a server, few enough tiles for one launch and
    (two of 175) too many: each result is the launch-per-iteration solve's, bit for bit."""
    big = [make_small_drive(700, 6000, seed=8 + k) for k in range(2)]
    few = [make_small_drive(70, 1500, seed=2), make_arc_scene(42, 500, seed=3), make_arc_scene(12, 300, seed=6)]
    o = balib.options(precision=prec, **KW)
    for scenes in (few, big + few):
        refs = []
        for s in scenes:
            p = balib.Problem.from_scene(s, precision=prec, **KW).set_pcg_form(balib.PCG_PER_LAUNCH)
            refs.append(p.solve().result())
            p.close()
        srv = balib.Server(1 << 30, 8, prec)
        ts = [srv.submit(balib.scene_desc(s), o) for s in scenes]
        for t, ref in zip(ts, refs):
            _same(ref, srv.wait(t))
        srv.close()


def test_a_flagged_request_counts_its_cus(balib):
    """A lone server request with the resident flag (14 tiles) runs in one launch in any case,
    so its CUs count: a solve of 250 tiles beside it, which they no longer hold, launches per
    iteration, and one after it does not."""
    A = make_small_drive(57, 6000, seed=140)
    s = make_small_drive(1000, 9000, seed=3)
    kw = dict(max_iters=3, pcg_max_iters=20, precision="f32")
    p = balib.Problem.from_scene(s, **kw)
    ref = p.solve().result()
    assert p.pcg_form() == balib.PCG_AUTO and p.info()["pcg_rows"] == 4
    srv = balib.Server(1 << 28, 2, "f32")
    t = srv.submit(balib.scene_desc(A), balib.options(max_iters=4000, precision="f32", flags=RESIDENT))
    time.sleep(0.1)  # the request is running
    t0 = time.perf_counter()
    b = p.reset().solve().result()
    form, ended = p.pcg_form(), time.perf_counter()
    r = srv.wait(t)
    _say("request latency", r["latency_ms"], "ms, solve beside it ended after", 100 + 1e3 * (ended - t0), "ms, form", form)
    assert r["latency_ms"] > 100 + 1e3 * (ended - t0)  # it was still running
    assert form == balib.PCG_PER_LAUNCH
    _same(ref, b)
    srv.close()
    _same(ref, p.reset().solve().result())
    assert p.pcg_form() == balib.PCG_AUTO
    p.close()


def test_a_server_gives_back_the_cus_of_a_batch_that_shrank(balib):
    """A long request (18 tiles) beside one of 175 tiles that ends soon: once that has ended, a
    solve of 230 tiles finds CUs enough, with the long request still running."""
    A, B = make_small_drive(70, 6000, seed=141), make_small_drive(700, 9000, seed=142)
    kw = dict(max_iters=3, pcg_max_iters=20, precision="f32")
    p = balib.Problem.from_scene(make_small_drive(920, 9000, seed=3), **kw)
    ref = p.solve().result()
    assert p.pcg_form() == balib.PCG_AUTO and p.info()["pcg_rows"] == 4
    srv = balib.Server(1 << 28, 4, "f32")
    tb = srv.submit(balib.scene_desc(B), balib.options(**kw))
    ta = srv.submit(balib.scene_desc(A), balib.options(max_iters=6000, precision="f32"))
    t0 = time.perf_counter()
    srv.wait(tb)
    time.sleep(0.05)
    b = p.reset().solve().result()
    form, ended = p.pcg_form(), time.perf_counter()
    ra = srv.wait(ta)
    _say("long request", ra["latency_ms"], "ms, solve beside it ended after", 1e3 * (ended - t0), "ms, form", form)
    assert ra["latency_ms"] > 1e3 * (ended - t0)  # it was still running
    assert form == balib.PCG_AUTO and p.pcg_fell_back() == 0
    _same(ref, b)
    srv.close()
    p.close()


def test_profiled_per_launch_runs(balib):
    """The PCG timed alone (segment graphs) and launch by launch, switching forms on one
    problem: the same solves, and a run counts its steps unless the flag made it one launch."""
    for extra in (0, RESIDENT):
        p = _problem(balib, "41 cameras", "f32", extra)
        ref = p.solve().result()
        k = list(p.kernel_times()).index("pcg_cg")
        for mask in (1 << k, -1):
            for form in (balib.PCG_PER_LAUNCH, balib.PCG_AUTO, balib.PCG_PER_LAUNCH):
                p.set_profiling(mask).set_pcg_form(form)
                _same(ref, p.reset().solve().result())
                assert p.pcg_form() == form
                n = p.kernel_times()["pcg_cg"][1]
                one = extra and form == balib.PCG_AUTO
                assert n == KW["max_iters"] * (1 if one else KW["pcg_max_iters"]), (extra, mask, form, n)
        p.close()
