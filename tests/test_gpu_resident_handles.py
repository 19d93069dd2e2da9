"""Handles whose steps run in one workgroup per replica, used in other ways than step after step:
replicas that retire and enter, analyses and steps captured into graphs of the caller's."""
import numpy as np
import pytest

import oracle
from paper_2609_07842_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

INTEG = dict(integrator="langevin", dt=0.005, kT=1.0, gamma=0.1, seed=5)
L = 24.0
SIZES = [600, 600, 601, 127, 300, 64, 500, 599]
PARAMS = W.vbc_params(E_a=5.0, f=2.0)


def _inputs(n, k):
    return W.uniform_positions(n, L, 30 + k), W.maxwell_boltzmann(n, 1.0, 60 + k, False)


def _set(vbc, sizes, precision):
    """A set of replicas in equal boxes (equal layouts) and its states, in dicts by slot."""
    s = vbc.System([vbc.replica(n, L, PARAMS, seed=k) for k, n in enumerate(sizes)], precision=precision, brick=2,
                   rho_max=1.5)
    x, v = zip(*(_inputs(n, k) for k, n in enumerate(sizes)))
    s.set_state(np.concatenate(x), np.concatenate(v))
    s._keep_admit = {}
    return s


def _state(s, rep, n):
    s.reps[rep]["n"] = n
    return [t.cpu().numpy() for t in s.get_state(rep)]


def _close_to_oracle(got, n, k, seed, steps, precision):
    """Bounds of the single-system trajectory tests."""
    x, v = _inputs(n, k)
    ref = oracle.run(x, v, L, PARAMS, steps, kind=oracle.LANGEVIN, dt=0.005, kT=1.0, gamma=0.1, seed=seed)
    d = got[0] - ref["x"]
    d -= L * np.rint(d / L)
    tol_x, tol_v = (1e-9 * L, 1e-9) if precision == "fp64" else (2e-5, 2e-4)
    assert np.abs(d).max() <= tol_x
    assert np.abs(got[1] - ref["v"]).max() <= tol_v * max(1.0, np.abs(ref["v"]).max())


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_an_admitted_replica_steps_like_the_rest(precision):
    """Three slots change their replica, one of them for a larger one than any before: the new
    ones end with the bits of a set that held them from the start, the old ones with theirs."""
    from paper_2609_07842_amd import vbc
    print(f"[resident admit] {precision}", flush=True)
    s = _set(vbc, SIZES, precision)
    s.step(20, **INTEG)
    new = {}
    for slots, n, k in (((5,), 63, 11), ((0, 1), 1024, 12)):  # the larger one takes two slots' ranges
        for r in slots:
            vbc.Pool.retire(s, r)
        x, v = _inputs(n, k)
        got = vbc.Pool.admit(s, vbc.replica(n, L, PARAMS, seed=100 + k), x, v)
        new[got] = (n, k)
        assert got == slots[0]
    s.profile(True, 8)
    s.step(30, **INTEG)
    assert s.profile_read()["force"][1] == 0  # no brick pass was launched
    s.check()
    fresh = _set(vbc, SIZES, precision)
    for n in (20, 30):
        fresh.step(n, **INTEG)
    whole = vbc.System([vbc.replica(n, L, PARAMS, seed=100 + k) for n, k in [(63, 11), (1024, 12)] * 4],
                       precision=precision, brick=2, rho_max=1.5)
    whole.set_state(*(np.concatenate(a) for a in zip(*[_inputs(n, k) for n, k in [(63, 11), (1024, 12)] * 4])))
    whole.step(30, **INTEG)
    for r, n in enumerate(SIZES):
        if r in new:
            a, b = _state(s, r, new[r][0]), _state(whole, [63, 1024].index(new[r][0]), new[r][0])
            _close_to_oracle(a, new[r][0], new[r][1], 100 + new[r][1] + 5, 30, precision)
        elif r == 1:
            continue
        else:
            a, b = _state(s, r, n), _state(fresh, r, n)
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), r


@pytest.mark.parametrize("between", ["nothing", "clusters", "force"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_a_replica_too_large_takes_the_set_to_the_bricks(precision, between):
    from paper_2609_07842_amd import vbc
    print(f"[resident leaves] {precision} {between}", flush=True)
    s = _set(vbc, SIZES, precision)
    s.step(20, **INTEG)
    if between == "clusters":
        s.clusters(hist_len=16)
    if between == "force":
        s.force()
    vbc.Pool.retire(s, 1)
    vbc.Pool.retire(s, 2)
    x, v = _inputs(1100, 13)
    assert vbc.Pool.admit(s, vbc.replica(1100, L, PARAMS, seed=77), x, v) == 1
    s.profile(True, 64)
    s.step(20, **INTEG)
    assert s.profile_read()["force"][1] > 0
    s.check()
    for r, n in enumerate(SIZES):
        if r == 1:
            _close_to_oracle(_state(s, 1, 1100), 1100, 13, 82, 20, precision)
        elif r != 2:
            _close_to_oracle(_state(s, r, n), n, r, r + 5, 40, precision)


def _analysis(s):
    z, pen, sums = s.observables()
    label, stats, hist = s.clusters(hist_len=16)
    F, e, UW = s.force()
    return z, pen, sums, label, stats, hist, F, e, UW


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_captured_analysis_replays_after_steps(precision):
    """Analyses and forces captured while the replicas stand in their brick layout, replayed after
    steps that took them out of it: the results and the further trajectory of a set that ran the
    same calls without a graph."""
    from paper_2609_07842_amd import vbc
    print(f"[resident captured analysis] {precision}", flush=True)
    s, ref = _set(vbc, SIZES, precision), _set(vbc, SIZES, precision)
    for h in (s, ref):
        h.step(10, **INTEG)
        _analysis(h)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = _analysis(s)
    for k in range(4):
        for h in (s, ref):
            h.step(15, **INTEG)
        g.replay()
        torch.cuda.synchronize()
        want = _analysis(ref)
        assert all(torch.equal(a, b) for a, b in zip(out, want)), k
        if k == 1:  # and an eager one between two replays
            assert all(torch.equal(a, b) for a, b in zip(_analysis(s), want))
        assert all(torch.equal(a, b) for a, b in zip(s.get_state(), ref.get_state())), k
    s.check()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_captured_steps_replay_between_analyses(precision):
    """Steps captured into a graph, replayed with reads, analyses, list builds and eager steps in
    between: the results of a set that ran the same calls without a graph.  Capturing itself
    changes nothing.  Then a replica admitted since is stepped by the same graph."""
    from paper_2609_07842_amd import vbc
    print(f"[resident captured steps] {precision}", flush=True)
    s, ref = _set(vbc, SIZES, precision), _set(vbc, SIZES, precision)
    for h in (s, ref):
        h.step(10, **INTEG)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        s.step(12, **INTEG)
    same = lambda a, b: all(torch.equal(p, q) for p, q in zip(a, b))
    assert same(s.get_state(), ref.get_state())
    assert same(_analysis(s), _analysis(ref))
    for k in range(5):
        g.replay()
        ref.step(12, **INTEG)
        torch.cuda.synchronize()
        if k != 2:
            assert same(_analysis(s), _analysis(ref)), k
        if k == 3:
            s.build_nlist()
            ref.build_nlist()
        if k == 4:
            s.step(3, **INTEG)
            ref.step(3, **INTEG)
        assert same(s.get_state(), ref.get_state()), k
    s.check()
    for h in (s, ref):
        for r in (0, 1):
            vbc.Pool.retire(h, r)
        assert vbc.Pool.admit(h, vbc.replica(1024, L, PARAMS, seed=9), *_inputs(1024, 12)) == 0
    g.replay()
    ref.step(12, **INTEG)
    torch.cuda.synchronize()
    for r, n in [(0, 1024), (3, SIZES[3]), (7, SIZES[7])]:
        a, b = _state(s, r, n), _state(ref, r, n)
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), r
    # a replica too large for the route: the set goes on by bricks, from where the graph left it
    for h in (s, ref):
        vbc.Pool.retire(h, 2)
        vbc.Pool.retire(h, 3)
    g.replay()
    ref.step(12, **INTEG)
    x, v = _inputs(1100, 13)
    for h in (s, ref):
        vbc.Pool.retire(h, 0)
        vbc.Pool.admit(h, vbc.replica(1100, L, PARAMS, seed=77), x, v)
        h.step(16, **INTEG)
        h.check()
    for r, n in [(0, 1100), (4, SIZES[4]), (7, SIZES[7])]:
        a, b = _state(s, r, n), _state(ref, r, n)
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), r


@pytest.mark.parametrize("nsteps,launches", [(1, 1), (1024, 1), (1025, 2), (2500, 3)])
def test_long_calls_are_several_launches(nsteps, launches):
    """A call of many steps is a launch per 1024 (counted as nodes of a captured call), with the
    bits, sums and samples of short calls."""
    import ctypes as C

    from paper_2609_07842_amd import vbc
    sizes, out = [60, 64, 40, 127, 30, 50, 20, 10], []
    for split in ([nsteps], [500] * (nsteps // 500) + [nsteps % 500]):
        s = _set(vbc, sizes, "fp32")
        s.thermo(True)
        for n in split:
            s.step(n, **INTEG)
        th = s.thermo_read()
        s.check()
        out.append([t.cpu().numpy() for t in s.get_state()] + [np.concatenate([q["last"], q["sum"]]) for q in th])
        assert all(q["steps"] == nsteps for q in th)
    assert all(np.array_equal(a, b) for a, b in zip(*out))
    hip, graph, nodes = vbc.lib(), C.c_void_p(), C.c_size_t(0)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        h = C.c_void_p(stream.cuda_stream)
        torch.cuda.synchronize()
        assert hip.hipStreamBeginCapture(h, 1) == 0  # this thread's calls only
        s.step(nsteps, **INTEG)
        assert hip.hipStreamEndCapture(h, C.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, C.byref(nodes)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    assert nodes.value == launches


def test_precision_in_a_large_box():
    """FP32 pair arithmetic of a step in a box of 500 (positions as fractions of the box): no
    further from the oracle than the brick passes, over the particles in a switching window."""
    from paper_2609_07842_amd import vbc
    n, box, rho = 1000, 500.0, 0.3
    p = W.vbc_params(E_a=5.0, f=4.0)
    x = W.uniform_positions(n, W.box_length(n, rho), 3) + 311.0
    v = np.zeros((n, 3))
    win = oracle.evaluate(x, box, p)["n"]
    win = (win > 4.0) & (win < 5.0)
    assert win.sum() > 100
    ref = oracle.run(x, v, box, p, 1, kind=oracle.NVE, dt=0.005)["v"]
    err = {}
    for k, m in ((8, 1), (1, 1)):  # a set that steps in one workgroup per replica; bricks
        small = [vbc.replica(10, 24.0, p) for _ in range(k - 1)]
        s = vbc.System([vbc.replica(n, box, p)] + small, precision="fp32", brick=6, k_max=96, stage_cap=4096,
                       rho_max=0.0 if k == 8 else 0.4)
        xs = np.concatenate([x] + [W.uniform_positions(10, 24.0, j) for j in range(k - 1)])
        s.set_state(xs, np.zeros_like(xs))
        s.profile(True, 8)
        s.step(1, integrator="nve", dt=0.005)
        assert (s.profile_read()["force"][1] == 0) == (k == 8)
        s.check()
        got = s.get_state()[1].cpu().numpy()[:n]
        err[k] = np.sqrt(((got - ref)[win] ** 2).mean() / (ref[win] ** 2).mean())
        print(f"[large box] {k} replicas: rms error {err[k]:.2e}", flush=True)
        s.close()
    assert err[8] <= err[1]
