"""Sets of small replicas, whose steps run in one workgroup per replica: trajectories against the
oracle, energies and virial of every step, and the same bits whatever stands between the
calls (splits, analyses that take the replicas into the brick layout, force evaluations,
list builds), at the edges of the kernel: one particle, below and above the size at which it
uses cells, partly filled waves, the largest size."""
import numpy as np
import pytest

import oracle
from paper_2609_07842_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [(1, 1e-3), (2, 1e-3), (60, 0.05), (127, 0.3), (128, 0.3), (700, 0.2), (1000, 0.1), (1024, 0.05)]
INTEG = dict(integrator="langevin", dt=0.005, kT=1.0, gamma=0.1, seed=5)


def _set(vbc, sizes, precision, f=2.0):
    """A set of at least eight replicas cycling through `sizes`, with its states."""
    idx = [k % len(sizes) for k in range(max(8, len(sizes)))]
    L = [W.box_length(*sizes[k]) for k in idx]
    p = W.vbc_params(E_a=5.0, f=f)
    x = [W.uniform_positions(sizes[k][0], l, 30 + j) for j, (k, l) in enumerate(zip(idx, L))]
    v = [W.maxwell_boltzmann(sizes[k][0], 1.0, 60 + j, False) for j, k in enumerate(idx)]
    s = vbc.System([vbc.replica(len(a), l, p, seed=j) for j, (a, l) in enumerate(zip(x, L))], precision=precision,
                   brick=2, rho_max=1.5)
    s.set_state(np.concatenate(x), np.concatenate(v))
    return s, x, v, L, p


@pytest.mark.parametrize("kind", ["nve", "langevin"])
@pytest.mark.parametrize("precision,tol_x,tol_v", [("fp64", 1e-9, 1e-9), ("fp32", 2e-5, 2e-4)])
def test_set_follows_the_oracle(precision, tol_x, tol_v, kind):
    # bounds of the single-system trajectory tests
    from paper_2609_07842_amd import vbc
    s, x, v, L, p = _set(vbc, SIZES, precision)
    print(f"[resident] {kind} {precision}", flush=True)
    s.thermo(True)
    s.profile(True, 8)
    s.step(50, **dict(INTEG, integrator=kind))
    assert s.profile_read()["force"][1] == 0  # no brick pass was launched
    s.profile(False)
    th = s.thermo_read()
    s.check()
    xg, vg = (t.cpu().numpy() for t in s.get_state())
    off = 0
    for j, (a, b, l) in enumerate(zip(x, v, L)):
        ref = oracle.run(a, b, l, p, 50, kind=oracle.NVE if kind == "nve" else oracle.LANGEVIN, dt=0.005, kT=1.0,
                         gamma=0.1, seed=5 + j)
        d = xg[off:off + len(a)] - ref["x"]
        d -= l * np.rint(d / l)
        assert np.abs(d).max() <= tol_x * max(1.0, l if precision == "fp64" else 1.0), j
        assert np.abs(vg[off:off + len(a)] - ref["v"]).max() <= tol_v * max(1.0, np.abs(ref["v"]).max()), j
        ev = oracle.evaluate(xg[off:off + len(a)], l, p)
        scale = np.abs(ev["e"]).sum() + np.abs(ev["Wt"]).max() + 1e-12
        assert th[j]["steps"] == 50
        got = np.concatenate([[ev["U"], ev["W"]], ev["Wt"]])
        assert np.abs(th[j]["last"] - got).max() <= (1e-10 if precision == "fp64" else 1e-5) * scale
        off += len(a)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_bits_do_not_depend_on_what_stands_between(precision):
    from paper_2609_07842_amd import vbc
    out = {}
    for mode in ("plain", "single", "observe", "force", "track", "stamps", "thermo"):
        s, *_ = _set(vbc, SIZES, precision, f=3.0)
        tr = s.bond_tracker() if mode == "track" else None
        if mode == "stamps":
            s.stamps(True)
        s.thermo(mode == "thermo")
        for k in range(9):
            for n in ([1] * 7 if mode == "single" else [7]):
                s.step(n, **INTEG)
            if mode == "observe":
                s.observables()
                s.clusters(hist_len=16)
            if mode == "force" and k % 2:
                s.force()
            if tr is not None:
                tr.sample()
        if mode == "stamps":
            assert len(s.stamps_read()) == 63
        s.check()
        out[mode] = [t.cpu().numpy().copy() for t in s.get_state()] + [s.stats()[6]["builds"]]
    for mode, (x, v, builds) in out.items():
        assert np.array_equal(x, out["plain"][0]) and np.array_equal(v, out["plain"][1]), mode
    assert 4 <= out["plain"][2] <= 40  # lists were built again on the way


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_list_build_is_a_checkpoint_and_rows_overflow_is_reported(precision):
    from paper_2609_07842_amd import vbc
    s, x, v, L, p = _set(vbc, SIZES, precision)
    s.step(20, **INTEG)
    xc, vc = (t.cpu().numpy().copy() for t in s.get_state())
    s.build_nlist()
    s.step(20, **INTEG)
    a = [t.cpu().numpy() for t in s.get_state()]
    t, *_ = _set(vbc, SIZES, precision)
    t.set_state(xc, vc, step0=20)
    t.step(20, **INTEG)
    b = [q.cpu().numpy() for q in t.get_state()]
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    # lists of at most eight entries
    u = vbc.System([vbc.replica(1000, W.box_length(1000, 0.3), p, seed=j) for j in range(8)], precision=precision,
                   k_max=8)
    u.set_state(np.concatenate([W.uniform_positions(1000, W.box_length(1000, 0.3), j) for j in range(8)]))
    u.step(1, **INTEG)
    st, flags = u.check(raise_on_error=False)
    assert st == vbc.VBC_ERR_NLIST_OVERFLOW and all(f & vbc.FLAG_NLIST_OVERFLOW for f in flags)


def test_lost_and_nonfinite_are_reported():
    from paper_2609_07842_amd import vbc
    N, L = 900, W.box_length(900, 0.1)
    p = W.vbc_params(E_r=0.0, E_a=0.0)
    x = [W.uniform_positions(N, L, j) for j in range(8)]
    v = np.zeros((8 * N, 3))
    v[3 * N + 5] = [1200.0, 0.0, 0.0]  # six length units in a step of 0.005: more than a cell
    x[6][17, 1] = np.nan
    s = vbc.System([vbc.replica(N, L, p) for _ in range(8)], precision="fp64")
    s.set_state(np.concatenate(x), v)
    s.step(2, integrator="nve", dt=0.005)
    st, flags = s.check(raise_on_error=False)
    assert st == vbc.VBC_ERR_NONFINITE
    assert flags[3] & vbc.FLAG_LOST and flags[6] & vbc.FLAG_NONFINITE
    assert not any(flags[j] for j in (0, 1, 2, 4, 5, 7))
