"""Passes in two launches (bricks of usual density, then dense ones) in sets and pools: three
dilute systems of many small bricks laid out for a high local density, two of them with a dense
ball, through several list builds: against the oracle, against fewer passes in two launches, and
the same in a pool."""
import ctypes as C
import math

import numpy as np
import pytest

import oracle
from paper_2609_07842_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

L, N, NC = 53.0, 3000, 22
P = W.vbc_params(E_a=0.3, f=2.0, E_r=0.05)
INTEG = dict(integrator="langevin", dt=0.01, kT=0.3, gamma=0.1, seed=5)
BALLS = (170, 0, 200)
OPTS = dict(brick=1, rho_max=3.6)


def _state(seed, ball):
    rng = np.random.default_rng(seed)
    d = rng.normal(size=(ball, 3))
    d *= 1.2 * rng.random((ball, 1)) ** (1 / 3) / np.linalg.norm(d, axis=1, keepdims=True)
    x = np.concatenate([rng.uniform(0, L, 3) + d, rng.uniform(0, L, size=(N - ball, 3))])
    x = np.mod(x[rng.permutation(N)], L)
    return np.where(x >= L, 0.0, x), W.maxwell_boltzmann(N, 0.3, 60 + seed)


def _staged(x):
    """Particles in the 27 cells that each brick (one cell) stages."""
    c = np.minimum((x * (NC / L)).astype(int), NC - 1)
    h = np.zeros((NC, NC, NC), dtype=int)
    np.add.at(h, tuple(c.T), 1)
    return sum(np.roll(h, s, axis=(0, 1, 2)) for s in np.ndindex(3, 3, 3))


def _usual():
    """Staged particles up to which a brick is of usual density (those of a layout without a
    stated maximum)."""
    return -(-math.ceil(N / NC ** 3 * 27 * 1.3 + 96) // 32) * 32


def _nodes(vbc, call):
    """Kernel launches of a captured call."""
    hip, graph, nodes = vbc.lib(), C.c_void_p(), C.c_size_t(0)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        h = C.c_void_p(stream.cuda_stream)
        torch.cuda.synchronize()
        assert hip.hipStreamBeginCapture(h, 1) == 0  # this thread's calls only
        call()
        assert hip.hipStreamEndCapture(h, C.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, C.byref(nodes)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return nodes.value


def _handle(vbc, kind, block, precision, states):
    reps = [vbc.replica(N, L, P, seed=k) for k in range(3)]
    if kind == "set":
        h = vbc.System(reps, precision=precision, block=block, **OPTS)
        h.set_state(np.concatenate([s[0] for s in states]), np.concatenate([s[1] for s in states]))
        return h
    fps = [vbc.footprint(r, precision, **OPTS) for r in reps]
    caps = dict(max_replicas=3, max_types=1, max_particles=3 * N, max_slots=sum(f["slots"] for f in fps),
                max_bricks=sum(f["bricks"] for f in fps), max_cells=sum(f["cells"] for f in fps),
                max_bcap=max(f["bcap"] for f in fps), chains=False)
    h = vbc.Pool(caps, precision=precision, block=block, k_max=fps[0]["k_max"], stage_cap=fps[0]["stage_cap"], **OPTS)
    for r, s in zip(reps, states):
        h.admit(r, *s)
    return h


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_dense_bricks_in_sets_and_pools(precision):
    from paper_2609_07842_amd import vbc
    states = [_state(k, b) for k, b in enumerate(BALLS)]
    usual = _usual()
    assert [int((_staged(x) > usual).any()) for x, _ in states] == [1, 0, 1]
    got, nodes = {}, {}
    for kind, block in (("set", 1024), ("set", 64), ("pool", 64)):
        print(f"[dense sets] {precision} {kind} {block}", flush=True)
        s = _handle(vbc, kind, block, precision, states)
        s.build_nlist()
        ints, reals = [], []
        tr = s.bond_tracker(max_partners=64, hist_len=64, bin_steps=1)
        for _ in range(3):
            reals += [s.count(), s.force()[0], s.force()[1]]
            z, pen, sums = s.observables()
            ints += [z, pen, sums, *s.clusters(hist_len=256)]
            s.step(25, **INTEG)
            tr.sample()
            reals += list(s.get_state())
        ints += [tr.hist, tr.stats]
        for r in range(3):
            x = s.get_state()[0][r * N:(r + 1) * N].cpu().numpy()
            # the list holds every pair within the cutoff, dense or not
            pairs, _ = s.nlist_pairs(r)
            have = {(min(a, b), max(a, b)) for a, b in pairs.tolist()}
            assert {tuple(q) for q in oracle.neighbor_pairs(x, L, 2.0).tolist()} <= have
        s.check()
        assert all(q["builds"] >= 3 for q in s.stats()[:3])
        # at the end too, some bricks are dense and the most are not
        dense = [int((_staged(s.get_state()[0][r * N:(r + 1) * N].cpu().numpy()) > usual).sum()) for r in range(3)]
        assert dense[0] > 0 and dense[2] > 0 and dense[1] == 0
        nodes[kind, block] = _nodes(vbc, lambda: lib_count(vbc, s))
        got[kind, block] = [[t.cpu().numpy().copy() for t in q] for q in (ints, reals)]
        if (kind, block) == ("set", 64):
            off = 0
            for k, (x, v) in enumerate(states):
                ref = oracle.evaluate(x, L, P)
                n, F = got[kind, block][1][0][off:off + N], got[kind, block][1][1][off:off + N]
                tol = 1e-10 if precision == "fp64" else 1e-5
                assert np.abs(n - ref["n"]).max() <= tol * ref["n"].max()
                err = np.linalg.norm(F - ref["F"], axis=1).max() / np.linalg.norm(ref["F"], axis=1).max()
                assert err <= tol, k
                off += N
        s.close()
    # work list, re-sort, list build in two, and the count in one launch or two
    assert nodes == {("set", 1024): 5, ("set", 64): 6, ("pool", 64): 6}
    for other in (("set", 1024), ("pool", 64)):
        for a, b in zip(got["set", 64], got[other]):
            assert all(np.array_equal(p, q) for p, q in zip(a, b)), other


def lib_count(vbc, s):
    assert vbc.lib().vbc_count(s.h, None, s._stream()) == vbc.VBC_OK
