"""States set, read and built for all replicas of a handle at once (one launch over all
bricks) against the same replicas one at a time: bit for bit, with several replicas pending
while others keep their layout, sizes from one particle up, in fixed sets and pools."""
import numpy as np
import pytest

from paper_2609_07842_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [(1, 1e-3), (700, 0.3), (2, 1e-3), (1500, 0.5), (65, 0.05)]
INTEG = dict(integrator="langevin", dt=0.005, kT=1.0, gamma=0.1, seed=5)
OPTS = dict(k_max=96, stage_cap=2112, block=256)


def _inputs(seed):
    return [(W.uniform_positions(n, W.box_length(n, r), seed + k), W.maxwell_boltzmann(n, 1.0, 9 + k, False))
            for k, (n, r) in enumerate(SIZES)]


def _handle(vbc, idx, pool, precision):
    d = [vbc.replica(SIZES[k][0], W.box_length(*SIZES[k]), W.vbc_params(E_a=4.0, f=2.0), seed=k) for k in idx]
    if not pool:
        return vbc.System(d, precision=precision, **OPTS), d
    fps = [vbc.footprint(q, precision, **OPTS) for q in d]
    caps = dict(max_replicas=len(d) + 1, max_types=1, max_particles=sum(SIZES[k][0] for k in idx),
                max_slots=sum(f["slots"] for f in fps), max_bricks=sum(f["bricks"] for f in fps),
                max_cells=sum(f["cells"] for f in fps), max_bcap=max(f["bcap"] for f in fps), chains=False)
    return vbc.Pool(caps, precision=precision, **OPTS), d


def _run(vbc, idx, pool, precision, again):
    """Step, give the replicas in `again` new states, step, evaluate; every replica's results."""
    first, second = _inputs(100), _inputs(200)
    h, d = _handle(vbc, idx, pool, precision)
    if pool:
        for k, q in zip(idx, d):
            h.admit(q, *first[k])
    else:
        h.set_state(np.concatenate([first[k][0] for k in idx]), np.concatenate([first[k][1] for k in idx]))
    x0, _ = h.get_state()
    h.step(9, **INTEG)
    for j, k in enumerate(idx):
        if k in again:
            h.set_state(second[k][0], second[k][1], rep=j)
    h.step(10, **INTEG)
    x, v = h.get_state()
    F, e, UW = h.force()
    h.check()
    out, off = {}, 0
    for j, k in enumerate(idx):
        sl = slice(off, off + SIZES[k][0])
        out[k] = [t[sl].cpu().numpy() for t in (x0, x, v, F, e)] + [UW[j].cpu().numpy()]
        off += SIZES[k][0]
    return out, first


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("pool", [False, True])
def test_batched_states_equal_single(pool, precision):
    from paper_2609_07842_amd import vbc
    again = (1, 2, 4)
    print(f"[batched state] pool {pool} {precision}", flush=True)
    got, first = _run(vbc, range(5), pool, precision, again)
    for k in range(5):
        assert np.array_equal(got[k][0], first[k][0])  # read back before any step
        alone, _ = _run(vbc, [k], pool, precision, again)
        for a, b in zip(got[k], alone[k]):
            assert np.array_equal(a, b), k


def test_captured_analysis_replays_after_steps():
    """An analysis captured into a graph while no list can be due still rebuilds the lists when
    it is replayed after steps (of even count: a captured call keeps its position buffer)."""
    from paper_2609_07842_amd import vbc
    N, L = 5000, W.box_length(5000, 0.3)
    s = vbc.System(vbc.replica(N, L, W.vbc_params(E_a=5.0, f=3.0)), precision="fp32", rho_max=1.0)
    s.set_state(W.uniform_positions(N, L, 3), W.maxwell_boltzmann(N, 1.0, 4))
    s.observables()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        z, pen, sums = s.observables()
    for _ in range(5):
        s.step(30, **INTEG)
        g.replay()
        torch.cuda.synchronize()
        ze, pe, se = s.observables()
        assert torch.equal(z, ze) and torch.equal(pen, pe) and torch.equal(sums, se)
    s.check()

