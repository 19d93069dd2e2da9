"""Results that do not depend on the workgroup size, hence not on what else a pool holds (fuller
replicas raise its automatic workgroup size): bit for bit, at valencies with few and many
particles per brick in a switching window."""
import numpy as np
import pytest

from paper_2609_07842_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

INTEG = dict(integrator="langevin", dt=0.005, kT=1.0, gamma=0.1, seed=5)
OPTS = dict(k_max=96, stage_cap=2720)


def _state(n, rho, k):
    return W.uniform_positions(n, W.box_length(n, rho), 30 + k), W.maxwell_boltzmann(n, 1.0, 60 + k)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("f", [2.0, 3.0, 4.0])
def test_counts_in_a_pool_equal_those_alone(f, precision):
    """A request of 290 particles per brick alone and beside one of 530, which widens the
    workgroup: its counts and trajectory.  (Lists of more than sixteen entries: a recount of
    fewer adds the same terms in the same order whatever its lanes.)"""
    from paper_2609_07842_amd import vbc
    print(f"[pool counts] f {f} {precision}", flush=True)
    reqs = [(6000, 0.3), (6000, 0.5)]
    descs = [vbc.replica(n, W.box_length(n, r), W.vbc_params(E_a=4.0, f=f), seed=n) for n, r in reqs]
    fps = [vbc.footprint(d, precision, brick=4, **OPTS) for d in descs]
    caps = dict(max_replicas=2, max_types=1, max_particles=sum(n for n, _ in reqs),
                max_slots=sum(q["slots"] for q in fps), max_bricks=sum(q["bricks"] for q in fps),
                max_cells=sum(q["cells"] for q in fps), max_bcap=max(q["bcap"] for q in fps), chains=False)
    got, blocks = [], []
    for mix in (False, True):
        pool = vbc.Pool(caps, precision=precision, brick=4, **OPTS)
        r = pool.admit(descs[0], *_state(*reqs[0], 0))
        if mix:
            pool.admit(descs[1], *_state(*reqs[1], 1))
        blocks.append(pool.options()["block"])
        off = pool.info(r)[1]
        out = []
        for _ in range(3):
            out.append(pool.count().cpu().numpy()[off:off + 6000].copy())
            pool.step(20, **INTEG)
            out += [t.cpu().numpy().copy() for t in pool.get_state(r)]
        pool.check()
        got.append(out)
    assert blocks[0] < 512 < blocks[1]
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("f", [2.0, 4.0])
def test_counts_do_not_depend_on_the_workgroup(f):
    from paper_2609_07842_amd import vbc
    n, rho = 6000, 0.3
    s = vbc.System(vbc.replica(n, W.box_length(n, rho), W.vbc_params(E_a=4.0, f=f)), precision="fp32", block=64)
    s.set_state(*_state(n, rho, 3))
    out = []
    for block in (64, 128, 256, 320, 512, 1024):
        s.tune_set(block=block)
        out.append(s.count().cpu().numpy().copy())
    assert all(np.array_equal(a, out[0]) for a in out)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_energies_in_a_pool_equal_those_alone(precision):
    """Per-system energy and virial, of an evaluation and summed over steps, of a request whose
    particles fill half of its box: its bricks of up to 600 particles take two rounds of the
    workgroup that its mean density asks for, one of the wider one it gets beside the other."""
    from paper_2609_07842_amd import vbc
    print(f"[pool energies] {precision}", flush=True)
    reqs = [(6000, 0.3), (6000, 0.5)]
    descs = [vbc.replica(n, W.box_length(n, r), W.vbc_params(E_a=4.0, f=4.0), seed=n) for n, r in reqs]
    fps = [vbc.footprint(d, precision, brick=4, rho_max=0.7, **OPTS) for d in descs]
    caps = dict(max_replicas=2, max_types=1, max_particles=sum(n for n, _ in reqs),
                max_slots=sum(q["slots"] for q in fps), max_bricks=sum(q["bricks"] for q in fps),
                max_cells=sum(q["cells"] for q in fps), max_bcap=max(q["bcap"] for q in fps), chains=False)
    x, v = _state(*reqs[0], 0)
    x[:, 0] *= 0.5
    got, blocks = [], []
    for mix in (False, True):
        pool = vbc.Pool(caps, precision=precision, brick=4, rho_max=0.7, **OPTS)
        r = pool.admit(descs[0], x, v)
        if mix:
            pool.admit(descs[1], *_state(*reqs[1], 1))
        blocks.append(pool.options()["block"])
        pool.thermo(True)
        UW = pool.force()[2][r].cpu().numpy().copy()
        pool.step(20, **INTEG)
        th = pool.thermo_read()[r]
        pool.check()
        got.append([UW, th["last"], th["sum"]])
    assert blocks[0] < 512 < blocks[1]
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("block", [256, 128])
def test_a_set_block_stays(block):
    """A pool's workgroup size, once set, does not follow the admitted replicas, also when it was
    set to the size that the pool had (256)."""
    from paper_2609_07842_amd import vbc
    d = vbc.replica(6000, W.box_length(6000, 0.5), W.vbc_params(E_a=4.0, f=4.0))
    fp = vbc.footprint(d, "fp32", brick=4, **OPTS)
    caps = dict(max_replicas=1, max_types=1, max_particles=6000, max_slots=fp["slots"], max_bricks=fp["bricks"],
                max_cells=fp["cells"], max_bcap=fp["bcap"], chains=False)
    pool = vbc.Pool(caps, precision="fp32", brick=4, **OPTS)
    assert pool.options()["block"] == 256
    pool.tune_set(block=block)
    pool.admit(d, *_state(6000, 0.5, 1))
    assert pool.options()["block"] == block
    pool.step(2, **INTEG)
    pool.check()


@pytest.mark.parametrize("precision,brick,n,rho,stage_cap", [("fp32", 5, 4400, 0.9, 4608), ("fp64", 4, 3700, 1.2, 3936)])
def test_energies_of_very_full_bricks(precision, brick, n, rho, stage_cap):
    """Bricks of more than 1024 particles (more sums of 64 than the force pass keeps at a time):
    energy and virial at every workgroup size, in bits, and against the oracle."""
    import oracle
    from paper_2609_07842_amd import vbc
    L, p = W.box_length(n, rho), W.vbc_params(E_a=4.0, f=9.0)
    x = W.uniform_positions(n, L, 5)
    nc = int(L / 2.4)
    c = np.minimum((x * (nc / L)).astype(int), nc - 1) // brick
    assert np.unique(c, axis=0, return_counts=True)[1].max() > 1024
    print(f"[full bricks] {precision} cells {nc}", flush=True)
    s = vbc.System(vbc.replica(n, L, p), precision=precision, brick=brick, block=64, k_max=160, stage_cap=stage_cap)
    s.set_state(x)
    out = []
    for block in (64, 320, 512, 1024):
        s.tune_set(block=block)
        out.append(s.force()[2].cpu().numpy()[0].copy())
    s.check()
    assert all(np.array_equal(a, out[0]) for a in out)
    ref = oracle.evaluate(x, L, p)
    want = np.concatenate([[ref["U"], ref["W"]], ref["Wt"]])
    assert np.abs(out[0] - want).max() <= (1e-10 if precision == "fp64" else 1e-5) * (np.abs(ref["e"]).sum() + np.abs(ref["Wt"]).max())
