"""Passes in two launches (bricks of usual density, then dense ones) against passes in one: a
dilute system of many small bricks, laid out for a high local density, with a dense ball in it.
The workgroup size decides which of the two the count and force passes are; one and several
replicas."""
import numpy as np
import pytest

import oracle
from paper_2609_07842_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

L = 53.0


def _state(seed, ball):
    rng = np.random.default_rng(seed)
    d = rng.normal(size=(ball, 3))
    d *= rng.random((ball, 1)) ** (1 / 3) / np.linalg.norm(d, axis=1, keepdims=True)
    x = np.concatenate([rng.uniform(0, L, 3) + d, rng.uniform(0, L, size=(3000 - ball, 3))])
    x = np.mod(x[rng.permutation(3000)], L)
    return np.where(x >= L, 0.0, x)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("reps,ball", [(1, 150), (1, 0), (3, 60)])
def test_two_launches_give_the_results_of_one(reps, ball, precision):
    from paper_2609_07842_amd import vbc

    p = W.vbc_params(E_a=5.0, f=2.0)
    x = np.concatenate([_state(k, ball) for k in range(reps)])
    v = W.maxwell_boltzmann(len(x), 1.0, 6)
    got = {}
    for block in (1024, 64):  # one launch; two
        print(f"[dense bricks] {reps} ball {ball} {precision} block {block}", flush=True)
        s = vbc.System([vbc.replica(3000, L, p) for _ in range(reps)], precision=precision, brick=1, block=block,
                       rho_max=3.0)
        s.set_state(x, v)
        s.build_nlist()
        for r in range(reps):
            pairs, cnt = s.nlist_pairs(r)
            ref = {tuple(q) for q in oracle.neighbor_pairs(x[3000 * r:3000 * (r + 1)], L, 2.4).tolist()}
            assert {(min(a, b), max(a, b)) for a, b in pairs.tolist()} == ref and cnt == 2 * len(ref)
        n = s.count().cpu().numpy()
        F, e, _ = s.force()
        z, pen, _ = s.observables()
        got[block] = [n, F.cpu().numpy(), e.cpu().numpy()]
        ints = [z.cpu().numpy(), pen.cpu().numpy(), s.clusters()[0].cpu().numpy()]
        tr = s.bond_tracker(max_partners=64, hist_len=16, bin_steps=1)
        s.step(3, integrator="nve", dt=0.0002)
        tr.sample()
        ints += [tr.stats.cpu().numpy(), tr.hist.cpu().numpy()]
        got[block].append(s.get_state()[0].cpu().numpy())
        got[block].append(ints)
        s.check()
    for a, b in zip(got[64][-1], got[1024][-1]):
        assert np.array_equal(a, b)
    for a, b in zip(got[64][:-1], got[1024][:-1]):
        if precision == "fp64":
            assert np.array_equal(a, b)
        else:
            # the recount of window particles adds a list's terms in an order that follows the
            # workgroup (1e-13 of a count), which can flip the last bit of a switching factor
            # (2^-24); a force has at most 150 terms of 50 times two such factors
            assert np.abs(a - b).max() <= 150 * 50 * 2 * 2.0 ** -24
