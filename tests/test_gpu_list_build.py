"""The list build where its lanes' shares differ most: rows of more candidates than the masks it
keeps, lists longer than one output window (and than k_max), particle counts around the
particles of a wave, and a second build from the layout of the first.  Lists against the
oracle's exact neighbour set."""
import numpy as np
import pytest

import oracle
from paper_2609_07842_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

RL = 2.4  # list radius: r_h + skin


def _ball(n, lone, L, seed):
    rng = np.random.default_rng(seed)
    d = rng.normal(size=(n, 3))
    d *= rng.random((n, 1)) ** (1 / 3) / np.linalg.norm(d, axis=1, keepdims=True)
    x = np.concatenate([L - 0.3 + d, rng.uniform(0, L, size=(lone, 3))])  # across the periodic faces
    x = np.mod(x[rng.permutation(len(x))], L)
    return np.where(x >= L, 0.0, x)


def _listed(s):
    pairs, cnt = s.nlist_pairs(0)
    gpu = {(min(a, b), max(a, b)) for a, b in pairs.tolist()}
    assert cnt == 2 * len(gpu)  # every pair from both ends, once
    return gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("ball,lone,L,brick", [
    (0, 20, 7.3, 1), (0, 22, 9.7, 2), (0, 63, 7.3, 3), (0, 800, 12.1, 4),  # remainders of a wave's particles
    (40, 300, 14.5, 2),   # lists a little longer than a window
    (70, 300, 14.5, 1),   # rows of 33 to 64 candidates
    (300, 600, 14.5, 3),  # rows of several hundred candidates, lists of several windows
])
def test_lists_match_the_exact_neighbours(ball, lone, L, brick, precision):
    from paper_2609_07842_amd import vbc

    print(f"[list build] ball {ball} lone {lone} brick {brick} {precision}", flush=True)
    N = ball + lone
    x = _ball(ball, lone, L, seed=N)
    s = vbc.System(vbc.replica(N, L, W.vbc_params(E_a=5.0, f=2.0)), precision=precision, brick=brick,
                   k_max=400, stage_cap=1000)
    s.set_state(x)
    for build in range(2):  # from caller order, then from the first build's layout
        s.build_nlist()
        got = _listed(s)
        s.check()
        assert got == {tuple(p) for p in oracle.neighbor_pairs(x, L, RL).tolist()}


@pytest.mark.parametrize("k_max", [8, 72, 296])
def test_lists_longer_than_k_max_are_reported_and_cut(k_max):
    from paper_2609_07842_amd import vbc

    x = _ball(300, 100, 14.5, seed=1)
    s = vbc.System(vbc.replica(400, 14.5, W.vbc_params(E_a=5.0, f=2.0)), precision="fp32", brick=2,
                   k_max=k_max, stage_cap=1000)
    s.set_state(x)
    s.build_nlist()
    st, _ = s.check(raise_on_error=False)
    assert st == vbc.VBC_ERR_NLIST_OVERFLOW
    pairs, cnt = s.nlist_pairs(0)
    ref = {tuple(p) for p in oracle.neighbor_pairs(x, 14.5, RL).tolist()}
    deg = np.bincount(np.array(sorted(ref)).ravel(), minlength=400)
    assert cnt == np.minimum(deg, k_max).sum()
    assert {(min(a, b), max(a, b)) for a, b in pairs.tolist()} <= ref
