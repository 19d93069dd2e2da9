"""Clusters where the analysis leaves its usual path: bricks with more bonds into their
neighbours than the record holds (dense balls cut by bricks of one cell), histograms longer
than the one summed in LDS, clusters that span several bricks beside lone particles, in one
and in several replicas.  Every label and integer against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2609_07842_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _balls(L, nball, per, radius, lone, seed):
    """`nball` balls of `per` particles on a cubic grid with random offsets, and lone particles."""
    rng = np.random.default_rng(seed)
    m = int(np.ceil(nball ** (1 / 3)))
    grid = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)[:nball]
    cent = (grid + 0.5 + rng.uniform(-0.1, 0.1, size=(nball, 3))) * (L / m)
    d = rng.normal(size=(nball, per, 3))
    d *= (radius * rng.random((nball, per, 1)) ** (1 / 3)) / np.linalg.norm(d, axis=2, keepdims=True)
    x = np.concatenate([(cent[:, None, :] + d).reshape(-1, 3), rng.uniform(0, L, size=(lone, 3))])
    x = np.mod(x[rng.permutation(len(x))], L)
    return np.where(x >= L, 0.0, x)


@pytest.mark.parametrize("hist_len", [64, 5000])
@pytest.mark.parametrize("per,brick", [(200, 1), (200, 3), (5, 2)])
def test_dense_clusters_every_label(per, brick, hist_len):
    from paper_2609_07842_amd import vbc
    L, p = 20.0, W.vbc_params(E_a=5.0, f=4.0)
    xs = [_balls(L, 27, per, 1.7, 300, seed) for seed in (1, 2)]
    print(f"[dense clusters] {per} per ball, brick {brick}, hist {hist_len}", flush=True)
    if per == 200 and brick == 1:
        # some brick (here a cell of edge 2.5) has more bonds into bricks behind it than three
        # per slot (256 slots)
        c = (xs[0] / 2.5).astype(int) @ np.array([1, 8, 64])
        pr = oracle.bond_pairs(xs[0], L, p["r_a"])
        pr = np.array(sorted(pr) if isinstance(pr, set) else pr)
        lo, hi = np.minimum(c[pr[:, 0]], c[pr[:, 1]]), np.maximum(c[pr[:, 0]], c[pr[:, 1]])
        assert np.bincount(lo[lo != hi]).max() > 3 * 256
    cap = 27 * 64 if brick == 1 else 4400
    s = vbc.System([vbc.replica(len(x), L, p) for x in xs], precision="fp32", brick=brick, rho_max=12.0,
                   k_max=512, stage_cap=cap)
    s.set_state(np.concatenate(xs))
    lab, stats, hist = s.clusters(hist_len=hist_len)
    s.check()
    lab, stats, hist = lab.cpu().numpy(), stats.cpu().numpy(), hist.cpu().numpy()
    off = 0
    for r, x in enumerate(xs):
        ref, z = oracle.bond_clusters(x, L, p)
        assert np.array_equal(lab[off:off + len(x)], ref)
        st = oracle.cluster_stats(ref, z, hist_len)
        assert stats[r].tolist() == [st["clusters"], st["largest"], st["cyclic_particles"], st["bonds"],
                                     st["cyclic_clusters"]]
        assert np.array_equal(hist[r], st["hist"])
        off += len(x)
