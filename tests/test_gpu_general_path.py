"""The general pair path (several types, count masks, chain exclusions) against the FP64
oracle where its branch-free pair terms could go wrong: absent attraction (E_a = 0), absent
core (E_r = 0), asymmetric count masks, a shifted window and different ranges per pair,
with 2 to 4 types, in both precisions (bars of the parity tests: 1e-10 and 1e-5 normwise)."""
import numpy as np
import pytest

import oracle
from paper_2609_07842_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _table(nt, rng):
    """Symmetric pair table: each absent term occurs, valencies and ranges differ by pair."""
    tab = [[None] * nt for _ in range(nt)]
    k = 0
    for a in range(nt):
        for b in range(a, nt):
            r_a = 1.5 - 0.1 * (k % 2)
            p = W.vbc_params(E_r=0.0 if k % 4 == 2 else 20.0, E_a=0.0 if k % 3 == 1 else 5.0, r_a=r_a,
                             r_l=1.4, r_h=1.9 + 0.1 * (k % 2), f=float(1 + k % 4), delta=0.2 * (k % 3))
            tab[a][b] = tab[b][a] = p
            k += 1
    return [tab[a][b] for a in range(nt) for b in range(nt)]


@pytest.mark.parametrize("excl", [0, 2])
@pytest.mark.parametrize("nt", [2, 3, 4])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("fp32", 1e-5)])
def test_general_path_parity(nt, excl, precision, tol):
    from paper_2609_07842_amd import vbc
    rng = np.random.default_rng(10 * nt + excl)
    N, L = 1210, W.box_length(1210, 0.25)
    params = _table(nt, rng)
    x = W.uniform_positions(N, L, seed=nt)
    types = rng.integers(0, nt, size=N).astype(np.int32)
    mask = np.array([(0b1011 >> t) | 1 << (nt - 1) for t in range(nt)], dtype=np.uint32)
    print(f"[general] types {nt} exclusions {excl} {precision}", flush=True)
    chain = dict(chain_len=10, excl_span=excl) if excl else {}
    ref = oracle.evaluate(x, L, params, types, mask, **chain)
    s = vbc.System(vbc.replica(N, L, params, mask=mask, **chain), precision=precision)
    s.set_state(x, types=types)
    n = s.count().cpu().numpy()
    F, e, UW = s.force()
    s.check()
    F = F.cpu().numpy()
    assert np.abs(n - ref["n"]).max() <= (1e-12 if precision == "fp64" else 1e-5)
    assert np.linalg.norm(F - ref["F"], axis=1).max() <= tol * np.linalg.norm(ref["F"], axis=1).max()
    es = np.abs(ref["e"]).sum()
    assert np.abs(e.cpu().numpy() - ref["e"]).max() <= tol * max(1.0, np.abs(ref["e"]).max())
    assert abs(UW[0, 0].item() - ref["U"]) <= tol * es
    Wref = np.concatenate([[ref["W"]], ref["Wt"]])
    assert np.abs(UW[0, 1:8].cpu().numpy() - Wref).max() <= tol * (np.abs(Wref).max() + es)
