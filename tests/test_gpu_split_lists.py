"""FP64 passes with several lanes per particle against the same passes with one, bit for bit:
workgroup sizes on both sides of the rule, lists of fewer chunks than lanes, brick remainders,
one and two types."""
import numpy as np
import pytest

from paper_2609_07842_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("types", [1, 2])
@pytest.mark.parametrize("N,rho,f", [(117, 0.3, 2.0), (1000, 0.15, 3.0), (4001, 0.5, 10.0)])
def test_lanes_per_particle_do_not_change_results(N, rho, f, types):
    from paper_2609_07842_amd import vbc

    L = W.box_length(N, rho)
    x = W.uniform_positions(N, L, 5)
    v = W.maxwell_boltzmann(N, 1.0, 6)
    p = W.vbc_params(E_a=5.0, f=f)
    if types == 2:
        p = [p] * 4
    got = {}
    for block in (512, 320, 192, 64):  # one lane; two; four; four over several rounds
        print(f"[split] N {N} types {types} block {block}", flush=True)
        s = vbc.System(vbc.replica(N, L, p), precision="fp64", block=block)
        s.set_state(x, v, types=np.arange(N, dtype=np.int32) % types)
        n = s.count().cpu().numpy()
        F = s.force(energies=False)[0].cpu().numpy()
        s.step(3, integrator="nve", dt=0.001)
        got[block] = (n, F, s.get_state()[0].cpu().numpy())
        s.check()
    n0, F0, x0 = got[512]
    for block in (320, 192, 64):
        n, F, x1 = got[block]
        # the chunks' sums are added in the same order whatever the lanes
        assert np.array_equal(n, n0) and np.array_equal(F, F0) and np.array_equal(x1, x0)
