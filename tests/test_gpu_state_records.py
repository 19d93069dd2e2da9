"""Reading back a large replica by way of records: every coordinate in its place, bit for bit,
on both sides of the sizes that take that path, before and after steps."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N", [299_999, 300_000, 300_001])
def test_large_states_come_back_in_caller_order(N):
    from paper_2609_07842_amd import vbc, workloads as W

    print(f"[state records] N {N}", flush=True)
    L = W.box_length(N, 0.3)
    gen = torch.Generator(device="cuda").manual_seed(N)
    x = torch.rand((N, 3), generator=gen, device="cuda", dtype=torch.float64) * L
    v = torch.randn((N, 3), generator=gen, device="cuda", dtype=torch.float64)
    s = vbc.System(vbc.replica(N, L, W.vbc_params(E_a=5.0, f=3.0)), precision="fp32")
    s.set_state(x, v)
    s.build_nlist()
    for _ in range(2):
        xs, vs = s.get_state()
        assert torch.equal(xs, x) and torch.equal(vs, v)
    # steps too short to change a double leave the state as it is
    s.step(2, integrator="nve", dt=1e-300)
    xs, vs = s.get_state()
    assert torch.equal(xs, x) and torch.equal(vs, v)
    s.clusters()  # its records share the space
    xs, vs = s.get_state()
    assert torch.equal(xs, x) and torch.equal(vs, v)
    s.check()
