"""Batches whose node fields outgrow the Infinity Cache run in parts that share the node
fields' memory: every field of such a batch is bitwise the field applied alone, in place
and with a last part that is not full, and solves of a batch match single ones."""
import numpy as np
import pytest
import torch

from paper_2409_16172_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hp():
    from paper_2409_16172_amd import binding
    binding.load_library()
    return binding


# fields of 2^20 points: 1024^2 FP64 (one field a part), 128^3 mixed with 4 nodes (three
# fields a part, five fields)
@pytest.mark.parametrize("shape,precision,m_real,nrhs", [((1024, 1024), "fp64", 12, 3), ((128, 128, 64), "mixed", 12, 5)])
def test_batch_parts_equal_single(hp, shape, precision, m_real, nrhs):
    print(f"[case] batch parts {shape} {precision} {nrhs}", flush=True)
    omega = 2 * np.pi * min(shape) / 10
    c = inputs.gaussian_random_field(shape, 4.0, 5)
    plan = hp.Plan(shape, omega, c, np.full(shape, 0.05 * omega), None, m_real=m_real, precision=precision, max_nrhs=nrhs)
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    g = torch.Generator(device="cuda").manual_seed(3)
    v = torch.view_as_complex(torch.randn((nrhs,) + shape + (2,), generator=g, dtype=torch.float64, device="cuda")).to(dt)
    one = torch.stack([plan.apply(v[k]) for k in range(nrhs)])
    assert torch.equal(plan.apply(v), one)
    w = v.clone()
    plan.apply(w, out=w)
    assert torch.equal(w, one)
    f = v[:2].to(torch.complex128).contiguous()
    x, info = plan.solve(f, rtol=1e-3, max_cycles=2, restart=5)
    for k in range(2):
        xk, ik = plan.solve(f[k].contiguous(), rtol=1e-3, max_cycles=2, restart=5)
        assert torch.equal(x[k], xk) and ik[0].iters == info[k].iters
    plan.close()


def test_pass_times_of_a_batch_in_parts(hp):
    """A pass of a batch that runs in parts is one entry of the pass timer, as it is when the
    batch runs whole, and the profile's figures cover all of its fields."""
    print("[case] pass timer of batch parts", flush=True)
    shape, nrhs = (1024, 1024), 3
    omega = 2 * np.pi * min(shape) / 10
    c = inputs.gaussian_random_field(shape, 4.0, 5)
    plan = hp.Plan(shape, omega, c, np.full(shape, 0.05 * omega), None, m_real=12, max_nrhs=nrhs)
    g = torch.Generator(device="cuda").manual_seed(3)
    v = torch.view_as_complex(torch.randn((nrhs,) + shape + (2,), generator=g, dtype=torch.float64, device="cuda"))
    one = [plan.apply(v[k]) for k in range(nrhs)]
    for slot in (0, 2, 4):
        plan.time_pass(slot)
        plan.apply(v)
        plan.apply(v[0])
        plan.apply(v)
        t = plan.pass_times()
        assert len(t) == 3 and min(t) > 0
        # three fields take longer than one (by 1.5 at least: a field fills the chip)
        assert min(t[0], t[2]) > 1.5 * t[1]
    plan.time_pass(None)
    u = torch.empty_like(v)
    ms, _ = plan.profile_apply(v, out=u, reps=3)
    assert all(torch.equal(u[k], one[k]) for k in range(nrhs))
    ms1, _ = plan.profile_apply(v[0].contiguous(), reps=3)
    for slot in (0, 2, 4):
        assert ms[slot] > 1.5 * ms1[slot]
    plan.close()
