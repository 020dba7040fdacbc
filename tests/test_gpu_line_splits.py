"""Pass C of mixed-radix rows on both sides of its choices: line splits by the radices and the
threads of the plan's largest launch, and the Lagrange rows that keep the LDS lines, against
the oracle; one field equals the same field of a batch."""
import numpy as np
import pytest
import torch

from paper_2409_16172_amd import inputs
from tests.util import rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hp():
    from paper_2409_16172_amd import binding
    binding.load_library()
    return binding


# rows of 320 points (8 8 5) take 64 threads: 200 of them 12.8k threads a
# field; 1296 = 12 12 9; 600 = 10 10 6, 100 threads
@pytest.mark.parametrize("order", [2, 3])
@pytest.mark.parametrize("shape,precision,nrhs", [((200, 320), "fp64", 1), ((200, 320), "fp64", 4), ((200, 320), "mixed", 8),
                                                  ((200, 320), "mixed", 2), ((36, 1296), "mixed", 2), ((36, 1296), "fp64", 2),
                                                  ((360, 600), "fp64", 3), ((10, 12, 90), "mixed", 3),
                                                  ((300, 576), "mixed", 1), ((400, 576), "mixed", 2), ((60, 144), "mixed", 2),
                                                  ((18, 1944), "fp64", 2), ((18, 2000), "mixed", 2),
                                                  ((18, 1620), "fp64", 2), ((18, 2500), "fp64", 1)])
def test_lagrange_lines_match_oracle(orc, hp, shape, precision, nrhs, order):
    print(f"[case] line splits {shape} {precision} x{nrhs} order {order}", flush=True)
    rng = np.random.default_rng(sum(shape) + nrhs)
    omega = 2 * np.pi * min(shape) / 8
    c = inputs.gaussian_random_field(shape, 4.0, 3, lo=0.8, hi=1.3)
    kw = dict(m_real=9, a_floor=0.05 * omega, interp_order=order)
    a = np.full(shape, 0.05 * omega)
    plan = hp.Plan(shape, omega, c, a, None, precision=precision, max_nrhs=nrhs, **kw)
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    v = rng.standard_normal((nrhs,) + shape) + 1j * rng.standard_normal((nrhs,) + shape)
    vd = torch.from_numpy(v).to("cuda").to(dt)
    u = plan.apply(vd)
    k = nrhs - 1
    ref = orc.Problem(shape, omega, c, a, None, **kw).apply(v[k])
    assert rel(u[k].cpu().numpy(), ref) < (1e-12 if precision == "fp64" else 1e-5)
    assert torch.equal(u[k], plan.apply(vd[k].contiguous()))
    plan.close()


# linear rows with radices above ten (1440) on both sides of 72k threads, others with four and
# two splits
@pytest.mark.parametrize("shape,precision,nrhs", [((180, 240), "fp64", 2), ((180, 240), "fp64", 8), ((128, 1440), "mixed", 1),
                                                  ((128, 1440), "mixed", 4), ((100, 576), "fp64", 12), ((60, 720), "mixed", 16)])
def test_linear_lines_match_oracle(orc, hp, shape, precision, nrhs):
    print(f"[case] linear line splits {shape} {precision} x{nrhs}", flush=True)
    rng = np.random.default_rng(sum(shape) + nrhs)
    omega = 2 * np.pi * min(shape) / 8
    c = 0.8 + 0.5 * rng.random(shape)
    a = np.full(shape, 0.05 * omega)
    kw = dict(m_real=9, a_floor=0.05 * omega)
    plan = hp.Plan(shape, omega, c, a, None, precision=precision, max_nrhs=nrhs, **kw)
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    v = rng.standard_normal((2,) + shape) + 1j * rng.standard_normal((2,) + shape)
    vd = torch.from_numpy(v).to("cuda").to(dt)
    u = plan.apply(vd)
    assert rel(u[1].cpu().numpy(), orc.Problem(shape, omega, c, a, None, **kw).apply(v[1])) < (1e-12 if precision == "fp64" else 1e-5)
    assert torch.equal(u[1], plan.apply(vd[1].contiguous()))
    plan.close()
