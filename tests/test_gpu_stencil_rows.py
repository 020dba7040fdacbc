"""The row-blocked 2-D stencil (grids of at least 2^18 points): row counts that its four
rows per thread do and do not divide, rows as short as eight points, and the residual and
mixed forms, against the oracle."""
import numpy as np
import pytest
import torch

from tests.util import rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hp():
    from paper_2409_16172_amd import binding
    binding.load_library()
    return binding


# 512 x 512 is the smallest the kernel takes; 486 = 4 * 121 + 2 rows; 10 and 4800 rows
@pytest.mark.parametrize("shape", [(512, 512), (486, 600), (4800, 60), (90, 3000)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_stencil_rows_match_oracle(orc, hp, shape, precision):
    print(f"[case] stencil rows {shape} {precision}", flush=True)
    rng = np.random.default_rng(sum(shape))
    omega = 2 * np.pi * min(shape) / 8
    c = 0.8 + 0.4 * rng.random(shape)
    a = omega * (0.05 + 0.1 * rng.random(shape))
    kw = dict(m_real=3, a_floor=0.05 * omega)
    plan = hp.Plan(shape, omega, c, a, None, precision=precision, max_nrhs=2, **kw)
    ref = orc.Problem(shape, omega, c, a, None, **kw)
    u = rng.standard_normal((2,) + shape) + 1j * rng.standard_normal((2,) + shape)
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    y = plan.matvec(torch.from_numpy(u).to("cuda").to(dt)).cpu().numpy()
    for k in range(2):
        assert rel(y[k], ref.matvec(u[k])) < (1e-13 if precision == "fp64" else 1e-6)
    plan.close()
