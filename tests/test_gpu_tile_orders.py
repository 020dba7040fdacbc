"""Power-of-two columns and rows at tile counts that eight does not divide (the workgroups'
column tiles are dealt to the XCDs over slabs and node groups) and FP32 lines of 256 points
on grids with many rows (node splits), against the oracle; a batch equals single applies."""
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


# columns beside a power-of-two axis 0 (and middle axis): one tile, fewer than eight, odd
# counts and a remainder inside a tile; then 256-point rows, 1024 to 4096 of them
@pytest.mark.parametrize("shape", [(1024, 8), (1024, 10), (256, 30), (512, 54), (128, 90), (64, 32, 18), (32, 16, 50),
                                   (16, 64, 10), (1024, 256), (16, 64, 256), (32, 128, 256)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("m_real", [2, 5])
def test_tile_orders_match_oracle(orc, hp, shape, precision, m_real):
    print(f"[case] tile orders {shape} {precision} {m_real}", flush=True)
    rng = np.random.default_rng(sum(shape) + m_real)
    omega = 2 * np.pi * max(shape) / 10
    c = 0.8 + 0.4 * rng.random(shape)
    a = omega * (0.05 + 0.1 * rng.random(shape))
    kw = dict(m_real=m_real, a_floor=0.05 * omega)
    plan = hp.Plan(shape, omega, c, a, None, precision=precision, max_nrhs=2, **kw)
    ref = orc.Problem(shape, omega, c, a, None, **kw)
    v = rng.standard_normal((2,) + shape) + 1j * rng.standard_normal((2,) + shape)
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    vd = torch.from_numpy(v).to("cuda").to(dt)
    u = plan.apply(vd)
    for k in range(2):
        assert rel(u[k].cpu().numpy(), ref.apply(v[k])) < (1e-12 if precision == "fp64" else 1e-5)
        assert torch.equal(u[k], plan.apply(vd[k].contiguous()))
    plan.close()
