"""Arnoldi on both sides of the sizes where its sweep and update change kernels: 4096 points
(update), 2^16 (sweep blocks), 2^17 (vectors in flight in the sweep) and 2^18 (update, 2-D
stencil).  The basis has to be orthonormal and satisfy A V = V H, with A applied by the
plan's own apply and matvec."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def hp():
    from paper_2409_16172_amd import binding
    binding.load_library()
    return binding


@pytest.mark.parametrize("shape", [(60, 64), (64, 64), (72, 60), (256, 256), (256, 270), (256, 512), (360, 384),
                                   (480, 540), (512, 512), (16, 16, 18), (64, 32, 32), (50, 54, 60)])
@pytest.mark.parametrize("side", ["none", "right"])
def test_arnoldi_relation_and_orthogonality(hp, shape, side):
    print(f"[case] arnoldi sizes {shape} {side}", flush=True)
    m = 20   # two rounds of the sweep (16 vectors each) and three of the update (8)
    rng = np.random.default_rng(sum(shape))
    omega = 2 * np.pi * min(shape) / 8
    c = 0.8 + 0.4 * rng.random(shape)
    plan = hp.Plan(shape, omega, c, np.full(shape, 0.1 * omega), None, m_real=3, a_floor=0.05 * omega)
    v0 = torch.from_numpy(rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).to("cuda")
    H, steps = plan.arnoldi(v0, m, side=side)
    assert steps == m
    V = torch.stack([plan.arnoldi_vector(np.eye(m)[k]).reshape(-1) for k in range(m)])
    # a second Gram-Schmidt pass leaves a few eps per vector; sums over N points in blocks
    # add a few more (100 allows for both)
    gram = (V.conj() @ V.T).cpu().numpy()
    assert np.abs(gram - np.eye(m)).max() < 100 * m * EPS
    for k in range(m - 1):   # column m - 1 has the provisional coefficients of its step
        v = V[k].reshape(shape).contiguous()
        w = plan.matvec(v if side == "none" else plan.apply(v)).reshape(-1)
        gap = w - torch.from_numpy(H[:m, k]).to("cuda") @ V
        assert float(gap.norm()) < 100 * m * EPS * np.abs(H).max(), k
    plan.close()
