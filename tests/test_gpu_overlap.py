"""Outputs that overlap the input by whole fields (a batch shifted inside one buffer): every
field of the input is read before any field of the output is written, also where the batch's
later passes run in parts (fields of 2^20 points whose node fields outgrow the Infinity
Cache)."""
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


# one part each, several fields a part, and (64^2) a batch that runs whole
@pytest.mark.parametrize("shape,precision,m_real,nrhs", [((1024, 1024), "fp64", 12, 3), ((128, 128, 64), "mixed", 12, 5),
                                                         ((1200, 960), "mixed", 16, 4), ((64, 64), "fp64", 5, 4)])
@pytest.mark.parametrize("shift", [1, 2, -1])
def test_shifted_output(hp, shape, precision, m_real, nrhs, shift):
    print(f"[case] overlap {shape} {precision} {nrhs} {shift}", flush=True)
    omega = 2 * np.pi * min(shape) / 10
    c = inputs.gaussian_random_field(shape, 4.0, 5)
    plan = hp.Plan(shape, omega, c, np.full(shape, 0.05 * omega), None, m_real=m_real, precision=precision, max_nrhs=nrhs)
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    g = torch.Generator(device="cuda").manual_seed(7)
    room = torch.view_as_complex(torch.randn((nrhs + abs(shift),) + shape + (2,), generator=g, dtype=torch.float64,
                                             device="cuda")).to(dt)
    v, out = (room[:nrhs], room[shift:]) if shift > 0 else (room[-shift:], room[:nrhs])
    want = plan.apply(v.clone())
    plan.apply(v, out=out)
    assert torch.equal(out, want)
    plan.close()
