"""Pass C of power-of-two rows with and without node splits: plans on both sides of the rule
that chooses them (row groups times max_nrhs, nodes, interpolation), and both forced by a
tuning file, against the oracle; one field equals the same field of a batch bit for bit."""
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


def _check(orc, hp, shape, precision, m_real, nrhs, mode):
    rng = np.random.default_rng(sum(shape) + nrhs)
    omega = 2 * np.pi * min(shape) / 8
    c = inputs.gaussian_random_field(shape, 4.0, 3, lo=0.8, hi=1.3)
    a = omega * (0.05 + 0.2 * rng.random(shape)) if mode == "bilinear" else np.full(shape, 0.05 * omega)
    kw = dict(m_real=m_real, a_floor=0.05 * omega)
    if mode == "lagrange":
        kw["interp_order"] = 3
    elif mode == "bilinear":
        kw["m_damp"] = 2
    plan = hp.Plan(shape, omega, c, a, None, precision=precision, max_nrhs=nrhs, **kw)
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    v = rng.standard_normal((nrhs,) + shape) + 1j * rng.standard_normal((nrhs,) + shape)
    vd = torch.from_numpy(v).to("cuda").to(dt)
    u = plan.apply(vd)
    ref = orc.Problem(shape, omega, c, a, None, **kw)
    k = nrhs - 1
    assert rel(u[k].cpu().numpy(), ref.apply(v[k])) < (1e-12 if precision == "fp64" else 1e-5)
    assert torch.equal(u[k], plan.apply(vd[k].contiguous()))
    plan.close()


# row groups x right-hand sides 512 and just above, 1024 and just above, with ten and eleven
# nodes (bilinear: twice six); one and more rows to a wavefront, a last group that is not full
@pytest.mark.parametrize("mode", ["linear", "lagrange", "bilinear"])
@pytest.mark.parametrize("shape,precision,m_real,nrhs",
                         [((256, 256), "mixed", 11, 8), ((256, 256), "mixed", 10, 8), ((180, 256), "mixed", 11, 12),
                          ((512, 512), "mixed", 11, 2), ((512, 512), "mixed", 10, 3), ((256, 512), "mixed", 11, 8),
                          ((256, 1024), "mixed", 6, 2), ((256, 1024), "mixed", 11, 3), ((1024, 1024), "mixed", 11, 1),
                          ((90, 128), "mixed", 5, 3), ((18, 64), "fp64", 5, 2), ((256, 128), "fp64", 6, 8),
                          ((512, 256), "fp64", 11, 4), ((128, 512), "fp64", 11, 8), ((128, 512), "fp64", 5, 5)])
def test_splits_match_oracle(orc, hp, shape, precision, m_real, nrhs, mode):
    print(f"[case] combine splits {shape} {precision} {m_real} x{nrhs} {mode}", flush=True)
    _check(orc, hp, shape, precision, m_real if mode != "bilinear" else (m_real + 1) // 2, nrhs, mode)


@pytest.mark.parametrize("ng", [1, 4])
@pytest.mark.parametrize("shape,precision", [((64, 8), "fp64"), ((30, 32), "mixed"), ((64, 256), "mixed"),
                                             ((48, 512), "mixed"), ((32, 1024), "mixed"), ((32, 512), "fp64")])
@pytest.mark.parametrize("mode", ["linear", "lagrange", "bilinear"])
def test_forced_splits_match_oracle(orc, hp, shape, precision, ng, mode, tmp_path, monkeypatch):
    print(f"[case] forced combine splits {shape} {precision} {ng} {mode}", flush=True)
    K = 5 if mode != "bilinear" else 10
    path = tmp_path / "tune.txt"
    path.write_text(f"hp-tune 2 {shape[0]} {shape[1]} 1 {int(precision != 'fp64')} {K} 4 0 0 0 {ng}\n")
    monkeypatch.setenv("HP_TUNE_CACHE", str(path))
    _check(orc, hp, shape, precision, 5, 2, mode)
