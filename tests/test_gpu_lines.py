"""The register mixed-radix lines (two, three and four stages, both radix bounds, rows and
columns that do not fill a workgroup, node splits and node groups) against the oracle:
lengths at the edges of the plan's rules, in both precisions and every interpolation."""
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


# lines: 10 = 5 2, 90 = 10 9 (radices up to 10), 240 = 16 15 (FP32) or 8 6 5 (FP64: the
# spectrum bound), 256 beside them, 486 and 600 (three stages), 1250 and 2000 (four),
# 2700 = 15 15 12 (the longest last radix), 2916 (four stages, FP32 and FP64); widths
# that are not multiples of the columns per workgroup, or fewer
SHAPES = [(10, 12), (90, 18), (240, 486), (1250, 10), (10, 2000), (2700, 18), (18, 2916), (256, 600), (30, 10, 54),
          (12, 250, 20)]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape", SHAPES)
def test_lines_match_oracle(orc, hp, shape, precision):
    print(f"[case] lines {shape} {precision}", flush=True)
    n = min(shape)
    rng = np.random.default_rng(sum(shape))
    c = 0.8 + 0.5 * rng.random(shape)
    omega = 2 * np.pi * n / 6
    a = np.full(shape, 0.05 * omega)
    kw = dict(m_real=9, a_floor=0.05 * omega)
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    v = rng.standard_normal((3,) + shape) + 1j * rng.standard_normal((3,) + shape)
    ref = orc.Problem(shape, omega, c, a, None, **kw)
    plan = hp.Plan(shape, omega, c, a, None, precision=precision, max_nrhs=2, **kw)
    u = plan.apply(torch.from_numpy(v).to("cuda").to(dt))
    one = plan.apply(torch.from_numpy(v[2].copy()).to("cuda").to(dt))
    assert torch.equal(u[2], one)            # batches of two and one sum alike
    for k in range(3):
        assert rel(u[k].cpu().numpy(), ref.apply(v[k])) < (1e-12 if precision == "fp64" else 1e-5)
    plan.close()


@pytest.mark.parametrize("kw", [dict(interp_order=3), dict(m_damp=3), dict(layer=True)])
@pytest.mark.parametrize("shape,precision", [((60, 600), "fp64"), ((96, 240), "mixed"), ((90, 1440), "fp64")])
def test_line_combine_interpolations(orc, hp, shape, precision, kw):
    print(f"[case] line combine {shape} {precision} {kw}", flush=True)
    kw = dict(kw)
    n = min(shape)
    rng = np.random.default_rng(sum(shape) + 1)
    omega = 2 * np.pi * n / 6
    c = inputs.gaussian_random_field(shape, 5.0, 3, lo=0.8, hi=1.3)
    a = omega * (0.05 + 0.2 * rng.random(shape)) if "m_damp" in kw else np.full(shape, 0.05 * omega)
    zeta = None
    if kw.pop("layer", False):
        c = inputs.blend_to_background(c, 6, 1.0, taper=4)
        zeta = inputs.frame_layer(shape, 6, 0.133)
        kw.update(m_layer=3)
    kw.update(m_real=8, a_floor=0.05 * omega)
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    v = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    plan = hp.Plan(shape, omega, c, a, zeta, precision=precision, **kw)
    u = plan.apply(torch.from_numpy(v).to("cuda").to(dt)).cpu().numpy()
    ref = orc.Problem(shape, omega, c, a, zeta, **kw).apply(v)
    assert rel(u, ref) < (1e-12 if precision == "fp64" else 1e-5)
    plan.close()


@pytest.mark.parametrize("shape,precision", [((180, 120), "mixed"), ((360, 240), "fp64"), ((90, 600), "fp64")])
def test_lines_per_workgroup_keep_results(hp, shape, precision, tmp_path, monkeypatch):
    """The lines a workgroup takes (a tuning choice) do not change a bit of the result."""
    print(f"[case] lines per workgroup {shape} {precision}", flush=True)
    omega = 2 * np.pi * min(shape) / 6
    c = inputs.gaussian_random_field(shape, 6.0, 9)
    a = np.full(shape, 0.05 * omega)
    make = lambda: hp.Plan(shape, omega, c, a, None, m_real=12, precision=precision)  # noqa: E731
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    rng = np.random.default_rng(4)
    v = torch.from_numpy(rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).to("cuda").to(dt)
    u0 = make().apply(v)
    for tc in (1, 2, 4, 8):
        path = tmp_path / f"tune{tc}.txt"
        prec = 0 if precision == "fp64" else 1
        path.write_text("".join(f"hp-tune 2 {shape[0]} {shape[1]} 1 {prec} 12 {s} 0 {tc} 0 0\n" for s in (0, 2, 4)))
        monkeypatch.setenv("HP_TUNE_CACHE", str(path))
        assert torch.equal(make().apply(v), u0)
        monkeypatch.delenv("HP_TUNE_CACHE")


@pytest.mark.parametrize("order,nthr", [(0, 128), (1, 0), (2, 0), (3, 0), (0, 192), (2, 128)])
@pytest.mark.parametrize("shape,precision", [((360, 240), "fp64"), ((240, 600), "mixed"), ((20, 60, 90), "fp64")])
def test_files_with_lds_schedules_keep_them(hp, shape, precision, order, nthr, tmp_path, monkeypatch):
    """A tuning file that names threads per line or a radix order means the LDS lines, as it
    did before lines were held in registers: the result is theirs, to rounding that of the
    register lines but not bit for bit, and lines per workgroup beside them change nothing."""
    print(f"[case] LDS schedules {shape} {precision} {order} {nthr}", flush=True)
    omega = 2 * np.pi * min(shape) / 6
    c = inputs.gaussian_random_field(shape, 5.0, 9)
    a = np.full(shape, 0.05 * omega)
    make = lambda: hp.Plan(shape, omega, c, a, None, m_real=6, precision=precision)  # noqa: E731
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    rng = np.random.default_rng(4)
    v = torch.from_numpy(rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).to("cuda").to(dt)
    u0 = make().apply(v)
    n = list(shape) + [1] * (3 - len(shape))
    got = []
    for tc in (0, 2):
        path = tmp_path / f"tune{tc}.txt"
        path.write_text("".join(f"hp-tune {len(shape)} {n[0]} {n[1]} {n[2]} {int(precision != 'fp64')} 6 {s} {nthr} {tc} "
                                f"{order} 0\n" for s in range(5)))
        monkeypatch.setenv("HP_TUNE_CACHE", str(path))
        plan = make()
        monkeypatch.delenv("HP_TUNE_CACHE")
        assert plan.info()["tune"] == [(nthr, tc, order, 0)] * 5
        got.append(plan.apply(v))
        assert rel(got[-1].cpu().numpy(), u0.cpu().numpy()) < (1e-12 if precision == "fp64" else 1e-5)
        assert not torch.equal(got[-1], u0)
    assert torch.equal(got[0], got[1])
