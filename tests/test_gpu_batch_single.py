"""Mixed-precision solves of several right-hand sides against the same solves one by one and
in groups: bit for bit.  A single right-hand side on these grids steps through the grouped
kernels, several through the plan's own; the grids lie on both sides of every size at which
either changes its kernels (node splits of pass C, blocks and vectors in flight of the
sweep, points per thread of the update), and past the grouped kernels' range."""
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


def _plan(hp, shape, m_real, nrhs, **kw):
    omega = 2 * np.pi * min(shape) / 10
    c = inputs.gaussian_random_field(shape, 6.0, sum(shape))
    a = np.full(shape, 0.05 * omega)
    if "m_damp" in kw:
        a = a * (1.0 + np.random.default_rng(3).random(shape))
    return hp.Plan(shape, omega, c, a, None, m_real=m_real, precision="mixed", max_nrhs=nrhs, **kw)


def _sources(shape, n):
    g = torch.Generator(device="cuda").manual_seed(sum(shape))
    return torch.view_as_complex(torch.randn((n,) + shape + (2,), generator=g, dtype=torch.float64, device="cuda"))


CASES = [((256, 256), 5, {}), ((256, 256), 16, {}), ((512, 256), 16, {}), ((256, 512), 5, {}), ((512, 512), 12, {}),
         ((512, 1024), 9, {}), ((1024, 512), 5, {}), ((1024, 1024), 16, {}), ((1024, 1024), 5, {}),
         ((512, 512), 12, {"interp_order": 3}), ((256, 256), 9, {"interp_order": 2}), ((1024, 256), 6, {"m_damp": 2}),
         ((128, 128, 128), 4, {}), ((128, 128, 256), 4, {}), ((240, 256), 9, {}), ((64, 96, 32), 5, {})]


@pytest.mark.parametrize("shape,m_real,kw", CASES)
def test_batch_solve_equals_single(hp, shape, m_real, kw):
    print(f"[case] batch solve {shape} {m_real} {kw}", flush=True)
    plan = _plan(hp, shape, m_real, 2, **kw)
    f = _sources(shape, 2)
    opts = dict(rtol=1e-12, max_cycles=2, restart=7)   # two cycles, seven steps each
    x, info = plan.solve(f, **opts)
    for k in range(2):
        xk, ik = plan.solve(f[k].contiguous(), **opts)
        assert ik[0].iters == info[k].iters
        assert torch.equal(x[k], xk), float((x[k] - xk).abs().max() / xk.abs().max())
    plan.close()


# FP64, where one right-hand side on up to 2^16 points takes a sweep of its own
@pytest.mark.parametrize("shape,side", [((64, 64), "right"), ((60, 54), "none"), ((128, 90), "left"), ((256, 256), "right"),
                                        ((256, 250), "none"), ((256, 270), "right"), ((16, 16, 18), "right"),
                                        ((40, 40, 40), "left"), ((48, 40, 36), "right")])
def test_fp64_batch_solve_equals_single(hp, shape, side):
    print(f"[case] FP64 batch solve {shape} {side}", flush=True)
    omega = 2 * np.pi * min(shape) / 10
    c = inputs.gaussian_random_field(shape, 4.0, sum(shape))
    plan = hp.Plan(shape, omega, c, np.full(shape, 0.05 * omega), None, m_real=5, max_nrhs=2)
    f = _sources(shape, 3)
    opts = dict(rtol=1e-12, max_cycles=2, restart=21, side=side)   # sweeps over one and two rounds of vectors
    x, info = plan.solve(f, **opts)
    for k in range(3):
        xk, ik = plan.solve(f[k].contiguous(), **opts)
        assert ik[0].iters == info[k].iters
        assert torch.equal(x[k], xk), float((x[k] - xk).abs().max() / xk.abs().max())
    plan.close()


def test_grouped_solves_equal_batch(hp):
    """Members with and without node splits, with either update, in one group."""
    print("[case] grouped against batch", flush=True)
    shapes = [((256, 256), 16, {}), ((1024, 1024), 5, {}), ((512, 512), 12, {"interp_order": 3}), ((512, 256), 9, {}),
              ((256, 1024), 9, {"interp_order": 3})]
    plans = [_plan(hp, s, m, 2, **kw) for s, m, kw in shapes]
    fs = [_sources(s, 2) for s, _, _ in shapes]
    want = [p.solve(f, rtol=1e-12, max_cycles=2, restart=7)[0][0] for p, f in zip(plans, fs)]
    solvers = [hp.Solver(p, 1, restart=7, rtol=1e-12, max_cycles=2) for p in plans]
    for s, f in zip(solvers, fs):
        s.start(f[0].contiguous())
    left = list(solvers)
    for _ in range(100000):
        left = [s for s, d in zip(left, hp.advance_group(left, 2)) if not d]
        if not left:
            break
    for s, w in zip(solvers, want):
        assert torch.equal(s.result()[0].reshape(w.shape), w)
        s.close()
    for p in plans:
        p.close()


@pytest.mark.parametrize("ng", [0, 1, 4])
@pytest.mark.parametrize("m_real", [5, 12])
def test_any_node_splits_step_in_groups(hp, ng, m_real, tmp_path, monkeypatch):
    """A tuned number of node splits, also the one that the plan takes by itself, leaves a
    session in the grouped launches (which the pass timer does not record, as it does the
    plan's own) and its solve bitwise that of a batch."""
    print(f"[case] grouped node splits {ng} {m_real}", flush=True)
    shapes = [(512, 512), (256, 1024)]
    path = tmp_path / "tune.txt"
    path.write_text("".join(f"hp-tune 2 {s[0]} {s[1]} 1 1 {m_real} 4 0 0 0 {ng}\n" for s in shapes))
    monkeypatch.setenv("HP_TUNE_CACHE", str(path))
    plans = [_plan(hp, s, m_real, 2) for s in shapes]
    monkeypatch.delenv("HP_TUNE_CACHE")
    fs = [_sources(s, 2) for s in shapes]
    opts = dict(restart=6, rtol=1e-12, max_cycles=1)
    want = [p.solve(f, **opts)[0][0] for p, f in zip(plans, fs)]
    solvers = [hp.Solver(p, 1, **opts) for p in plans]
    for p, s, f in zip(plans, solvers, fs):
        assert p.info()["tune"][4][3] == ng
        s.start(f[0].contiguous())
        p.time_pass(2)
    left = list(solvers)
    for _ in range(100000):
        left = [s for s, d in zip(left, hp.advance_group(left, 2)) if not d]
        if not left:
            break
    for p, s, w in zip(plans, solvers, want):
        assert torch.equal(s.result()[0].reshape(w.shape), w)
        assert len(p.pass_times()) <= 2     # start and end of the cycle, no step
        s.close()
        p.close()


@pytest.mark.parametrize("shape,m_real,nrhs,own", [((256, 256), 12, 1, 4), ((512, 512), 5, 8, 1)])
def test_autotuner_leaves_the_own_node_splits(hp, shape, m_real, nrhs, own):
    print(f"[case] autotuned node splits {shape} {m_real} x{nrhs}", flush=True)
    plan = _plan(hp, shape, m_real, nrhs)
    for _ in range(3):
        plan.autotune()
        assert plan.info()["tune"][4][3] != own
    plan.close()
