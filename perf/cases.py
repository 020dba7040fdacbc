"""The work a user of the preconditioner has it do, as cases that can be timed and compared.

A case is one call, or one short sequence of calls, through the Python binding: applies of
Q_M (the inner operation of every Krylov step), products with P_N, whole GMRES solves, and
several resumable solves advanced together as a serving loop does.

listed()              the cases
draw(rng)             one more case of the same ranges
prepare(case, seed)   inputs on the GPU and the plan a program keeps
run(state)            one pass
work(case)            bytes and floating point operations the pass cannot do without
exact(case, seed)     the pass's result in 64-bit torch, without the library
"""
import math

import numpy as np
import torch

from paper_2409_16172_amd import binding

C0 = 1.0            # background wave speed
ZETA_MAX = 0.133    # absorbing layer strength at the edge
NODES_LAYER = 3


def _case(name, op, shape, precision, medium, m_real, nrhs=1, order=1, symbol="continuous", rtol=0.0):
    return {"name": name, "op": op, "shape": shape, "precision": precision, "medium": medium, "m_real": m_real,
            "nrhs": nrhs, "order": order, "symbol": symbol, "rtol": rtol}


def listed():
    return [
        # the smallest call: one apply on the 64 x 64 bump, bound by latency and launches
        _case("apply_64_fp64", "apply", "64x64", "fp64", "bump", 8),
        # a small served grid in mixed precision
        _case("apply_256_mixed", "apply", "256x256", "mixed", "grf", 16),
        # the apply inside the benchmark solve
        _case("apply_1024_fp64", "apply", "1024x1024", "fp64", "grf", 16),
        # the large mixed-precision grid, 24 + 3 nodes
        _case("apply_2048_mixed", "apply", "2048x2048", "mixed", "grf", 24),
        # a middle size of the paper's Table 1, N = 180 * 2^k, lines of mixed radix
        _case("apply_720_fp64", "apply", "720x720", "fp64", "inclusion", 4),
        # Example 1 of the paper: 200 wavelengths at 12 points each
        _case("apply_2400_fp64", "apply", "2400x2400", "fp64", "inclusion", 8),
        # a batch of sources in a 3-D medium
        _case("apply_128c_mixed_x4", "apply", "128x128x128", "mixed", "grf", 16, nrhs=4),
        # a 3-D box with three different sides, none a power of two
        _case("apply_box_fp64", "apply", "90x120x150", "fp64", "grf", 8),
        # the finite-difference operator by itself (residuals, other solvers)
        _case("matvec_1024_fp64", "matvec", "1024x1024", "fp64", "grf", 16),
        # whole solves: a small grid (short kernels, many steps) and the benchmark's
        _case("solve_256_fp64", "solve", "256x256", "fp64", "grf", 16, rtol=1e-8),
        _case("solve_1024_fp64", "solve", "1024x1024", "fp64", "grf", 16, rtol=1e-8),
        # a server's turn loop: uneven grids in mixed precision, two streams, tight tolerance
        _case("serve_mixed", "serve", "256x256,512x512,128x128x128,512x256,256x512,1024x512", "mixed", "grf", 16,
              rtol=1e-10),
    ]


def _smooth(lo, hi):
    """Even products of 2, 3 and 5 in [lo, hi]."""
    out = []
    for n in range(lo + lo % 2, hi + 1, 2):
        m = n
        for p in (2, 3, 5):
            while m % p == 0:
                m //= p
        if m == 1:
            out.append(n)
    return out


def _side(rng, lo, hi, pow2):
    """A side length, spread over the logarithm of [lo, hi]."""
    pick = [n for n in _smooth(lo, hi) if (n & (n - 1) == 0) == pow2]
    at = math.log(lo) + rng.random() * math.log(hi / lo)
    return min(pick, key=lambda n: abs(math.log(n) - at))


def draw(rng):
    op = rng.choice(["apply2", "apply2", "apply2", "apply2", "apply3", "apply3", "matvec", "solve", "solve", "serve"])
    precision = rng.choice(["fp64", "mixed"])
    medium = rng.choice(["grf", "grf", "inclusion"])
    m_real = rng.choice([4, 8, 12, 16, 24])
    order = rng.choice([1, 1, 1, 1, 3])
    symbol = rng.choice(["continuous", "continuous", "discrete"])
    pow2 = rng.random() < 0.5
    if op == "serve":
        sides = [_side(rng, 256, 512, True) for _ in range(8)]
        shape = ",".join("%dx%d" % (sides[2 * k], sides[2 * k + 1]) for k in range(rng.choice([3, 4])))
        return _drawn("serve", shape, "mixed", "grf", rng.choice([8, 12, 16]), rtol=1e-10)
    if op == "solve":
        n = _side(rng, 96, 768, pow2)
        return _drawn("solve", "%dx%d" % (n, _side(rng, max(96, n // 2), min(768, 2 * n), pow2)), "fp64", "grf",
                      rng.choice([8, 12, 16]), rtol=1e-8)
    if op == "matvec":
        n = _side(rng, 64, 2400, pow2)
        return _drawn("matvec", "%dx%d" % (n, _side(rng, max(64, n // 2), min(2400, 2 * n), pow2)), precision, medium,
                      m_real, nrhs=rng.choice([1, 1, 4]))
    if op == "apply3":
        while True:
            n = [_side(rng, 32, 192, pow2 if k else rng.random() < 0.5) for k in range(3)]
            nrhs = rng.choice([1, 2, 4])
            if n[0] * n[1] * n[2] * nrhs * (m_real + 4) <= 160 * 160 * 160 * 40:
                return _drawn("apply", "x".join(map(str, n)), precision, "grf", m_real, nrhs, order, symbol)
    while True:
        n = _side(rng, 64, 2400, pow2)
        m = n if rng.random() < 0.5 else _side(rng, max(64, n // 4), min(2400, 4 * n), rng.random() < 0.5)
        nrhs = rng.choice([1, 1, 1, 2, 3, 8])
        if n * m * nrhs * (m_real + 4) <= 2400 * 2400 * 12:
            return _drawn("apply", "%dx%d" % (n, m), precision, medium, m_real, nrhs, order, symbol)


def _drawn(op, shape, precision, medium, m_real, nrhs=1, order=1, symbol="continuous", rtol=0.0):
    c = _case("", op, shape, precision, medium, m_real, nrhs, order, symbol, rtol)
    del c["name"]
    return c


def _shapes(case):
    return [tuple(int(s) for s in t.split("x")) for t in case["shape"].split(",")]


# ---------------------------------------------------------------- inputs
def _along(x, k, dim):
    """The 1-D tensor x along axis k of dim, broadcastable."""
    return x.reshape([-1 if i == k else 1 for i in range(dim)])


def _axes(shape):
    """Coordinates of the unit box centred at the origin, one broadcastable tensor per axis."""
    return [_along(torch.arange(n, dtype=torch.float64, device="cuda") / n - 0.5, k, len(shape))
            for k, n in enumerate(shape)]


def _edge_cells(shape):
    """Cells to the nearest edge of the box."""
    e = torch.full(shape, math.inf, dtype=torch.float64, device="cuda")
    for k, n in enumerate(shape):
        i = torch.arange(n, dtype=torch.float64, device="cuda")
        e = torch.minimum(e, _along(torch.minimum(i, n - 1 - i), k, len(shape)))
    return e


def _medium(case, shape, seed):
    """Wave speed, damping, layer profile (or None), frequency and damping floor."""
    x = _axes(shape)
    n = min(shape)
    if case["medium"] == "inclusion":      # no layer, constant damping, 12 points per wavelength
        r = torch.sqrt(sum(t * t for t in x))
        radius = 0.05 * (1.0 + 0.01 * (seed % 7))
        c = C0 + 4.0 * 0.5 * (1.0 + torch.tanh(0.5 * (radius - r) * 800.0))
        a = torch.full(shape, 20.0, dtype=torch.float64, device="cuda")
        return c.expand(shape), a, None, 2.0 * math.pi * n / 12.0, 0.0
    gen = torch.Generator().manual_seed(seed)
    if case["medium"] == "bump":
        width, omega = max(2, n // 8), 2.0 * math.pi * n / 8.0
        at = torch.rand(len(shape), generator=gen, dtype=torch.float64).tolist()
        c = C0 + 0.3 * torch.exp(-sum((t - 0.1 * (p - 0.5)) ** 2 for t, p in zip(x, at)) / 0.02)
        a = torch.zeros(shape, dtype=torch.float64, device="cuda")
    else:                                  # Gaussian random field in [0.8, 1.2], about ten points per wavelength
        width, omega = max(8, n // 32) if len(shape) == 2 else max(4, 24 * n // 256), 2.0 * math.pi * n / 10.24
        corr = 20.0 if len(shape) == 2 else 12.0 * n / 256.0
        noise = torch.randn(shape, generator=gen, dtype=torch.float64).to("cuda")
        k2 = sum(_along(torch.fft.fftfreq(m, dtype=torch.float64, device="cuda") ** 2, k, len(shape))
                 for k, m in enumerate(shape))
        g = torch.fft.ifftn(torch.fft.fftn(noise) * torch.exp(-0.5 * (2.0 * math.pi * corr) ** 2 * k2)).real
        c = 0.8 + 0.4 * (g - g.min()) / (g.max() - g.min())
        a = torch.full(shape, 0.05 * omega, dtype=torch.float64, device="cuda")
    e = _edge_cells(shape)
    ramp = 0.5 - 0.5 * torch.cos(math.pi * torch.clamp((e - width) / min(8, max(2, n // 8)), 0.0, 1.0))
    c = torch.where(e < width, torch.full_like(e, C0), C0 + (c - C0) * ramp)
    zeta = torch.where(e < width, ZETA_MAX * (width - e) / width, torch.zeros_like(e))
    return c, a, zeta, omega, 0.05 * omega


def _field(case, shape, seed):
    """The fields an apply or a product takes: dense, of order one, as a Krylov vector."""
    gen = torch.Generator(device="cuda").manual_seed(seed + 1)
    v = torch.randn((case["nrhs"],) + shape + (2,), generator=gen, dtype=torch.float64, device="cuda")
    v = torch.view_as_complex(v)
    v = v if case["precision"] == "fp64" else v.to(torch.complex64)
    return v if case["nrhs"] > 1 else v[0].contiguous()


def _source(shape, seed):
    """A narrow Gaussian source away from the layer."""
    gen = torch.Generator().manual_seed(seed + 2)
    at = (0.5 * torch.rand(len(shape), generator=gen, dtype=torch.float64) - 0.25).tolist()
    d2 = sum(((t - p) * n / 2.0) ** 2 for t, p, n in zip(_axes(shape), at, shape))
    return torch.exp(-0.5 * d2).to(torch.complex128).expand(shape).contiguous()


def _plan(case, shape, seed):
    c, a, zeta, omega, floor = _medium(case, shape, seed)
    host = lambda t: None if t is None else np.ascontiguousarray(t.cpu().numpy())  # noqa: E731
    return binding.Plan(shape, omega, host(c), host(a), host(zeta), c0=C0, m_real=case["m_real"], m_layer=NODES_LAYER,
                        a_floor=floor, precision=case["precision"], max_nrhs=case["nrhs"],
                        interp_order=case["order"], symbol=case["symbol"])


def prepare(case, seed):
    shapes = _shapes(case)
    state = {"op": case["op"], "rtol": case["rtol"]}
    if case["op"] == "serve":
        streams = [torch.cuda.Stream() for _ in range(2)]
        state["members"] = []
        for k, s in enumerate(shapes):
            plan = _plan(case, s, seed + 100 * k)
            state["members"].append((binding.Solver(plan, 1, restart=30, rtol=case["rtol"]),
                                     _source(s, seed + 100 * k), streams[k % 2]))
        return state
    state["plan"] = _plan(case, shapes[0], seed)
    if case["op"] == "solve":
        state["f"] = _source(shapes[0], seed)
    else:
        state["v"] = _field(case, shapes[0], seed)
    return state


def run(state):
    if state["op"] == "apply":
        return state["plan"].apply(state["v"])
    if state["op"] == "matvec":
        return state["plan"].matvec(state["v"])
    if state["op"] == "solve":
        return state["plan"].solve(state["f"], restart=30, rtol=state["rtol"])[0]
    left = []
    for solver, f, stream in state["members"]:
        solver.start(f, stream=stream)
        left.append(solver)
    while left:
        done = binding.advance_group(left, 2)
        left = [s for s, d in zip(left, done) if not d]
    return [solver.result()[0] for solver, _, _ in state["members"]]


# Arnoldi steps a solve to 1e-8 on these media takes, about (for the work of a solve)
SOLVE_STEPS = 40


def work(case):
    size = 16 if case["precision"] == "fp64" else 8
    total = {"bytes": 0.0, "flops": 0.0}
    for shape in _shapes(case):
        pts = float(np.prod(shape))
        layer = case["medium"] != "inclusion"
        k = case["m_real"] + (NODES_LAYER if layer else 0)
        # one apply: the field in and out and the 8-byte interpolation record of each point;
        # 1 + K transforms, K symbol multiplies, two weighted terms
        apply_b = 2.0 * size * pts
        apply_f = pts * ((1 + k) * 5.0 * math.log2(pts) + 6.0 * k + 8.0)
        # one product with P_N: the field in and out and two coefficients of each point
        matvec_b, matvec_f = 2.0 * size * pts, 30.0 * pts
        if case["op"] == "apply":
            total["bytes"] += case["nrhs"] * apply_b + 8.0 * pts
            total["flops"] += case["nrhs"] * apply_f
        elif case["op"] == "matvec":
            total["bytes"] += case["nrhs"] * matvec_b + 2.0 * size * pts
            total["flops"] += case["nrhs"] * matvec_f
        else:
            # each step: an apply, a product, and one read of the basis (15 vectors on average)
            # with the new vector written; 16 operations per point and basis vector
            total["bytes"] += SOLVE_STEPS * (apply_b + matvec_b + (8.0 + 2.0 * size) * pts + 16.0 * 16.0 * pts)
            total["flops"] += SOLVE_STEPS * (apply_f + matvec_f + 15.0 * 32.0 * pts)
    return total


# ---------------------------------------------------------------- in 64 bits, without the library
class _Reference:
    """Q_M and P_N on one medium in plain 64-bit torch: node placement, piecewise weights,
    one forward and K inverse transforms, periodic central differences."""

    def __init__(self, case, shape, seed):
        c, a, zeta, omega, floor = _medium(case, shape, seed)
        self.shape = shape
        layer = zeta is not None and float(zeta.max()) > 0.0
        m, lo, hi = case["m_real"], float(c.min()), float(c.max())
        if layer:       # equidistant on [lo, c0] and on [c0, hi], c0 itself a node
            m = max(m, 3)
            below = min(max(math.ceil((C0 - lo) / (hi - lo) * (m - 1) - 0.5), 1), m - 2)
            if C0 in (lo, hi):
                below = 0 if C0 == lo else m - 1
            nodes = [lo + (C0 - lo) * (i / below) if i < below else C0 for i in range(below + 1)]
            nodes += [C0 + (hi - C0) * (i / (m - 1 - below)) for i in range(1, m - below)]
        else:
            below, nodes = 0, [lo + (hi - lo) / (m - 1) * i for i in range(m - 1)] + [hi]
        cn = torch.tensor(nodes, dtype=torch.float64, device="cuda")
        damp = float(a.reshape(-1)[0])
        gamma = [complex(v, 0.0) for v in nodes]
        ahat = [max(damp, floor)] * m
        self.weight = [torch.zeros(shape, dtype=torch.float64, device="cuda") for _ in range(m)]
        real = torch.ones(shape, dtype=torch.bool, device="cuda") if not layer else zeta <= 0.0
        seg = (torch.searchsorted(cn, c.contiguous(), right=True) - 1).clamp(0, m - 2)
        order = max(1, min(case["order"], m - 1))
        first = seg if order == 1 else (seg - (order - 1) // 2).clamp(0, m - 1 - order)
        for i in range(m):
            inside = real & (first <= i) & (i <= first + order)
            w = torch.ones(shape, dtype=torch.float64, device="cuda")
            for k in range(order + 1):      # Lagrange basis over the nodes first .. first + order
                other = (first + k).clamp(max=m - 1)
                gap = cn[i] - cn[other]
                same = other == i
                w = w * torch.where(same, torch.ones_like(w), (c - cn[other]) / torch.where(same, torch.ones_like(w), gap))
            self.weight[i] = torch.where(inside, w, self.weight[i])
        if layer:
            zmax = float(zeta.max())
            pos = zeta / zmax * NODES_LAYER
            leg = pos.floor().clamp(0, NODES_LAYER - 1)
            t = pos - leg
            self.weight[below] = self.weight[below] + torch.where(~real & (leg == 0), 1.0 - t, torch.zeros_like(t))
            for j in range(1, NODES_LAYER + 1):
                w = torch.where(leg == j - 1, t, torch.where(leg == j, 1.0 - t, torch.zeros_like(t)))
                self.weight.append(torch.where(real, torch.zeros_like(w), w))
                gamma.append(C0 * complex(1.0, -zmax * j / NODES_LAYER))
                ahat.append(damp)       # the damping floor is for nodes of real speed
        lam = 0.0
        for k, n in enumerate(shape):
            f = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device="cuda")
            f = (2.0 * math.pi * f) ** 2 if case["symbol"] == "continuous" else 4.0 * n * n * torch.sin(math.pi * f / n) ** 2
            lam = lam + _along(f, k, len(shape))
        self.lam, self.node = lam, [(complex(omega ** 2, omega * h), g * g) for h, g in zip(ahat, gamma)]
        speed = c.to(torch.complex128) if not layer else c * torch.complex(torch.ones_like(c), -zeta)
        self.g2 = speed * speed
        self.beta = omega ** 2 + 1j * omega * a - 2.0 * self.g2 * sum(float(n) ** 2 for n in shape)

    def apply(self, v):
        spec = torch.fft.fftn(v.to(torch.complex128))
        u = torch.zeros_like(spec)
        for (num, g2), w in zip(self.node, self.weight):
            u += w * torch.fft.ifftn(spec / (num - g2 * self.lam))
        return u

    def matvec(self, u):
        u = u.to(torch.complex128)
        lap = 0.0
        for k, n in enumerate(self.shape):
            lap = lap + (torch.roll(u, 1, k) + torch.roll(u, -1, k)) * float(n) ** 2
        return self.g2 * lap + self.beta * u

    def solve(self, f, tol=1e-13, restart=50, cycles=12):
        """Right-preconditioned GMRES far below the tolerance of the case."""
        x = torch.zeros_like(f)
        size, best = f.numel(), math.inf
        for _ in range(cycles):
            r = f - self.matvec(x)
            beta = float(torch.linalg.norm(r))
            if beta <= tol * float(torch.linalg.norm(f)) or beta > 0.5 * best:
                break
            best = beta
            basis = torch.zeros((restart + 1, size), dtype=torch.complex128, device=f.device)
            basis[0] = r.reshape(-1) / beta
            h = torch.zeros((restart + 1, restart), dtype=torch.complex128)
            for j in range(restart):
                w = self.matvec(self.apply(basis[j].reshape(self.shape))).reshape(-1)
                for _ in range(2):
                    d = basis[: j + 1].conj() @ w
                    w = w - d @ basis[: j + 1]
                    h[: j + 1, j] += d.cpu()
                h[j + 1, j] = torch.linalg.norm(w).cpu()
                basis[j + 1] = w / h[j + 1, j].to(f.device)
            rhs = torch.zeros((restart + 1, 1), dtype=torch.complex128)
            rhs[0] = beta
            y = torch.linalg.lstsq(h, rhs).solution[:, 0].to(f.device)
            x = x + self.apply((y @ basis[:restart]).reshape(self.shape))
        return x


def exact(case, seed):
    shapes = _shapes(case)
    if case["op"] == "serve":
        return [_Reference(case, s, seed + 100 * k).solve(_source(s, seed + 100 * k)) for k, s in enumerate(shapes)]
    ref = _Reference(case, shapes[0], seed)
    if case["op"] == "solve":
        return ref.solve(_source(shapes[0], seed))
    v = _field(case, shapes[0], seed)
    one = ref.apply if case["op"] == "apply" else ref.matvec
    return torch.stack([one(x) for x in v]) if case["nrhs"] > 1 else one(v)
