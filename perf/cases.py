"""The reconstructions whose speed is followed, over the range a user asks for.

A case is one call as a program makes it: a seeded synthetic density (or
particle set) resident on the GPU, a context made once for its grid and
config, and then a whole reconstruction, or a reconstruction and its gradient.
The sizes and amplitudes are those of ``paper_1611_09638_amd/inputs.py``, the
tests and ``bench.py``, and ragged edges (coarsest grid 6, 10 or 12) beside
them.  ``exact`` is the same reconstruction in plain torch, FP64, with every
linear solve carried to rounding by a method of its own.
"""
import math

import torch

from paper_1611_09638_amd import binding

STEPS = 10  # outer steps of a solve (the library's default)


def _case(name, call, n, box, amp, **more):
    c = dict(name=name, call=call, n=n, box=box, amp=amp, coarse_n=8, mixed=False, mass_update=False,
             full_operator=False, tape_fp32=False, tol=1e-10)
    c.update(more)
    return c


def listed():
    return [
        # the smallest workload in use: a coarse particle snapshot, default config
        _case("particles_32", "particles", 32, 250.0, 0.8),
        # a serving loop that may not allocate: small densities, one after the other
        _case("noalloc_64_mixed", "noalloc", 64, 500.0, 1.0, mixed=True),
        # a ragged survey box (coarsest grid 6)
        _case("density_48_ragged", "density", 48, 375.0, 1.0, coarse_n=6),
        # parameter studies on a moderate grid, all in FP64
        _case("density_128", "density", 128, 500.0, 1.5),
        # one step of a gradient-based inference: reconstruction and dL/d(density)
        _case("gradient_64", "gradient", 64, 1000.0, 0.5, tol=1e-12),
        # the same on a larger grid, with the memory-saving options
        _case("gradient_128_mixed", "gradient", 128, 2000.0, 0.5, mixed=True, tape_fp32=True, tol=1e-12),
        # inference on particle positions: deposit at the Lagrangian positions and its reverse mode
        _case("particle_gradient_64", "particle_gradient", 64, 500.0, 0.8, tol=1e-12),
        # the exact-Jacobian operator, where rms(Sigma) has to fall further
        _case("full_operator_128_mixed", "density", 128, 2000.0, 0.5, mixed=True, full_operator=True),
        # the paper's own mass update on a ragged grid
        _case("mass_update_96", "density", 96, 1500.0, 0.5, coarse_n=6, mass_update=True),
        # a catalogue-sized particle run that takes full steps
        _case("particles_256_mixed", "particles", 256, 600.0, 1.5, mixed=True),
        # a strongly nonlinear density, FP64, large ragged grid
        _case("density_320_ragged", "density", 320, 1250.0, 1.5, coarse_n=10),
        # the paper-sized density of the benchmark
        _case("density_512_mixed", "density", 512, 1000.0, 2.0, mixed=True),
    ]


def draw(rng):
    """One more call of the same ranges."""
    call = rng.choice(["density", "density", "particles", "noalloc", "gradient", "particle_gradient"])
    grids = [(24, 6), (32, 8), (40, 10), (48, 6), (48, 12), (56, 14), (64, 8), (80, 10), (96, 6), (96, 12), (112, 14),
             (128, 8), (160, 10), (192, 6), (192, 12), (256, 8), (320, 10), (384, 12)]
    top = {"noalloc": 64, "gradient": 160, "particle_gradient": 128}.get(call, 384)
    n, coarse = rng.choice([g for g in grids if g[0] <= top])
    mixed = rng.random() < 0.5
    mass = call == "density" and n <= 256 and rng.random() < 0.2
    full = call in ("density", "noalloc") and n <= 256 and not mass and rng.random() < 0.2
    if call == "particle_gradient":
        # larger displacements put particles on the kinks of the deposit's weights
        cell, amp = rng.uniform(2.5, 8.0), rng.uniform(0.4, 0.8)
    elif call == "particles":
        cell, amp = rng.uniform(2.5, 8.0), rng.uniform(0.6, 1.4)
    elif mass or full or call == "gradient":
        cell, amp = rng.uniform(12.0, 16.0), rng.uniform(0.3, 0.5)
    else:
        cell, amp = rng.uniform(3.0, 10.0), rng.uniform(0.5, 1.5)
    return dict(call=call, n=n, box=round(cell * n, 1), amp=round(amp, 2), coarse_n=coarse, mixed=mixed,
                mass_update=mass, full_operator=full, tape_fp32=call == "gradient" and mixed,
                tol=1e-12 if "gradient" in call else 1e-10)


# ------------------------------------------------------------------- inputs


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _modes(n, box, device):
    k = 2.0 * math.pi * torch.fft.fftfreq(n, d=box / n, dtype=torch.float64, device=device)
    kz = 2.0 * math.pi * torch.fft.rfftfreq(n, d=box / n, dtype=torch.float64, device=device)
    return k[:, None, None], k[None, :, None], kz[None, None, :]


def _gaussian_modes(n, box, seed, device):
    """Fourier modes of a Gaussian field with P(k) ~ k / (1 + (k/0.02)^2)^2."""
    gen = torch.Generator(device=device)
    gen.manual_seed(seed)
    gk = torch.fft.rfftn(torch.randn((n, n, n), generator=gen, dtype=torch.float64, device=device))
    kx, ky, kz = _modes(n, box, device)
    k = torch.sqrt(kx ** 2 + ky ** 2 + kz ** 2)
    gk *= torch.sqrt(k) / (1.0 + (k / 0.02) ** 2)
    return gk


def _density(case, seed):
    n = case["n"]
    g = torch.fft.irfftn(_gaussian_modes(n, case["box"], seed, _device()), s=(n, n, n))
    g -= g.mean()
    g *= case["amp"] / g.std(correction=0)
    rho = torch.exp_(g)
    return (rho / rho.mean()).contiguous()


def _particles(case, seed):
    """n^3 lattice particles with a Zel'dovich displacement of `amp` cells rms, float32 in [0, box)."""
    n, box, device = case["n"], case["box"], _device()
    gk = _gaussian_modes(n, box, seed, device)
    ks = _modes(n, box, device)
    k2 = ks[0] ** 2 + ks[1] ** 2 + ks[2] ** 2
    k2[0, 0, 0] = 1.0
    psi = torch.stack([torch.fft.irfftn(1j * ka / k2 * gk, s=(n, n, n)) for ka in ks], dim=-1)
    psi *= case["amp"] / torch.sqrt((psi ** 2).sum(-1).mean())
    q = torch.arange(n, dtype=torch.float64, device=device)
    psi += torch.stack(torch.meshgrid(q, q, q, indexing="ij"), dim=-1)
    pos = torch.remainder(psi * (box / n), box).reshape(-1, 3).float()
    pos[pos >= torch.tensor(box, dtype=torch.float32)] = 0.0
    return pos.contiguous()


def _cotangent(case, seed):
    """dL/d(delta_r) of a smooth-weighted loss: white noise with its large scales raised."""
    n = case["n"]
    gk = _gaussian_modes(n, case["box"], seed + 7919, _device())
    g = torch.fft.irfftn(gk, s=(n, n, n))
    return (g / g.std()).contiguous()


def _config(case):
    return binding.Config(
        max_outer=STEPS, coarse_n=case["coarse_n"], tol=case["tol"],
        precision=binding.MIXED if case["mixed"] else binding.FP64, mass_update=int(case["mass_update"]),
        full_operator=int(case["full_operator"]), particle_deposit=int(case["call"] == "particle_gradient"),
        record_tape=int("gradient" in case["call"]), tape_fp32=int(case["tape_fp32"]))


def prepare(case, seed):
    cfg = _config(case)
    state = dict(call=case["call"], box=case["box"], cfg=cfg)
    if case["call"] in ("particles", "particle_gradient"):
        state["x"] = _particles(case, seed)
    else:
        state["x"] = _density(case, seed)
    if "gradient" in case["call"]:
        state["x"].requires_grad_(True)
        state["g"] = _cotangent(case, seed)
    if case["call"] == "noalloc":
        # outputs that the serving loop owns
        state["phi"] = torch.empty_like(state["x"])
        state["delta"] = torch.empty_like(state["x"])
    else:
        state["rec"] = binding.Recon(case["n"], cfg)
    return state


def run(state):
    call, x, box = state["call"], state["x"], state["box"]
    if call == "noalloc":
        phi, delta, st = binding.solve_noalloc(x, box, state["cfg"], phi=state["phi"], delta=state["delta"])
    elif call == "density":
        phi, delta, st = state["rec"].solve(x, box)
    elif call == "particles":
        phi, delta, st = state["rec"].solve_particles(x, box)
    else:
        fn = binding.Reconstruct if call == "gradient" else binding.ReconstructParticles
        delta, phi = fn.apply(x, state["rec"], box)
        (grad,) = torch.autograd.grad(delta, x, state["g"])
        st = state["rec"].last_stats
        return dict(phi=phi.detach(), delta=delta.detach(), grad=grad, alpha=st["alpha"], rms_sigma=st["rms_sigma"])
    return dict(phi=phi, delta=delta, alpha=st["alpha"], rms_sigma=st["rms_sigma"])


def work(case):
    """Inputs read and outputs written once.  Operations per node: in each
    outer step the mass, source, smoothing and step test (about 250), and a
    linear solve of one V(2,2) cycle (four sweeps, residual and transfers on
    levels that add a seventh) and one conjugate-gradient step per decade of
    its tolerance; a gradient reads and solves once more per step."""
    n3 = case["n"] ** 3
    particles = case["call"] in ("particles", "particle_gradient")
    grad = "gradient" in case["call"]
    cycles = -math.log10(case["tol"])
    solve = cycles * (4 * 26 + 40) * 8 / 7 + cycles * (110 if case["full_operator"] else 35)
    flops = n3 * STEPS * (250 + solve) * (2 if grad else 1)
    nbytes = n3 * ((12 if particles else 8) + 16)
    if grad:
        nbytes += n3 * (8 + (12 if particles else 8))
    return dict(bytes=nbytes, flops=flops)


# ---------------------------------------------------- the 64-bit reference


def _at(f, *d):
    """f at the node shifted by d = (di, dj, dk), periodic."""
    ax = [a for a in range(3) if d[a]]
    return torch.roll(f, [-d[a] for a in ax], ax) if ax else f


def _unit(a, s=1):
    d = [0, 0, 0]
    d[a] = s
    return d


def _both(a, b, sa, sb):
    d = [0, 0, 0]
    d[a], d[b] = sa, sb
    return d


PAIRS = ((0, 1), (0, 2), (1, 2))


def _triad(phi):
    """I + compact Hessian: (xx, yy, zz, xy, xz, yz)."""
    e = [1.0 + _at(phi, *_unit(a)) - 2.0 * phi + _at(phi, *_unit(a, -1)) for a in range(3)]
    for a, b in PAIRS:
        e.append(0.25 * (_at(phi, *_both(a, b, 1, 1)) - _at(phi, *_both(a, b, 1, -1)) -
                         _at(phi, *_both(a, b, -1, 1)) + _at(phi, *_both(a, b, -1, -1))))
    return e


def _det(e):
    xx, yy, zz, xy, xz, yz = e
    return xx * (yy * zz - yz * yz) - xy * (xy * zz - yz * xz) + xz * (xy * yz - yy * xz)


def _smooth(f, c0=0.5):
    nb = sum(_at(f, *_unit(a, s)) for a in range(3) for s in (1, -1))
    return c0 * f + (1.0 - c0) / 6.0 * nb


def _cells(x, n):
    """Lower corner (as a long index) and offset of positions x (..., 3) in cells."""
    lo = torch.floor(x.detach())
    return lo.long() % n, x - lo


def _corners(lo, w, n):
    for c in range(8):
        o = ((c >> 2) & 1, (c >> 1) & 1, c & 1)
        idx = 0
        for a in range(3):
            idx = idx * n + (lo[..., a] + o[a]) % n
        yield o, idx, math.prod((w[..., a] if o[a] else 1.0 - w[..., a]) for a in range(3))


def _deposit(x, n, weight):
    lo, w = _cells(x, n)
    rho = torch.zeros(n ** 3, dtype=torch.float64, device=x.device)
    for _, idx, wt in _corners(lo, w, n):
        rho = rho.index_add(0, idx.reshape(-1), (wt * weight).reshape(-1))
    return rho.reshape(n, n, n)


def _shifts(phi):
    return torch.stack([0.5 * (_at(phi, *_unit(a)) - _at(phi, *_unit(a, -1))) for a in range(3)], -1)


def _interp(f, x, n):
    lo, w = _cells(x, n)
    f = f.reshape(n ** 3, -1)
    return sum(wt[..., None] * f[idx] for _, idx, wt in _corners(lo, w, n))


def _jacobian(s, x, n):
    lo, w = _cells(x, n)
    s = s.reshape(n ** 3, 3)
    J = torch.eye(3, dtype=torch.float64, device=x.device).repeat(x.shape[0], 1, 1)
    for o, idx, _ in _corners(lo, w, n):
        for b in range(3):
            g = 1.0 if o[b] else -1.0
            for a in range(3):
                if a != b:
                    g = g * (w[..., a] if o[a] else 1.0 - w[..., a])
            J[:, :, b] += s[idx] * g[:, None]
    return J


def _invert(phi, y, n):
    """xi with xi + trilinear(D_c phi)(xi) = y, by damped Newton; differentiable in phi and y."""
    s = _shifts(phi)

    def off(x, s, y):
        r = x + _interp(s, x, n) - y
        return r - n * torch.round(r.detach() / n)
    sd, yd = s.detach(), y.detach()
    xi = yd.clone()
    r = off(xi, sd, yd)
    for _ in range(100):
        norm = r.abs().amax(1)
        if float(norm.max()) < 1e-13:
            break
        step = torch.linalg.solve(_jacobian(sd, xi, n), r)
        t = torch.ones_like(norm)
        best, rb = xi - step, off(xi - step, sd, yd)
        for _ in range(30):
            bad = (rb.abs().amax(1) >= norm) & (norm > 1e-13)
            if not bool(bad.any()):
                break
            t = torch.where(bad, 0.5 * t, t)
            best = xi - t[:, None] * step
            rb = off(best, sd, yd)
        xi = torch.remainder(best, n)
        r = off(xi, sd, yd)
    return xi - torch.linalg.solve(_jacobian(sd, xi, n), off(xi, s, y))


def _apply(a, u, a_min=1e-3):
    out = 0.0
    for ax in range(3):
        c = torch.clamp(0.5 * (a + _at(a, *_unit(ax))), min=a_min)
        f = c * (_at(u, *_unit(ax)) - u)
        out = out + f - _at(f, *_unit(ax, -1))
    return out


def _tensor(phi, M):
    xx, yy, zz, xy, xz, yz = e = _triad(phi)
    w = M / _det(e)
    return [w * (yy * zz - yz * yz), w * (xx * zz - xz * xz), w * (xx * yy - xy * xy),
            w * (xz * yz - xy * zz), w * (xy * yz - xz * yy), w * (xy * xz - xx * yz)]


def _apply_full(K, u, a_min):
    out = 0.0
    for ax in range(3):
        c = 0.5 * (K[ax] + _at(K[ax], *_unit(ax)))
        f = (torch.clamp(c, min=a_min) if a_min else c) * (_at(u, *_unit(ax)) - u)
        out = out + f - _at(f, *_unit(ax, -1))
    for q, pair in enumerate(PAIRS):
        for mu, nu in (pair, pair[::-1]):
            f = K[3 + q] * (_at(u, *_unit(nu)) - _at(u, *_unit(nu, -1)))
            out = out + 0.25 * (_at(f, *_unit(mu)) - _at(f, *_unit(mu, -1)))
    return out


def _pcg(op, a, b, most=5000):
    """op u = b, mean-free: conjugate gradients with the FFT inverse of the unit
    Laplacian between two scalings by a^(-1/2); restarted on its true residual."""
    n = b.shape[0]
    k = 2.0 * math.pi * torch.fft.fftfreq(n, dtype=torch.float64, device=b.device)
    lam = 2.0 * torch.cos(k) - 2.0
    sym = lam[:, None, None] + lam[None, :, None] + lam[None, None, : n // 2 + 1]
    sym[0, 0, 0] = 1.0
    root = torch.rsqrt(torch.clamp(a, min=1e-3))

    def pre(r):
        zk = torch.fft.rfftn(root * r) / sym
        zk[0, 0, 0] = 0.0
        return root * torch.fft.irfftn(zk, s=(n, n, n))
    b = b - b.mean()
    u, target = torch.zeros_like(b), 1e-13 * float(b.norm())
    r = b
    for _ in range(4):
        if float(r.norm()) <= target:
            break
        z = pre(r)
        p, rz, drop = z, (r * z).sum(), 1e-9 * float(r.norm())
        for it in range(most):
            q = op(p)
            step = rz / (p * q).sum()
            u = u + step * p
            r = r - step * q
            if it % 10 == 9 and float(r.norm()) <= max(drop, 0.3 * target):
                break
            z = pre(r)
            rz, old = (r * z).sum(), rz
            p = z + (rz / old) * p
        r = b - op(u)
        r = r - r.mean()
    return u - u.mean()


class _Solve(torch.autograd.Function):
    """u = A(a)^+ b, differentiated as exact."""

    @staticmethod
    def forward(ctx, a, b):
        u = _pcg(lambda v: _apply(a, v), a, b)
        ctx.save_for_backward(a, u)
        return u

    @staticmethod
    def backward(ctx, g):
        a, u = ctx.saved_tensors
        lam = _pcg(lambda v: _apply(a, v), a, g)
        with torch.enable_grad():
            ad = a.detach().requires_grad_(True)
            (ga,) = torch.autograd.grad(_apply(ad, u), ad, -lam)
        return ga, lam


def _positive(e):
    return bool(((e[0] > 0) & (e[0] * e[1] - e[3] * e[3] > 0) & (_det(e) > 0)).all())


def _compression(e, xi_m=0.1):
    """4 max(0, xi_m / lambda_0 - 1)^2, zero where e - xi_m I is positive definite."""
    d = [e[0] - xi_m, e[1] - xi_m, e[2] - xi_m, e[3], e[4], e[5]]
    at = ~((d[0] > 0) & (d[0] * d[1] - d[3] * d[3] > 0) & (_det(d) > 0))
    if not bool(at.any()):
        return torch.zeros_like(e[0])
    xx, yy, zz, xy, xz, yz = [v[at] for v in e]
    mat = torch.stack([xx, xy, xz, xy, yy, yz, xz, yz, zz], -1).reshape(-1, 3, 3)
    lam = torch.linalg.eigvalsh(mat.cpu())[:, 0].to(mat.device)
    full = torch.zeros_like(e[0])
    return full.masked_scatter(at, 4.0 * torch.clamp(xi_m / lam - 1.0, min=0.0) ** 2)


def exact(case, seed):
    if case["n"] > 64:
        return None  # over the time that a reference may take
    n, box = case["n"], case["box"]
    deposit = case["call"] == "particle_gradient"
    particles = case["call"] in ("particles", "particle_gradient")
    grad = "gradient" in case["call"]
    x = (_particles if particles else _density)(case, seed).double()
    x.requires_grad_(grad)
    with torch.set_grad_enabled(grad):
        y = x * (n / box)
        rho = x if not particles else _deposit(y.detach(), n, torch.ones((), dtype=torch.float64, device=x.device))
        m = rho / rho.mean()
        phi = torch.zeros((n, n, n), dtype=torch.float64, device=x.device)
        base = torch.stack(torch.meshgrid(*[torch.arange(n, dtype=torch.float64, device=x.device)] * 3,
                                          indexing="ij"), -1)
        alphas, rms, M = [], [], None
        for it in range(STEPS + 1):
            e = _triad(phi)
            det = _det(e)
            if deposit:
                M = _deposit(_invert(phi, y, n), n, n ** 3 / y.shape[0])
            elif M is None or not case["mass_update"]:
                M = det * _interp(m, base + _shifts(phi), n)[..., 0]
            sigma = M.mean() - M
            rms.append(float(torch.sqrt((sigma.detach() ** 2).mean())))
            if it == STEPS:
                break
            t = sigma + _compression(e) - 2.0 * (det > 10.0) * sigma.abs()
            b = _smooth(t) - t.mean()
            if case["full_operator"]:
                K = _tensor(phi, M)
                u = _pcg(lambda v: _apply_full(K, v, 1e-3), (K[0] + K[1] + K[2]) / 3.0, b)
            else:
                u = _Solve.apply(M, b)
            dphi = _smooth(u)
            D = _apply_full(_tensor(phi, M), dphi, 0.0) if case["mass_update"] else None
            shift = float(_shifts(dphi.detach()).abs().max())
            for j in range(31):
                alpha = 2.0 ** -j
                if alpha * shift <= 1.0 and _positive(_triad((phi + alpha * dphi).detach())) and (
                        D is None or bool((M + alpha * D > 0).all())):
                    break
            alphas.append(alpha)
            phi = phi + alpha * dphi
            if D is not None:
                M = M + alpha * D
        delta = 3.0 - sum(_triad(phi)[:3])
        out = dict(phi=(phi * (box / n) ** 2).detach(), delta=delta.detach(), alpha=alphas, rms_sigma=rms)
        if grad:
            (out["grad"],) = torch.autograd.grad(delta, x, _cotangent(case, seed))
    return out
