"""The small levels of the V-cycle (one workgroup from 16^3 down) against the
FP64 oracle, on every chain of edges that it has an instance for and on
hierarchies that enter it from a larger level."""
import numpy as np
import pytest

import oracle as orc

pytestmark = pytest.mark.gpu

# (edge, coarsest edge, pre-sweeps, post-sweeps)
CYCLES = [(2, 2, 2, 2), (4, 4, 2, 2), (4, 2, 2, 2), (6, 6, 2, 2), (8, 8, 2, 2), (8, 4, 2, 2), (8, 2, 2, 2),
          (10, 10, 2, 2), (12, 12, 2, 2), (12, 6, 2, 2), (14, 14, 2, 2), (16, 16, 2, 2), (16, 8, 2, 2),
          (16, 4, 2, 2), (16, 2, 2, 2), (16, 8, 1, 3), (16, 8, 0, 1), (16, 8, 2, 0), (20, 10, 2, 2), (24, 6, 2, 2),
          (24, 12, 2, 2), (28, 14, 2, 2), (32, 16, 2, 2), (32, 4, 1, 1), (40, 10, 2, 2), (128, 8, 2, 2)]


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("pairs", [64, 3, 0])
@pytest.mark.parametrize("n,cn,pre,post", CYCLES)
def test_small_cycle_against_oracle(torch_cuda, n, cn, pre, post, pairs):
    """FP64 to 1e-12 (the oracle's own rounding over the cycle); FP32 to 1e-4:
    the cycle applies about 130 relaxations, each with a relative rounding of
    a few 6e-8, to a field whose smooth part the coarsest level has scaled up
    by less than 100."""
    torch = torch_cuda
    from paper_1611_09638_amd import binding
    if pairs != 64 and n > 40:
        pytest.skip("the count of coarsest sweeps is covered by the smaller grids")
    rng = np.random.default_rng(500 + n + cn)
    a = np.exp(1.5 * rng.normal(size=(n, n, n)))
    r = rng.normal(size=(n, n, n))
    r -= r.mean()
    kw = dict(coarse_n=cn, n_pre=pre, n_post=post, coarse_sweeps=pairs)
    z = orc.vcycle(a, r, orc.Config(**kw))
    rec = binding.Recon(n, binding.Config(precision=binding.MIXED, **kw))
    g = rec.vcycle(torch.from_numpy(a).cuda(), torch.from_numpy(r).cuda()).cpu().numpy()
    assert rel(g, z) < 1e-12
    g = rec.vcycle(torch.from_numpy(a).float().cuda(), torch.from_numpy(r).float().cuda()).double().cpu().numpy()
    assert rel(g, z) < 1e-4


@pytest.mark.parametrize("n,cn,dtype", [(20, 10, 64), (20, 10, 32), (24, 6, 64), (28, 14, 32), (32, 8, 64), (32, 8, 32),
                                        (40, 10, 64), (48, 6, 64), (56, 14, 32), (64, 8, 64), (64, 8, 32), (80, 10, 32)])
def test_tiles_equal_the_separate_kernels(torch_cuda, n, cn, dtype):
    """A V-cycle whose finest level runs in two tile launches, against the
    same cycle from the sweep, residual, restriction and prolongation kernels
    of the stage calls around the V-cycle of the next level: bit for bit (the
    level scale 1/4 is a power of two)."""
    torch = torch_cuda
    from paper_1611_09638_amd import binding
    rng = np.random.default_rng(900 + n)
    t = torch.float64 if dtype == 64 else torch.float32
    a = torch.from_numpy(np.exp(2.0 * rng.normal(size=(n, n, n)))).cuda().to(t)
    r = torch.from_numpy(rng.normal(size=(n, n, n))).cuda().to(t)
    cfg = binding.Config(coarse_n=cn, precision=binding.MIXED)
    rec = binding.Recon(n, cfg)
    z = rec.vcycle(a, r)
    u = torch.zeros_like(r)
    for _ in range(2):
        u = rec.rbgs(u, a, r, first=0, variant=1)
    c = rec.residual_restrict(u, a, r, variant=1)
    e = binding.Recon(n // 2, cfg).vcycle(rec.restrict(a, variant=1), 4.0 * c)
    u = rec.prolong_add(u, e, variant=1)
    for _ in range(2):
        u = rec.rbgs(u, a, r, first=1, variant=1)
    assert torch.equal(z, u)


@pytest.mark.parametrize("n,cn,dtype", [(10, 10, 64), (16, 8, 64), (16, 8, 32), (48, 6, 64), (64, 8, 32), (96, 6, 64),
                                        (112, 14, 64)])
def test_krylov_steps_on_small_grids(torch_cuda, n, cn, dtype):
    """The conjugate-gradient loop at the edges of the grids whose consumers
    fold the partial sums (10^3 and 96^3; 112^3 folds them in a launch): a
    fixed number of steps against the oracle's solution at the same tolerance,
    to the conditioning of the input times the solve's tolerance (contrast
    below 100, tol 1e-12)."""
    torch = torch_cuda
    from paper_1611_09638_amd import binding
    rng = np.random.default_rng(1200 + n)
    a = np.exp(0.7 * rng.normal(size=(n, n, n)))
    b = rng.normal(size=(n, n, n))
    b -= b.mean()
    u, cycles, _ = orc.mg_solve(a, b, orc.Config(coarse_n=cn, tol=1e-12))
    rec = binding.Recon(n, binding.Config(coarse_n=cn, precision=binding.FP64 if dtype == 64 else binding.MIXED))
    g, cyc, res = rec.mg_solve(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), tol=1e-12)
    assert res <= 1e-12
    assert rel(g.cpu().numpy(), u) < 1e-9
    if dtype == 64:
        assert cyc == cycles


@pytest.mark.parametrize("n,cn,dtype", [(192, 6, 64), (320, 10, 64), (320, 10, 32), (384, 12, 64), (384, 12, 32)])
def test_sweeps_on_ragged_edges(torch_cuda, n, cn, dtype):
    """The fused sweep at the edges whose chunk length or tile is not that of a
    power of two: every kind (from zero, plain, with the coarse correction)
    equals the per-colour kernels bit for bit."""
    torch = torch_cuda
    from paper_1611_09638_amd import binding
    t = torch.float64 if dtype == 64 else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(n)
    u, a, b = (torch.randn((n, n, n), generator=gen, device="cuda", dtype=t) for _ in range(3))
    a = torch.exp(a)
    e = torch.randn((n // 2,) * 3, generator=gen, device="cuda", dtype=t)
    rec = binding.Recon(n, binding.Config(coarse_n=cn, precision=binding.MIXED))
    for first in (0, 1):
        for x in (u, torch.zeros_like(u)):
            assert torch.equal(rec.rbgs(x, a, b, first=first, variant=2), rec.rbgs(x, a, b, first=first, variant=1))
    want = rec.rbgs(rec.prolong_add(u, e, variant=1), a, b, first=1, variant=1)
    assert torch.equal(rec.prolong_sweep(u, e, a, b, first=1, variant=2), want)


@pytest.mark.parametrize("n,cn,mixed", [(128, 8, False), (192, 12, True), (320, 10, False)])
def test_grouped_direction_sums_like_the_gather(torch_cuda, n, cn, mixed):
    """The streamed direction of edges that are multiples of 64 leaves the
    gather kernels' partial sums, so one conjugate-gradient step (one V-cycle,
    alpha = z.r / p.q) equals the step formed from the stage calls to FP64
    rounding of the final update alone."""
    torch = torch_cuda
    from paper_1611_09638_amd import binding
    gen = torch.Generator(device="cuda").manual_seed(n + 1)
    a = torch.exp(torch.randn((n, n, n), generator=gen, device="cuda", dtype=torch.float64))
    b = torch.randn((n, n, n), generator=gen, device="cuda", dtype=torch.float64)
    b -= b.mean()
    cfg = binding.Config(coarse_n=cn, precision=binding.MIXED if mixed else binding.FP64, fixed_cycles=2)
    rec = binding.Recon(n, cfg)
    u, cycles, _ = rec.mg_solve(a, b)
    assert cycles == 2
    # one V-cycle on the solve's own hierarchy (in mixed mode the FP64 one,
    # rounded): the plain iteration's first step from zero, less its mean, which
    # neither the operator nor a product with a mean-free field sees
    one = binding.Recon(n, binding.Config(coarse_n=cn, precision=cfg.precision, solver=binding.SOLVER_VCYCLE,
                                          fixed_cycles=1))
    r, want, p, q, alpha, rz = b.clone(), torch.zeros_like(b), None, None, 0.0, 0.0
    for step in range(2):
        z, _, _ = one.mg_solve(a, r)
        old, rz = rz, float((z * r).sum())
        beta = 0.0 if step == 0 else -alpha * float((z * q).sum()) / old
        p, q, pq = rec.direction(z, p, a, beta, first=step == 0, variant=1)
        alpha = rz / pq
        want += alpha * p
        r -= alpha * q
    want -= want.mean()
    # the stage steps' sums (torch's) differ from the loop's by about n^1.5 ulp
    assert float((u - want).norm() / want.norm()) < 1e-11


@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("n,cn,mixed", [(128, 8, False), (128, 8, True), (256, 16, False), (256, 16, True)])
def test_deferred_solution_updates(torch_cuda, n, cn, mixed, steps):
    """Solution updates applied two steps (FP64 directions) or three steps
    (FP32 directions, 256^3 mixed) at a time, for every count left due when the
    loop ends: u against the sum of alpha p of a loop made of stage calls.  The
    k-th update is about 0.2^k of u, the fifth 3e-4; the loops differ by the
    rounding of their sums (1e-14) in FP64, and in mixed mode by the rounding
    of z and p to FP32 (1e-7 a step) after the mean that only one of them has
    taken off."""
    torch = torch_cuda
    from paper_1611_09638_amd import binding
    gen = torch.Generator(device="cuda").manual_seed(n + 7)
    a = torch.exp(torch.randn((n, n, n), generator=gen, device="cuda", dtype=torch.float64))
    b = torch.randn((n, n, n), generator=gen, device="cuda", dtype=torch.float64)
    b -= b.mean()
    kw = dict(coarse_n=cn, precision=binding.MIXED if mixed else binding.FP64)
    u, cycles, _ = binding.Recon(n, binding.Config(fixed_cycles=steps, **kw)).mg_solve(a, b)
    assert cycles == steps
    one = binding.Recon(n, binding.Config(solver=binding.SOLVER_VCYCLE, fixed_cycles=1, **kw))
    r, want, p, q, alpha, rz = b.clone(), torch.zeros_like(b), None, None, 0.0, 0.0
    for step in range(steps):
        z, _, _ = one.mg_solve(a, r)
        old, rz = rz, float((z * r).sum())
        p = z if step == 0 else z - alpha * float((z * q).sum()) / old * p
        if mixed and n == 256:
            p = p.float().double()
        _, q, pq = one.direction(p, None, a, 0.0, first=True, variant=1)
        alpha = rz / pq
        want += alpha * p
        r -= alpha * q
    want -= want.mean()
    assert float((u - want).norm() / want.norm()) < (1e-5 if mixed else 1e-10)


@pytest.mark.parametrize("steps", [1, 3, 4])
@pytest.mark.parametrize("n,cn,mixed", [(128, 8, False), (192, 12, True), (256, 16, False), (256, 16, True)])
def test_streamed_full_operator_steps(torch_cuda, n, cn, mixed, steps):
    """The exact-Jacobian loop with the streamed direction (128^3 and 192^3
    with the gather launches' partial sums) and its deferred solution updates,
    against a loop of stage calls; bounds as for the x ~ xi loop."""
    torch = torch_cuda
    from paper_1611_09638_amd import binding
    gen = torch.Generator(device="cuda").manual_seed(n + 11)
    a = torch.exp(0.5 * torch.randn((n, n, n), generator=gen, device="cuda", dtype=torch.float64))
    phi = 0.02 * torch.randn((n, n, n), generator=gen, device="cuda", dtype=torch.float64)
    b = torch.randn((n, n, n), generator=gen, device="cuda", dtype=torch.float64)
    b -= b.mean()
    kw = dict(coarse_n=cn, full_operator=1, precision=binding.MIXED if mixed else binding.FP64)
    rec = binding.Recon(n, binding.Config(fixed_cycles=steps, **kw))
    u, cycles, _ = rec.mg_solve_full(a, phi, b)
    assert cycles == steps
    one = binding.Recon(n, binding.Config(solver=binding.SOLVER_VCYCLE, fixed_cycles=1, **kw))
    r, want, p, q, alpha, rz = b.clone(), torch.zeros_like(b), None, None, 0.0, 0.0
    for step in range(steps):
        z, _, _ = one.mg_solve_full(a, phi, r)
        old, rz = rz, float((z * r).sum())
        p = z if step == 0 else z - alpha * float((z * q).sum()) / old * p
        if mixed and n == 256:
            p = p.float().double()
        _, q, pq = one.full_direction(phi, a, p, None, 0.0, first=True, variant=1)
        alpha = rz / pq
        want += alpha * p
        r -= alpha * q
    want -= want.mean()
    assert float((u - want).norm() / want.norm()) < (1e-5 if mixed else 1e-10)


@pytest.mark.parametrize("n,cn,sigma", [(10, 10, 2.0), (80, 10, 1.5), (96, 6, 2.0)])
def test_gradient_with_combined_deposits(torch_cuda, n, cn, sigma):
    """The transposed deposit where sums pass between lanes and planes before
    they become atomics: several rows in a wave (10), two and more planes a
    thread, rows that end inside a wave (80, 96) and meshes that move by more
    than a cell, against the oracle, to the bound of the smaller grids."""
    torch = torch_cuda
    from paper_1611_09638_amd import binding, inputs
    box = 15.6 * n
    rho = inputs.lognormal_density(n, box, sigma, n)
    base = dict(max_outer=2, tol=1e-13, max_vcycles=300, coarse_n=cn)
    gd = np.random.default_rng(n).normal(size=rho.shape)
    orc.solve(rho, box, orc.Config(record_tape=1, **base))
    want = orc.backward(gd, None, box, orc.Config(**base))
    rec = binding.Recon(n, binding.Config(record_tape=1, **base))
    rec.solve(torch.from_numpy(rho).cuda(), box)
    assert rel(rec.backward(torch.from_numpy(gd).cuda()).cpu().numpy(), want) < 1e-8


@pytest.mark.parametrize("n,cn,mixed", [(128, 8, False), (192, 12, True), (320, 10, False)])
def test_streamed_residual_norm(torch_cuda, n, cn, mixed):
    """The streamed residual with the gather launch's partial sums: the norm
    that a solve reports against that of the residual from the stage call, to
    the rounding of n^3 summands (n^1.5 ulp), and the plain V-cycle iteration,
    whose steps start from it, against the same iteration made of one-cycle
    solves of the residual equation (the FP64 corrections round alike; in mixed
    mode z and its mean are rounded to FP32 around different means)."""
    torch = torch_cuda
    from paper_1611_09638_amd import binding
    gen = torch.Generator(device="cuda").manual_seed(n + 3)
    a = torch.exp(torch.randn((n, n, n), generator=gen, device="cuda", dtype=torch.float64))
    b = torch.randn((n, n, n), generator=gen, device="cuda", dtype=torch.float64)
    b -= b.mean()
    kw = dict(coarse_n=cn, precision=binding.MIXED if mixed else binding.FP64, solver=binding.SOLVER_VCYCLE)
    rec = binding.Recon(n, binding.Config(fixed_cycles=3, **kw))
    u, _, res = rec.mg_solve(a, b)
    one = binding.Recon(n, binding.Config(fixed_cycles=1, **kw))
    want, r = torch.zeros_like(b), b
    for _ in range(3):
        want += one.mg_solve(a, r)[0]
        r = rec.residual(want, a, b, variant=1)
    assert float((u - want).norm() / want.norm()) < (1e-5 if mixed else 1e-11)
    true = rec.residual(u, a, b, variant=1)
    assert abs(res - float(true.norm() / b.norm())) <= 1e-11 * res


@pytest.mark.parametrize("dtype", [64, 32])
@pytest.mark.parametrize("n,cn", [(160, 10), (224, 14)])
def test_coarse_right_hand_side_on_narrow_tiles(torch_cuda, n, cn, dtype):
    """The fused residual and restriction on edges that are odd multiples of
    32, against the two kernels that it replaces: bit for bit."""
    torch = torch_cuda
    from paper_1611_09638_amd import binding
    t = torch.float64 if dtype == 64 else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(n + 5)
    u, a, b = (torch.randn((n, n, n), generator=gen, device="cuda", dtype=t) for _ in range(3))
    rec = binding.Recon(n, binding.Config(coarse_n=cn, precision=binding.MIXED))
    assert torch.equal(rec.residual_restrict(u, torch.exp(a), b), rec.residual_restrict(u, torch.exp(a), b, variant=1))


@pytest.mark.parametrize("n,cn,dtype", [(320, 10, 32), (448, 14, 32), (384, 12, 32), (320, 10, 64), (448, 14, 64)])
def test_large_ragged_vcycle_equals_the_separate_kernels(torch_cuda, n, cn, dtype):
    """A V-cycle on the edges from 256 whose fused sweeps are in tiles of 64 (in
    FP32 odd multiples of 64) or in chunks that no power of two has, with the
    sweep that starts from u = 0, which no stage call reaches: bit for bit the
    cycle made of per-colour sweeps and single transfers around the V-cycle of
    the next level."""
    torch = torch_cuda
    from paper_1611_09638_amd import binding
    t = torch.float64 if dtype == 64 else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(n + 13)
    a = torch.exp(torch.randn((n, n, n), generator=gen, device="cuda", dtype=t))
    r = torch.randn((n, n, n), generator=gen, device="cuda", dtype=t)
    cfg = binding.Config(coarse_n=cn, precision=binding.MIXED)
    rec = binding.Recon(n, cfg)
    z = rec.vcycle(a, r)
    u = torch.zeros_like(r)
    for _ in range(2):
        u = rec.rbgs(u, a, r, first=0, variant=1)
    c = rec.residual_restrict(u, a, r, variant=1)
    e = binding.Recon(n // 2, cfg).vcycle(rec.restrict(a, variant=1), 4.0 * c)
    u = rec.prolong_add(u, e, variant=1)
    for _ in range(2):
        u = rec.rbgs(u, a, r, first=1, variant=1)
    assert torch.equal(z, u)


@pytest.mark.parametrize("n,cn", [(320, 10), (448, 14)])
def test_mixed_solve_on_large_ragged_edges(torch_cuda, n, cn):
    """The mixed solve at those edges reaches its tolerance, with the residual
    taken by the gather kernel (twice the tolerance: the loop stops on its
    recurrence, whose drift is a few 1e-13 at this contrast)."""
    torch = torch_cuda
    from paper_1611_09638_amd import binding
    gen = torch.Generator(device="cuda").manual_seed(n + 17)
    a = torch.exp(torch.randn((n, n, n), generator=gen, device="cuda", dtype=torch.float64))
    b = torch.randn((n, n, n), generator=gen, device="cuda", dtype=torch.float64)
    b -= b.mean()
    rec = binding.Recon(n, binding.Config(coarse_n=cn, precision=binding.MIXED))
    u, _, _ = rec.mg_solve(a, b, tol=1e-10)
    assert float(rec.residual(u, a, b, variant=1).norm() / b.norm()) < 2e-10
