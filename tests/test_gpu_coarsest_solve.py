"""The coarsest level's direct solve in the persistent kernel, 7 x 7, 3 x 3 and 1 x 1, against the oracle
bit for bit (FP32 cycles: its emulation), whatever the levels above and the relaxation.  The substitution
runs in one order everywhere, so the tolerance is 0."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("specs,prec,smoother,ex", [
    ([(7, 0.3, 1e-2, 7)], "f64", "jacobi", {}), ([(15, 0.3, 1e-2, 7)], "f64", "jacobi", {}),
    ([(127, 1.7, 1e-3, 7)], "f64", "jacobi", {}), ([(127, 1.7, 1e-3, 7)], "f64", "jacobi", dict(coarse_cutover=7)),
    ([(63, 0.9, 1e-2, 7)], "f32", "jacobi", {}), ([(31, 0.9, 1e-2, 7)], "f64", "zebra", {}),
    ([(63, 0.9, 1e-2, 3)], "f64", "jacobi", dict(wave_regs=0)), ([(63, 0.9, 1e-2, 3)], "f32", "jacobi", dict(wave_regs=0)),
    ([(31, 0.2, 1e-1, 3)], "f64", "jacobi", dict(coarse_wave_n=0)), ([(31, 0.2, 1e-1, 1)], "f64", "zebra", {}),
    ([(63, 0.9, 1e-2, 7), (15, 0.1, 1e-1, 3), (127, 2.2, 1e-2, 1)], "f64", "jacobi", {})])
def test_solve_bits(specs, prec, smoother, ex):
    from paper_2010_00626_amd import kcycle as K
    print(f"[coarsest] {specs} {prec} {smoother} {ex}", flush=True)
    rng = np.random.default_rng(sum(s[0] for s in specs))
    f = [rng.uniform(-1, 1, (s[0], s[0])) for s in specs]
    maxit = 1 if prec == "f32" else 5
    H = K.Hierarchy(specs, prec, exec=ex)
    u = [torch.zeros((s[0], s[0]), dtype=torch.float64, device="cuda") for s in specs]
    H.solve(u, [torch.from_numpy(a).cuda() for a in f], kappa=2, tol=1e-300, maxit=maxit, smoother=smoother)
    for k, s in enumerate(specs):
        Ho = O.Hierarchy(*s, smoother=smoother)
        ref = (Ho.ir_solve if prec == "f32" else Ho.solve)(f[k], kappa=2, tol=1e-300, maxit=maxit)[0]
        assert np.array_equal(u[k].cpu().numpy(), ref), k
    H.close()


@pytest.mark.parametrize("f0,bx", [(float.fromhex("0x1.74p-900") * float.fromhex("0x1.8p+170"), 2.25 * 2.0 ** 341),
                                   (float.fromhex("0x1.74p-900") * float.fromhex("0x1.8p+120"), 2.25 * 2.0 ** 241),
                                   (2.0 ** 880, 0.0), (2.0 ** -880, 0.0), (float.fromhex("0x1.74p-899"), 0.0)])
def test_quotients_at_the_ends_of_the_range(f0, bx):
    """A right-hand side that reaches the 1 x 1 level as f0, divided twice by the root of its matrix: quotients
    below the normal numbers (the first row's second one lies next to a tie), divisors and dividends at the
    limits of the reciprocal's range."""
    from paper_2010_00626_amd import kcycle as K
    n = 15
    print(f"[coarsest] f0={f0} bx={bx}", flush=True)
    v, f = np.zeros((n, n)), np.zeros((n, n))
    f[7, 7] = f0 * (n + 1) ** 2
    Ho = O.Hierarchy(n, 0.4, 1e-2, convection=(bx, 0.0)) if bx else O.Hierarchy(n, 0.4, 1e-2)
    out = []
    for ex in (dict(), dict(wave_regs=0)):   # the register kernel; the LDS kernel, which divides
        H = K.Hierarchy([(n, 0.4, 1e-2)], exec=ex)
        if bx:
            H.set_convection(bx, 0.0)
        d = torch.from_numpy(v.copy()).cuda()
        H.cycle(d, torch.from_numpy(f).cuda(), kappa=1, nu1=0, nu2=0)
        out.append(d.cpu().numpy())
        H.close()
    ref = Ho.cycle(v, f, kappa=1, nu1=0, nu2=0)[0]
    assert np.array_equal(*out)
    # the point above the 1 x 1 level's; interpolation between points adds before it scales, so that below the
    # normal numbers the kernels round once where the oracle rounds each product
    assert ref[7, 7] != 0.0 and out[0][7, 7] == ref[7, 7]
    if abs(ref[7, 7]) > 1e-300:
        assert np.array_equal(out[0], ref)


@pytest.mark.parametrize("nc", [1, 3])
@pytest.mark.parametrize("scale", [2.0 ** -60, 2.0 ** -77, 2.0 ** -79, 2.0 ** -98, 2.0 ** -101, 2.0 ** -125, 0.0])
def test_f32_small_dividends(nc, scale):
    """FP32 cycles whose coarsest dividends lie around the limits of the reciprocal's range, among them those
    whose remainder would be below the normal numbers: one point holds the norm, the rest is small."""
    from paper_2010_00626_amd import kcycle as K
    n = 15
    print(f"[coarsest] f32 nc={nc} scale={scale}", flush=True)
    f = scale * np.random.default_rng(nc).uniform(-1, 1, (n, n))
    if nc == 3:
        f[11, 11] = 1.0   # the last of the 3 x 3 points
    H = K.Hierarchy([(n, 0.4, 1e-2, nc)], "f32")
    u = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    H.solve(u, torch.from_numpy(f).cuda(), kappa=1, nu1=0, nu2=0, tol=1e-300, maxit=1)
    ref = O.Hierarchy(n, 0.4, 1e-2, nc).ir_solve(f, kappa=1, nu1=0, nu2=0, tol=1e-300, maxit=1)[0]
    assert np.array_equal(u.cpu().numpy(), ref)
    H.close()
