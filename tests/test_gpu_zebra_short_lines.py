"""zebra_wave_n below 63: short lines in the registers mapping (a line of 3 points fills one lane), bit for bit
against the oracle: every length from 3, batches whose shortest lines do not fill a lane of the launch laid out
for the longest, semi-coarsened levels of few lines, FP32 cycles.  The tolerance is 0."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("sizes,ex,coarsening", [
    ((3,), dict(mode="paper", zebra_wave_n=1), "full"), ((7,), dict(mode="paper", zebra_wave_n=3), "full"),
    ((31,), dict(mode="paper", zebra_wave_n=2, zebra_quad_n=7), "full"), ((127,), dict(coarse_cutover=7, zebra_wave_n=15), "full"),
    ((1023, 7, 31, 3, 255, 15, 511), dict(mode="paper", zebra_wave_n=1), "full"),
    ((511, 3, 7, 15), dict(mode="paper", zebra_wave_n=3, zebra_quad_n=1), "full"),
    ((3,), dict(zebra_wave_n=1), "semi"), ((7,), dict(zebra_wave_n=7), "semi"), ((15,), dict(zebra_wave_n=1), "semi"),
    ((31,), dict(zebra_wave_n=15, zebra_quad_n=1), "semi")])
def test_cycle_bits(sizes, ex, coarsening):
    from paper_2010_00626_amd import kcycle as K
    print(f"[zebra-short] {sizes} {ex} {coarsening}", flush=True)
    rng = np.random.default_rng(sum(sizes))
    specs = [(n, 0.3 + 0.5 * k, 1e-3) for k, n in enumerate(sizes)]
    v0 = [rng.uniform(-1, 1, (n, n)) for n in sizes]
    f = [rng.uniform(-1, 1, (n, n)) for n in sizes]
    H = K.Hierarchy(specs, exec=ex, coarsening=coarsening)
    v = [torch.from_numpy(a.copy()).cuda() for a in v0]
    H.cycle(v, [torch.from_numpy(a).cuda() for a in f], kappa=2, nu1=2, nu2=1, smoother="zebra")
    for k, s in enumerate(specs):
        Ho = O.Hierarchy(*s, smoother="zebra", coarsening=coarsening)
        assert np.array_equal(Ho.stencils, K.level_stencils(*s) if coarsening == "full" else K.semi_stencils(*s)), k
        assert np.array_equal(v[k].cpu().numpy(), Ho.cycle(v0[k], f[k], kappa=2, nu1=2, nu2=1)[0]), k
    H.close()


@pytest.mark.parametrize("n", [3, 15, 63])
def test_f32_step_bits(n):
    from paper_2010_00626_amd import kcycle as K
    print(f"[zebra-short] f32 n={n}", flush=True)
    f = np.random.default_rng(n).uniform(-1, 1, (n, n))
    H = K.Hierarchy([(n, 0.7, 1e-2)], "f32", exec=dict(mode="paper", zebra_wave_n=1))
    u = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    H.solve(u, torch.from_numpy(f).cuda(), kappa=2, tol=1e-300, maxit=1, smoother="zebra")
    ref = O.Hierarchy(n, 0.7, 1e-2, smoother="zebra").ir_solve(f, kappa=2, nu1=2, nu2=2, tol=1e-300, maxit=1)[0]
    assert np.array_equal(u.cpu().numpy(), ref)
    H.close()


def test_short_lines_take_the_registers():
    """The launches of a 31-point problem's levels name four points per lane (0: one thread per line)."""
    from paper_2010_00626_amd import kcycle as K
    n = 31
    H = K.Hierarchy([(n, 0.7, 1e-2)], exec=dict(mode="paper", zebra_wave_n=7))
    f = torch.rand((n, n), dtype=torch.float64, device="cuda")
    H.solve(torch.zeros_like(f), f, kappa=1, tol=1e-300, maxit=1, smoother="zebra")
    seq = [(x[0], x[1]) for x in H.profile_iteration(kappa=1, reps=1, smoother="zebra")["sequence"] if x[0].startswith("k_zebra")]
    assert {d: nm.split(", ")[2] for nm, d in seq} == {0: "4>", 1: "4>", 2: "4>", 3: "0>"}
    H.close()
