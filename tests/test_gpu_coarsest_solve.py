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
