"""The fused CG kernels (search direction, operator and dot product in one pass, the update forming
q again) against the oracle at the sizes where their tiles end: part of one tile, a tile's last
column absent, tiles meeting side by side and above each other; one to four iterations (the two
arrays of the search direction by turns), arrays with padding, and a ragged batch.  The tolerances
are those of the repository's PCG comparisons: 1e-11 (FP64), 1e-6 (FP32 preconditioner)."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def array(n, pad, a=None):
    t = torch.full((n, n + pad), float("nan"), dtype=torch.float64, device="cuda")[:, :n]
    if a is not None:
        t.copy_(torch.from_numpy(a))
    return t


def close(got, ref, tol):
    return np.abs(got - ref).max() <= tol * np.abs(ref).max()


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,pad", [(3, 1), (31, 0), (63, 2), (127, 1), (255, 0)])
@pytest.mark.parametrize("maxit", [1, 2, 3, 4])
def test_iterates(n, pad, prec, maxit):
    from paper_2010_00626_amd import kcycle as K
    print(f"[pcg-fused] n={n} pad={pad} {prec} maxit={maxit}", flush=True)
    f = np.random.default_rng(n).uniform(-1, 1, (n, n))
    u = array(n, pad)
    H = K.Hierarchy([(n, 0.9, 1e-3)], prec)
    it, rr, st = H.pcg(u, array(n, pad, f), kappa=2, nu1=1, nu2=1, tol=1e-30, maxit=maxit)
    ref = O.Hierarchy(n, 0.9, 1e-3).pcg(f, kappa=2, nu1=1, nu2=1, tol=1e-30, maxit=maxit, precond_f32=prec == "f32")[0]
    assert it == [maxit] and close(u.cpu().numpy(), ref, 1e-11 if prec == "f64" else 1e-6)
    H.close()


def test_batch():
    from paper_2010_00626_amd import kcycle as K
    print("[pcg-fused] batch", flush=True)
    specs = [(63, 0.4, 1e-2), (15, 1.2, 1e-1), (255, 2.0, 1e-3)]
    rng = np.random.default_rng(2)
    f = [rng.uniform(-1, 1, (s[0], s[0])) for s in specs]
    u = [array(s[0], 0) for s in specs]
    H = K.Hierarchy(specs)
    it, rr, st = H.pcg(u, [array(s[0], 0, a) for s, a in zip(specs, f)], kappa=2, nu1=1, nu2=1, tol=1e-8, maxit=100)
    for k, s in enumerate(specs):
        ref, rc, itr, hist = O.Hierarchy(*s).pcg(f[k], kappa=2, nu1=1, nu2=1, tol=1e-8, maxit=100)
        assert it[k] == itr and st[k] == 0 and close(u[k].cpu().numpy(), ref, 1e-11), k
    H.close()
