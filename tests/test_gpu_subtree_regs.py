"""The register kernel of the coarse levels (k_subtree_regs) against the oracle, bit for bit: every
top level it takes (15, 31, 63), 1 x 1 and 3 x 3 coarsest levels, the counters' and sweeps' extremes,
problems that it runs whole (stop test included), dividends outside the range of its division, and
batches whose instances it shares a depth with.  The arithmetic of a point is the LDS kernel's, so
the tolerance is 0."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
W = 2 ** 31 - 1


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("n,nc,cutover,kappa,nu1,nu2,scale", [
    (127, 1, 15, 3, 2, 2, 1.0), (127, 3, 15, W, 1, 0, 1.0), (127, 1, 31, 1, 0, 1, 1.0), (255, 3, 31, 2, 3, 3, 1.0),
    (127, 1, 31, W, 2, 1, 1.0), (127, 1, 63, 4, 1, 2, 1.0), (255, 3, 63, 3, 2, 2, 1.0), (15, 1, 31, 2, 2, 2, 1.0),
    (15, 3, 15, 3, 0, 0, 1.0), (31, 3, 31, 1, 2, 2, 1.0), (63, 1, 63, W, 2, 2, 1.0), (63, 1, 31, 2, 2, 2, 1e-280),
    (31, 3, 31, 2, 2, 2, 1e-280), (63, 3, 31, 2, 2, 2, 0.0)])
def test_cycle_bits(n, nc, cutover, kappa, nu1, nu2, scale):
    from paper_2010_00626_amd import kcycle as K
    print(f"[subtree-regs] n={n} nc={nc} cutover={cutover} kappa={kappa} nu={nu1}+{nu2} scale={scale}", flush=True)
    rng = np.random.default_rng(n + cutover)
    v0, f = scale * rng.uniform(-1, 1, (n, n)), scale * rng.uniform(-1, 1, (n, n))
    H = K.Hierarchy([(n, 1.1, 1e-2, nc)], exec=dict(coarse_cutover=cutover))
    v = dev(v0)
    H.cycle(v, dev(f), kappa=kappa, nu1=nu1, nu2=nu2)
    ref = O.Hierarchy(n, 1.1, 1e-2, nc).cycle(v0, f, kappa=min(kappa, 64), nu1=nu1, nu2=nu2)[0]
    assert np.array_equal(v.cpu().numpy(), ref)
    H.close()


@pytest.mark.parametrize("n,nc,cutover", [(15, 1, 31), (31, 3, 31), (31, 1, 63), (63, 1, 63), (63, 3, 63)])
def test_whole_solve_bits(n, nc, cutover):
    from paper_2010_00626_amd import kcycle as K
    print(f"[subtree-regs] whole solve n={n} nc={nc} cutover={cutover}", flush=True)
    f = np.random.default_rng(n).uniform(-1, 1, (n, n))
    H = K.Hierarchy([(n, 0.6, 1e-2, nc)], exec=dict(coarse_cutover=cutover))
    u = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    it, rr, st = H.solve(u, dev(f), kappa=2, tol=1e-9, maxit=300)
    ref, rc, itr, hist = O.Hierarchy(n, 0.6, 1e-2, nc).solve(f, kappa=2, tol=1e-9, maxit=300)
    assert st == [0] and it == [itr] and np.array_equal(u.cpu().numpy(), ref)
    H.close()


@pytest.mark.parametrize("specs", [[(63, 0.3, 1e-2), (255, 1.9, 1e-3), (127, 2.5, 1e-1)],      # one top level size
                                   [(63, 0.3, 1e-2), (15, 1.9, 1e-3), (31, 2.5, 1e-1)],        # whole problems, two sizes
                                   [(63, 0.3, 1e-2, 3), (127, 1.9, 1e-3, 1)]])                 # two coarsest sizes
def test_batch_bits(specs):
    from paper_2010_00626_amd import kcycle as K
    print(f"[subtree-regs] batch {specs}", flush=True)
    rng = np.random.default_rng(8)
    f = [rng.uniform(-1, 1, (s[0], s[0])) for s in specs]
    H = K.Hierarchy(specs)
    u = [torch.zeros_like(dev(a)) for a in f]
    it, rr, st = H.solve(u, [dev(a) for a in f], kappa=3, tol=1e-8, maxit=300)
    for k, s in enumerate(specs):
        ref, rc, itr, hist = O.Hierarchy(*s).solve(f[k], kappa=3, tol=1e-8, maxit=300)
        assert it[k] == itr and np.array_equal(u[k].cpu().numpy(), ref), k
    H.close()
