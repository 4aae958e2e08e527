"""Register kernels where the other tests do not reach, bit for bit: FP32 cycles of k_subtree_regs above 1 x 1
and 3 x 3 coarsest levels and its launches of many instances (257 problems keep a cutover of 31), FP32 zebra
lines in registers with several chunks per line, and the default mapping of 8191-point y-lines.  The
arithmetic of a point does not depend on the kernel, so the tolerance is 0."""
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


def solve(specs, prec, f, ex, kappa, nu, maxit, smoother="jacobi", profile=False):
    from paper_2010_00626_amd import kcycle as K
    H = K.Hierarchy(specs, prec, exec=ex)
    u = [torch.zeros((s[0], s[0]), dtype=torch.float64, device="cuda") for s in specs]
    it, rr, st = H.solve(u, [torch.from_numpy(a).cuda() for a in f], kappa=kappa, nu1=nu[0], nu2=nu[1], tol=1e-300,
                         maxit=maxit, smoother=smoother)
    assert it == [maxit] * len(specs)
    out = [t.cpu().numpy() for t in u]
    names = []
    if profile:
        p = H.profile_iteration(kappa=kappa, nu1=nu[0], nu2=nu[1], smoother=smoother, reps=1)
        names = [k["name"] for k in p["kernels"]]
    H.close()
    return out, names


@pytest.mark.parametrize("n,nc,cutover,kappa,nu,kernel", [
    (15, 3, 31, 3, (2, 2), "15, 1, 3"), (31, 3, 31, 2, (1, 2), "31, 4, 3"), (63, 3, 63, W, (2, 2), "63, 8, 3"),
    (63, 3, 15, 4, (2, 1), "15, 1, 3"), (127, 3, 31, 3, (2, 2), "31, 4, 3"), (255, 3, 0, 2, (3, 0), "63, 8, 3"),
    (255, 3, 63, 1, (0, 2), "63, 8, 3"), (127, 1, 31, W, (2, 2), "31, 4, 1"), (255, 1, 31, 2, (0, 3), "31, 4, 1"),
    (127, 1, 0, 3, (1, 1), "63, 8, 1"), (31, 1, 31, 4, (3, 3), "31, 4, 1")])
def test_f32_step_bits(n, nc, cutover, kappa, nu, kernel):
    print(f"[register-kernels] f32 n={n} nc={nc} cutover={cutover} kappa={kappa} nu={nu}", flush=True)
    f = np.random.default_rng(n + 5 * nc + cutover).uniform(-1, 1, (n, n))
    (u,), names = solve([(n, 0.8, 1e-2, nc)], "f32", [f], dict(coarse_cutover=cutover), kappa, nu, 1, profile=True)
    assert f"k_subtree_regs<float, {kernel}>" in names, names
    ref = O.Hierarchy(n, 0.8, 1e-2, nc).ir_solve(f, kappa=min(kappa, 64), nu1=nu[0], nu2=nu[1], tol=1e-300, maxit=1)[0]
    assert np.array_equal(u, ref)


@pytest.mark.parametrize("prec,nc", [("f64", 1), ("f32", 1), ("f64", 3), ("f32", 3)])
def test_many_instances(prec, nc):
    from paper_2010_00626_amd.kcycle import level_stencils
    print(f"[register-kernels] 257 problems {prec} nc={nc}", flush=True)
    rng = np.random.default_rng(257 + nc)
    specs = [((63, 127, 31)[k % 3], 0.01 * k, (1e-1, 1e-3)[k % 2], nc) for k in range(257)]
    f = [rng.uniform(-1, 1, (s[0], s[0])) for s in specs]
    maxit = 1 if prec == "f32" else 3
    u, names = solve(specs, prec, f, {}, 3, (2, 1), maxit, profile=True)
    assert [x for x in names if x.startswith("k_subtree")] == [f"k_subtree_regs<{'float' if prec == 'f32' else 'double'}, 31, 4, {nc}>"]
    same = 0
    for k, s in enumerate(specs):
        if k % 8 == 3:   # alone, in the LDS kernel
            assert np.array_equal(u[k], solve([s], prec, [f[k]], dict(wave_regs=0), 3, (2, 1), maxit)[0][0]), k
        Ho = O.Hierarchy(*s)
        if not np.array_equal(level_stencils(*s), Ho.stencils):
            continue   # cos or sin of the angle, called apart or together, differ in the last bit
        same += 1
        ref = (Ho.ir_solve if prec == "f32" else Ho.solve)(f[k], kappa=3, nu1=2, nu2=1, tol=1e-300, maxit=maxit)[0]
        assert np.array_equal(u[k], ref), k
    assert same > 250


@pytest.mark.parametrize("n,quad_n", [(63, 0), (255, 255), (511, 8191), (1023, 8191), (1023, 1023), (2047, 8191),
                                      (2047, 1023), (4095, 2047)])
def test_f32_zebra_step_bits(n, quad_n):
    print(f"[register-kernels] f32 zebra n={n} quad_n={quad_n}", flush=True)
    f = np.random.default_rng(n + quad_n).uniform(-1, 1, (n, n))
    spec = [(n, 2.1, 1e-3)]
    (a,), _ = solve(spec, "f32", [f], dict(zebra_quad_n=quad_n), 1, (2, 2), 1, "zebra")
    (b,), _ = solve(spec, "f32", [f], dict(zebra_wave_n=0), 1, (2, 2), 1, "zebra")   # one thread per line
    assert np.isfinite(a).all() and np.array_equal(a, b)
    ref = O.Hierarchy(*spec[0], smoother="zebra").ir_solve(f, kappa=1, nu1=2, nu2=2, tol=1e-300, maxit=1)[0]
    assert np.array_equal(a, ref)


@pytest.mark.parametrize("n,coarsening", [(8191, "full"), (2047, "semi"), (4095, "semi")])
def test_long_lines_as_one_thread_per_line(n, coarsening):
    """FP64 at the default options against one thread per line: 32 lanes per y-line in 16 chunks; x-lines alone."""
    from paper_2010_00626_amd import kcycle as K
    print(f"[register-kernels] zebra n={n} {coarsening}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    f, v0 = (2 * torch.rand((n, n), generator=g, dtype=torch.float64, device="cuda") - 1 for _ in range(2))
    out = []
    for ex in (dict(), dict(zebra_wave_n=0)):
        H = K.Hierarchy([(n, 2.1, 1e-3)], exec=ex, coarsening=coarsening)
        v = v0.clone()
        H.cycle(v, f, kappa=1, nu1=2, nu2=2, smoother="zebra")
        out.append(v)
        H.close()
    assert bool(torch.isfinite(out[0]).all()) and torch.equal(*out)
