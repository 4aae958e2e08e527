"""Zebra cycles whose transfers run as one launch each way against one kernel
per operation (mode 1), bit for bit: every tile size of the fused kernels, the
streaming kernels, no relaxation on one side, padded arrays, mixed batches,
FP32 cycles.  The arithmetic of a point is the same, so the tolerance is 0."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def padded(a, pad):
    n = a.shape[0]
    t = torch.full((n, n + pad), float("nan"), dtype=torch.float64, device="cuda")[:, :n]
    t.copy_(torch.from_numpy(a))
    return t


@pytest.mark.parametrize("sizes,cutover,kappa,nu,pad", [
    ((63,), 7, 3, (2, 2), 0), ((127,), 15, 2, (1, 0), 1), ((255,), 31, 2, (0, 2), 3), ((511,), 63, 1, (2, 1), 0),
    ((1023,), 63, 2, (2, 2), 5), ((2047,), 63, 1, (1, 1), 1), ((4095,), 63, 1, (1, 0), 0),
    ((31, 255, 63, 1023), 15, 2, (2, 1), 2), ((2047, 63, 511), 31, 1, (1, 1), 0)])
def test_modes_agree(sizes, cutover, kappa, nu, pad):
    from paper_2010_00626_amd import kcycle as K
    print(f"[zebra-transfers] {sizes} cutover={cutover} kappa={kappa} nu={nu} pad={pad}", flush=True)
    rng = np.random.default_rng(sum(sizes) + kappa)
    specs = [(n, 0.2 + 0.4 * k, 1e-3) for k, n in enumerate(sizes)]
    v0 = [rng.uniform(-1, 1, (n, n)) for n in sizes]
    f = [rng.uniform(-1, 1, (n, n)) for n in sizes]
    out = []
    for ex in (dict(coarse_cutover=cutover), dict(mode=1)):
        H = K.Hierarchy(specs, exec=ex)
        v = [padded(a, pad) for a in v0]
        fd = [padded(a, pad) for a in f]
        for _ in range(2):
            H.cycle(v, fd, kappa=kappa, nu1=nu[0], nu2=nu[1], smoother="zebra")
        out.append([t.cpu().numpy() for t in v])
        H.close()
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("n", [255, 1023])
def test_f32_modes_agree(n):
    from paper_2010_00626_amd import kcycle as K
    print(f"[zebra-transfers] f32 n={n}", flush=True)
    f = torch.from_numpy(np.random.default_rng(n).uniform(-1, 1, (n, n))).cuda()
    out = []
    for ex in (dict(), dict(mode=1)):
        H = K.Hierarchy([(n, 0.7, 1e-2)], precision="f32", exec=ex)
        u = torch.zeros_like(f)
        H.solve(u, f, kappa=2, nu1=2, nu2=2, smoother="zebra", tol=1e-8, maxit=60)
        out.append(u.cpu().numpy())
        H.close()
    assert np.isfinite(out[0]).all() and np.array_equal(*out)
