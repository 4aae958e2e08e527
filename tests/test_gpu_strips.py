"""Levels that take the streaming strips below stream_n (the next smaller size,
and levels whose problems are many) against the same cycles in tiles
(stream_n = 0), bit for bit: sizes at both sides of each rule, no smoothing on
one side, uneven batches, instances that stop early, FP32 cycles.  The
arithmetic of a point does not depend on the shape, so the tolerance is 0."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("sizes,precision,kappa,nu,smoother", [
    ((1023,), "f64", 2, (2, 2), "jacobi"), ((1023,), "f32", 3, (1, 3), "jacobi"), ((1023, 1023), "f32", 2, (2, 1), "jacobi"),
    ((511,) * 4, "f64", 3, (1, 1), "jacobi"), ((511,) * 3, "f64", 2, (2, 2), "jacobi"),
    ((255,) * 8, "f32", 2, (3, 0), "jacobi"), ((255,) * 7 + (127,), "f64", 2, (0, 2), "jacobi"),
    ((127,) * 32, "f64", 3, (2, 2), "jacobi"), ((127,) * 31 + (63,), "f32", 2, (1, 2), "jacobi"),
    ((511, 1023, 255, 127, 511, 1023), "f64", 3, (2, 2), "jacobi"), ((511,) * 4, "f64", 2, (1, 1), "zebra")])
def test_same_bits_as_tiles(sizes, precision, kappa, nu, smoother):
    from paper_2010_00626_amd import kcycle as K
    print(f"[strips] {sizes} {precision} kappa={kappa} nu={nu} {smoother}", flush=True)
    rng = np.random.default_rng(sum(sizes) + kappa)
    specs = [(n, 0.1 + 0.37 * k, (1e-1, 1e-3)[k % 2]) for k, n in enumerate(sizes)]
    f = [torch.from_numpy(rng.uniform(-1, 1, (n, n))).cuda() for n in sizes]
    out = []
    for ex in (dict(), dict(stream_n=0)):
        H = K.Hierarchy(specs, precision=precision, exec=ex)
        u = [torch.zeros_like(t) for t in f]
        res = H.solve(u, f, kappa=kappa, nu1=nu[0], nu2=nu[1], tol=1e-3, maxit=9, smoother=smoother)
        out.append(([t.cpu().numpy() for t in u], res))
        H.close()
    for a, b in zip(out[0][0], out[1][0]):
        assert np.isfinite(a).all() and np.array_equal(a, b)
    assert np.array_equal(np.asarray(out[0][1][0]), np.asarray(out[1][1][0]))
    assert np.array_equal(np.asarray(out[0][1][1]), np.asarray(out[1][1][1]))
