"""Fused sibling junctions on launches of far more tiles than the GPU runs at once, whose tiles read points of
neighbours that may long be written: against separate post- and pre-smoothing launches, bit for bit, and against
themselves, run after run."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n,count,kappa,nu,precision,shape", [
    (1023, 4, 2, (2, 2), "f64", dict(tiny_tile_n=4095)), (1023, 4, 3, (1, 3), "f32", dict(tiny_tile_n=4095)),
    (1023, 4, 3, (2, 1), "f64", dict(tiny_tile_n=0, small_tile_n=4095)), (255, 64, 2 ** 31 - 1, (0, 2), "f64", dict(tiny_tile_n=4095)),
    (511, 16, 4, (3, 0), "f32", dict(tiny_tile_n=255)), (2047, 2, 2, (1, 1), "f64", dict(tiny_tile_n=4095))])
def test_many_tiles(n, count, kappa, nu, precision, shape):
    from paper_2010_00626_amd import kcycle as K
    print(f"[junction-buffers] {count} x {n} kappa={kappa} nu={nu} {precision} {shape}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + count)
    f = [2 * torch.rand((n, n), generator=g, dtype=torch.float64, device="cuda") - 1 for _ in range(count)]
    specs = [(n, 0.2 + 0.04 * k, 1e-2) for k in range(count)]
    out = []
    for fuse in (1, 0):
        H = K.Hierarchy(specs, precision, exec=dict(shape, stream_n=0, fuse_junctions=fuse))
        for _ in range(3 if fuse else 1):
            u = [torch.zeros_like(x) for x in f]
            it, rr, st = H.solve(u, f, kappa=kappa, nu1=nu[0], nu2=nu[1], tol=1e-300, maxit=6)
            out.append(u)
        launches = H.stats()["grid_launches_per_iteration"]
        if fuse:
            fused = launches
        H.close()
    assert fused < launches
    for u in out[:-1]:
        assert all(torch.equal(a, b) and bool(torch.isfinite(a).all()) for a, b in zip(u, out[-1]))


def test_mixed_sizes_and_early_stops():
    """Instances of several depths, some finished while others go on, against their own solves without junctions."""
    from paper_2010_00626_amd import kcycle as K
    print("[junction-buffers] mixed sizes", flush=True)
    sizes = (255, 511, 127, 1023, 255, 63)
    specs = [(n, 0.3 * k, (1e-1, 1e-2)[k % 2]) for k, n in enumerate(sizes)]
    rng = np.random.default_rng(6)
    f = [torch.from_numpy(rng.uniform(-1, 1, (n, n))).cuda() for n in sizes]
    H = K.Hierarchy(specs, exec=dict(stream_n=0))
    u = [torch.zeros_like(x) for x in f]
    it, rr, st = H.solve(u, f, kappa=3, tol=1e-5, maxit=200)
    H.close()
    for k, s in enumerate(specs):
        H1 = K.Hierarchy([s], exec=dict(stream_n=0, fuse_junctions=0))
        v = torch.zeros_like(f[k])
        it1, rr1, st1 = H1.solve(v, f[k], kappa=3, tol=1e-5, maxit=200)
        assert it1 == [it[k]] and st1 == [st[k]] and torch.equal(u[k], v), k
        H1.close()
