"""The zebra line kernel's registers mapping against the oracle, bit for bit,
at the sizes where its layout changes: 4, 8 and 16 points per lane, part of a
wave or a whole one per line, one chunk or several, 32 or 64 lanes per y-line,
and batches whose smaller instances run in a launch laid out for a larger one.
The arithmetic of a point does not depend on the layout, so the tolerance is 0.
"""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def padded(a, pad):
    """a GPU array with leading dimension n + pad holding a"""
    n = a.shape[0]
    t = torch.full((n, n + pad), float("nan"), dtype=torch.float64, device="cuda")[:, :n]
    t.copy_(torch.from_numpy(a))
    return t


@pytest.mark.parametrize("n,quad_n,pad", [(63, 0, 0), (63, 63, 3), (127, 0, 1), (255, 255, 0), (511, 0, 0),
                                          (511, 127, 7), (1023, 8191, 2), (1023, 1023, 1), (2047, 0, 0),
                                          (2047, 2047, 1), (4095, 8191, 0)])
def test_cycle_bits(n, quad_n, pad):
    from paper_2010_00626_amd import kcycle as K
    print(f"[zebra-registers] n={n} quad_n={quad_n} pad={pad}", flush=True)
    rng = np.random.default_rng(3 * n + pad)
    v0, f = rng.uniform(-1, 1, (n, n)), rng.uniform(-1, 1, (n, n))
    H = K.Hierarchy([(n, 2.1, 1e-3)], exec=dict(zebra_quad_n=quad_n))
    v = padded(v0, pad)
    H.cycle(v, padded(f, pad), kappa=1, nu1=2, nu2=2, smoother="zebra")
    ref = O.Hierarchy(n, 2.1, 1e-3, smoother="zebra").cycle(v0, f, kappa=1, nu1=2, nu2=2)[0]
    assert np.array_equal(v.cpu().numpy(), ref)
    H.close()


@pytest.mark.parametrize("sizes,quad_n", [((63, 1023, 127, 255), 8191), ((1023, 511, 63), 63), ((255, 63, 511), 0)])
def test_batch_bits(sizes, quad_n):
    from paper_2010_00626_amd import kcycle as K
    print(f"[zebra-registers] batch {sizes} quad_n={quad_n}", flush=True)
    rng = np.random.default_rng(sum(sizes))
    specs = [(n, 0.3 + 0.5 * k, 1e-3) for k, n in enumerate(sizes)]
    v0 = [rng.uniform(-1, 1, (n, n)) for n in sizes]
    f = [rng.uniform(-1, 1, (n, n)) for n in sizes]
    H = K.Hierarchy(specs, exec=dict(zebra_quad_n=quad_n))
    v = [padded(a, 0) for a in v0]
    H.cycle(v, [padded(a, 0) for a in f], kappa=2, nu1=2, nu2=1, smoother="zebra")
    for k, s in enumerate(specs):
        ref = O.Hierarchy(*s, smoother="zebra").cycle(v0[k], f[k], kappa=2, nu1=2, nu2=1)[0]
        assert np.array_equal(v[k].cpu().numpy(), ref), k
    H.close()


@pytest.mark.parametrize("n", [255, 2047])
def test_semi_cycle_bits(n):
    from paper_2010_00626_amd import kcycle as K
    print(f"[zebra-registers] semi n={n}", flush=True)
    rng = np.random.default_rng(n)
    v0, f = rng.uniform(-1, 1, (n, n)), rng.uniform(-1, 1, (n, n))
    H = K.Hierarchy([(n, 0.2, 1e-4)], coarsening="semi")
    v = padded(v0, 0)
    H.cycle(v, padded(f, 0), kappa=1, nu1=1, nu2=1, smoother="zebra")
    ref = O.Hierarchy(n, 0.2, 1e-4, smoother="zebra", coarsening="semi").cycle(v0, f, kappa=1, nu1=1, nu2=1)[0]
    assert np.array_equal(v.cpu().numpy(), ref)
    H.close()
