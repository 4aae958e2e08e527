"""Zebra relaxation in the persistent kernel (lines over the lanes, four points
each) against the oracle, bit for bit: every level size it holds, the smallest
thread count of each cutover, FP64 and mixed batches.  The arithmetic of a
point does not depend on the layout, so the tolerance is 0."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("sizes,cutover,threads,wave_n,kappa", [
    ((3,), 31, 512, 15, 1), ((7,), 31, 512, 0, 2), ((15,), 31, 256, 7, 3), ((31,), 31, 256, 15, 2),
    ((63,), 63, 512, 0, 2), ((63,), 63, 512, 15, 3), ((127,), 63, 512, 15, 2),
    ((31, 63, 15, 7, 3), 63, 512, 15, 2), ((63, 127, 31), 31, 256, 3, 2)])
def test_cycle_bits(sizes, cutover, threads, wave_n, kappa):
    from paper_2010_00626_amd import kcycle as K
    print(f"[zebra-lds] {sizes} cutover={cutover} threads={threads} wave_n={wave_n} kappa={kappa}", flush=True)
    rng = np.random.default_rng(sum(sizes) + 7 * kappa)
    specs = [(n, 0.2 + 0.4 * k, 1e-3) for k, n in enumerate(sizes)]
    v0 = [rng.uniform(-1, 1, (n, n)) for n in sizes]
    f = [rng.uniform(-1, 1, (n, n)) for n in sizes]
    H = K.Hierarchy(specs, exec=dict(coarse_cutover=cutover, coarse_threads=threads, coarse_wave_n=wave_n))
    v = [torch.from_numpy(a.copy()).cuda() for a in v0]
    H.cycle(v, [torch.from_numpy(a).cuda() for a in f], kappa=kappa, nu1=2, nu2=2, smoother="zebra")
    for k, s in enumerate(specs):
        ref = O.Hierarchy(*s, smoother="zebra").cycle(v0[k], f[k], kappa=kappa, nu1=2, nu2=2)[0]
        assert np.array_equal(v[k].cpu().numpy(), ref), k
    H.close()
