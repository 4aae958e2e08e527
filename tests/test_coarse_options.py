"""The persistent kernel's options are honoured: an explicit coarse cutover is the one that is planned,
the automatic one (0, the default) is what the header states, and the statistics name the plan."""
import numpy as np
import pytest

from paper_2010_00626_amd import autotune, kcycle as K

P1023 = [(1023, 0.4, 1e-3)]


def counts(problems, **ex):
    return K.schedule_counts(problems, 3, **ex)


@pytest.mark.parametrize("problems,ex,planned", [
    (P1023, {}, 63), ([(255, 0.4, 1e-3, 3)] * 256, {}, 63), ([(511, 0.4, 1e-3), (127, 1.0, 1e-2)], {}, 63),
    ([(1023, 0.4, 1e-3, 7)], {}, 31), ([(255, 0.4, 1e-3)] * 257, {}, 31), ([(255, 0.4, 1e-3, 3), (255, 0.4, 1e-3, 1)], {}, 31),
    (P1023, dict(wave_regs=0), 31), (P1023, dict(coarse_wave_n=7), 31), (P1023, dict(coarse_threads=256), 31),
    (P1023, dict(coarse_threads=1024), 31)])
def test_automatic_cutover(problems, ex, planned):
    assert counts(problems, **ex) == counts(problems, coarse_cutover=planned, **ex)
    other = 31 if planned == 63 and not ex else 15
    assert counts(problems, **ex) != counts(problems, coarse_cutover=other, **ex)


def test_cutover_range():
    for bad in (-1, 1, 6, 64):
        with pytest.raises(K.KCycleError) as ei:
            counts(P1023, coarse_cutover=bad)
        assert ei.value.status == K.KC_ERR_ARG
    e = K.exec_options()
    assert e.coarse_cutover == 0


def test_tuner_tells_cutovers_apart():
    seen = set()
    for cut in (15, 31, 63):
        cand = dict(coarse_cutover=cut, coarse_threads=512, coarse_wave_n=15)
        assert autotune._relevant(cand, seen, [255])
        assert not autotune._relevant(dict(cand), seen, [255])


@pytest.mark.gpu
@pytest.mark.parametrize("nc,cutover,planned,kernel", [(1, 31, 31, "k_subtree_regs<double, 31, 4, 1>"),
                                                       (3, 31, 31, "k_subtree_regs<double, 31, 4, 3>"),
                                                       (1, 0, 63, "k_subtree_regs<double, 63, 8, 1>"),
                                                       (3, 63, 63, "k_subtree_regs<double, 63, 4, 3>"),
                                                       (7, 0, 31, "k_subtree<double, 512, false>")])
def test_planned_cutover_runs(nc, cutover, planned, kernel):
    from oracle import oracle as O
    import torch
    n = 127
    print(f"[coarse-options] nc={nc} cutover={cutover}", flush=True)
    rng = np.random.default_rng(nc + cutover)
    f = rng.uniform(-1, 1, (n, n))
    H = K.Hierarchy([(n, 0.9, 1e-2, nc)], exec=dict(coarse_cutover=cutover))
    u = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    it, rr, st = H.solve(u, torch.from_numpy(f).cuda(), kappa=3, tol=1e-8, maxit=300)
    ref, rc, itr, hist = O.Hierarchy(n, 0.9, 1e-2, nc).solve(f, kappa=3, tol=1e-8, maxit=300)
    assert st == [0] and it == [itr] and np.array_equal(u.cpu().numpy(), ref)
    s = H.stats()
    assert s["coarse_cutover"] == planned and (n >> s["levels"][0]["cut"]) == planned
    names = [k["name"] for k in H.profile_iteration(kappa=3, reps=1)["kernels"]]
    assert kernel in names and sum(x.startswith("k_subtree") for x in names) == 1, names
    H.close()


@pytest.mark.gpu
def test_tuner_plans_what_it_times():
    """A stage that leaves the cutover open is timed, kept and reported with the planned one."""
    import torch
    n = 127
    H = K.Hierarchy([(n, 0.9, 1e-2)])
    f = torch.rand((n, n), dtype=torch.float64, device="cuda")
    res = autotune.tune(H, torch.zeros_like(f), f, 2, iters=2, force=True,
                        stages=((dict(tiny_tile_n=255), dict(tiny_tile_n=0), dict(coarse_cutover=63), dict(coarse_cutover=31)),))
    assert sorted(t["exec"]["coarse_cutover"] for t in res["trials"]) == [31, 63, 63]
    assert H.stats()["coarse_cutover"] == res["exec"]["coarse_cutover"]
    H.close()


@pytest.mark.gpu
@pytest.mark.parametrize("prec,ex,kernel", [
    ("f32", dict(coarse_cutover=63, coarse_threads=1024), "k_subtree<float, 1024, false>"),
    ("f32", dict(coarse_cutover=31, coarse_threads=1024), "k_subtree<float, 1024, false>"),
    ("f32", dict(coarse_cutover=31, coarse_threads=256), "k_subtree<float, 256, false>"),
    ("f64", dict(coarse_cutover=15, coarse_threads=256), "k_subtree<double, 256, false>"),
    ("f32", dict(coarse_cutover=63, wave_regs=0), "k_subtree<float, 512, false>"),
    ("f32", dict(coarse_cutover=31, wave_regs=0), "k_subtree<float, 512, false>"),
    ("f64", dict(coarse_cutover=63, wave_regs=0), "k_subtree<double, 512, false>"),
    ("f64", dict(coarse_cutover=31, coarse_wave_n=7), "k_subtree<double, 512, false>"),
    ("f32", dict(coarse_cutover=31), "k_subtree_regs<float, 31, 4, 1>")])
def test_threads_are_honoured(prec, ex, kernel):
    """The kernel asked for runs, and its step is the oracle's (FP32: its emulation) bit for bit."""
    from oracle import oracle as O
    import torch
    n = 127
    print(f"[coarse-options] {prec} {ex}", flush=True)
    f = np.random.default_rng(5).uniform(-1, 1, (n, n))
    Ho = O.Hierarchy(n, 0.9, 1e-2)
    ref = (Ho.ir_solve if prec == "f32" else Ho.solve)(f, kappa=3, tol=1e-300, maxit=1)[0]
    H = K.Hierarchy([(n, 0.9, 1e-2)], prec, exec=ex)
    u = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    it, rr, st = H.solve(u, torch.from_numpy(f).cuda(), kappa=3, tol=1e-300, maxit=1)
    assert it == [1] and np.array_equal(u.cpu().numpy(), ref)
    names = [k["name"] for k in H.profile_iteration(kappa=3, reps=1)["kernels"]]
    assert [x for x in names if x.startswith("k_subtree")] == [kernel], names
    H.close()


def test_counts_of_streamed_levels():
    """Levels that a batch streams below stream_n have no fused sibling launches, in the counts too."""
    four = [(1023, 0.4, 1e-3)] * 4
    assert counts(four) == counts(four, stream_n=0, small_tile_n=0, mid_tile_n=4095)
    assert counts(four) != counts(four, stream_n=0)


@pytest.mark.gpu
@pytest.mark.parametrize("problems,ex,smoother", [
    ([(1023, 0.4, 1e-3)], {}, "jacobi"), ([(1023, 0.4, 1e-3)] * 4, {}, "jacobi"), ([(255, 0.4, 1e-3, 7)], {}, "jacobi"),
    ([(255, 0.4, 1e-3)], dict(coarse_cutover=31), "jacobi"), ([(255, 0.4, 1e-3)], dict(mode="paper"), "zebra"),
    ([(255, 0.4, 1e-3)], {}, "zebra")])
def test_counts_are_the_launches(problems, ex, smoother):
    import torch
    print(f"[coarse-options] counts {problems[0]} x {len(problems)} {ex} {smoother}", flush=True)
    c = K.schedule_counts(problems, 2, smoother=smoother, **ex)
    H = K.Hierarchy(problems, exec=ex)
    v = [torch.zeros((p[0], p[0]), dtype=torch.float64, device="cuda") for p in problems]
    H.cycle(v, [torch.ones_like(t) for t in v], kappa=2, smoother=smoother)
    s = H.stats()
    # zebra in the fused mode: three launches fewer per call above the cutover (one call on 255, two on 127)
    fewer = 3 * 3 if smoother == "zebra" and not ex else 0
    assert s["grid_launches_per_iteration"] == c["grid_launches"] - fewer
    assert s["subtree_launches_per_iteration"] == c["subtree_launches"]
    H.close()
