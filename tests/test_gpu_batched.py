"""GPU parity of the batched form (8 right-hand sides per launch) through the
C ABI: the batched symmetric V-cycle against the oracle's cycle right-hand
side by right-hand side, and the batched CG against the oracle's CG per
right-hand side (tolerance model of test_gpu_pcg: the dot products are
summed in another order).
"""
import sys

import numpy as np
import pytest

import oracle
import synth
from tests.conftest import problem
from tests.test_gpu_pcg import PREC, both
from tests.test_gpu_parity import assert_same_bits

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def rhs_block(prob, nrhs, seed=3):
    y = synth.uniform(seed, "noise", nrhs * prob.n, -1.0, 1.0).reshape(nrhs, prob.n)
    return np.ascontiguousarray(prob.mass[None, :] * y) if prob.mass is not None else y


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("name,minc,nrhs", [("ico4", 100, 8), ("torus96", 200, 3), ("pc20k", 500, 11),
                                            ("ico3", 100, 1), ("hubs_big", 1000, 8), ("torus256", 1000, 8)])
def test_batched_preconditioner_parity(name, minc, nrhs, precision):
    _say(f"[gpu] batched preconditioner {precision} {name} nrhs={nrhs}")
    prob = problem(name)
    orc, gpu = both(prob, min_coarse_points=minc)
    R = np.random.default_rng(8).uniform(-1, 1, (nrhs, prob.n))
    Z = gpu.precondition_batched(torch.from_numpy(R).cuda(), precision=precision).cpu().numpy()
    single = [gpu.precondition(torch.from_numpy(R[q].copy()).cuda(), precision=precision).cpu().numpy()
              for q in range(nrhs)]
    for q in range(nrhs):
        zo = orc.precondition(R[q], PREC[precision])
        assert_same_bits(zo, Z[q], f"{name} {precision} right-hand side {q}")
        # each right-hand side gets the single-vector arithmetic
        assert np.array_equal(Z[q], single[q]), q


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("name,minc,nrhs", [("ico4", 100, 8), ("torus96", 200, 5), ("pc20k", 500, 10),
                                            ("hubs_big", 1000, 8)])
def test_batched_pcg_parity(name, minc, nrhs, precision):
    _say(f"[gpu] batched CG {precision} {name} nrhs={nrhs}")
    prob = problem(name)
    orc, gpu = both(prob, min_coarse_points=minc)
    B = rhs_block(prob, nrhs)
    tol = 1e-8
    X, infos, st = gpu.solve_pcg_batched(torch.from_numpy(B).cuda(), tol=tol, precision=precision)
    assert st == 0
    X = X.cpu().numpy()
    A = prob.matrix()
    u = 2.0 ** -53 if precision == "f64" else 2.0 ** -24
    for q in range(nrhs):
        x_o, it_o, hist_o, st_o, fin_o = orc.solve_pcg(B[q], tol=tol, precision=PREC[precision])
        assert st_o == 0
        res = np.linalg.norm(B[q] - A @ X[q]) / np.linalg.norm(B[q])
        assert res <= tol * (1 + 1e-9), (q, res)
        assert abs(res - infos[q].rel_residual) <= 1e-6 * res
        bound = 1e-6 * hist_o[-1] + 64 * u * len(hist_o) * (hist_o[-2] if len(hist_o) > 1 else 1.0)
        near = abs(hist_o[-1] - tol) <= bound
        assert infos[q].iterations == it_o or (near and abs(infos[q].iterations - it_o) == 1), \
            (q, infos[q].iterations, it_o)
        assert np.linalg.norm(X[q] - x_o) <= 1e-6 * np.linalg.norm(x_o), q


def test_batched_edge_cases():
    _say("[gpu] batched CG edge cases")
    g = pytest.importorskip("paper_2307_04886_amd")
    prob = problem("ico4")
    orc, gpu = both(prob, min_coarse_points=100)
    n = prob.n
    B = rhs_block(prob, 4)
    B[2] = 0.0                                                   # a zero right-hand side
    X0 = np.random.default_rng(1).uniform(-1, 1, (4, n))         # non-zero initial guesses
    X, infos, st = gpu.solve_pcg_batched(torch.from_numpy(B).cuda(), torch.from_numpy(X0).cuda(), precision="f32")
    assert st == 0
    X = X.cpu().numpy()
    assert not X[2].any() and infos[2].iterations == 0
    A = prob.matrix()
    for q in (0, 1, 3):
        assert np.linalg.norm(B[q] - A @ X[q]) <= 1e-8 * np.linalg.norm(B[q])
    # no right-hand sides
    X, infos, st = gpu.solve_pcg_batched(torch.zeros((0, n), dtype=torch.float64).cuda())
    assert st == 0 and infos == []
    # iteration cap
    X, infos, st = gpu.solve_pcg_batched(torch.from_numpy(B).cuda(), tol=1e-15, max_iters=2)
    assert st == 1
    bad = torch.from_numpy(B).cuda()
    bad[1, 7] = float("inf")
    with pytest.raises(g.GMGError) as e:
        gpu.solve_pcg_batched(bad)
    assert e.value.status == -1


def test_batched_workload_sample():
    """Four meshes of the many-mesh workload, 8 right-hand sides each, float
    preconditioner, 1e-8: every solution meets the tolerance; the first mesh
    against the oracle."""
    _say("[gpu] batched workload sample")
    import paper_2307_04886_amd as g
    from paper_2307_04886_amd.binding import from_problem
    g.library()
    batch = synth.config_batched(count=4)
    for i, (prob, B) in enumerate(batch):
        h, _ = from_problem(prob)
        X, infos, st = h.solve_pcg_batched(torch.from_numpy(B).cuda(), tol=1e-8, precision="f32")
        assert st == 0
        X = X.cpu().numpy()
        A = prob.matrix()
        for q in range(B.shape[0]):
            assert np.linalg.norm(B[q] - A @ X[q]) <= 1e-8 * (1 + 1e-9) * np.linalg.norm(B[q])
        if i == 0:
            orc = oracle.Hierarchy.from_problem(prob)
            for q in range(0, B.shape[0], 3):
                x_o = orc.solve_pcg(B[q], tol=1e-8, precision=1)[0]
                assert np.linalg.norm(X[q] - x_o) <= 1e-6 * np.linalg.norm(x_o)
        _say(f"[gpu]   mesh {i}: n={prob.n}, CG iterations {[inf.iterations for inf in infos]}")


def test_many_meshes_on_concurrent_streams():
    """The many-mesh driver (one stream per worker thread) gives the same bits as
    running the meshes one after another."""
    _say("[gpu] many meshes on concurrent streams")
    import paper_2307_04886_amd as g
    from paper_2307_04886_amd.batch import solve_many
    g.library()
    batch = synth.config_batched(count=6, hi=40_000)
    systems = []
    for prob, B in batch:
        t = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in
             (prob.points, prob.edges, prob.indptr, prob.indices, prob.data)]
        systems.append(tuple(t) + (torch.from_numpy(B).cuda(),))
    seq = solve_many(systems, streams=1)
    par = solve_many(systems, streams=4)
    for (xa, ia, sa), (xb, ib, sb), (prob, B) in zip(seq, par, batch):
        assert sa == sb == 0
        assert torch.equal(xa, xb)
        A = prob.matrix()
        X = xb.cpu().numpy()
        for q in range(B.shape[0]):
            assert np.linalg.norm(B[q] - A @ X[q]) <= 1e-8 * (1 + 1e-9) * np.linalg.norm(B[q])


GROUP = [("ico4", 100, 8), ("torus96", 200, 5), ("pc20k", 500, 3), ("hubs_big", 1000, 8), ("ico3", 100, 1),
         ("torus256", 1000, 8), ("flat", 100, 0), ("pc4k", 200, 7)]


def _group(seed=5):
    import paper_2307_04886_amd as g
    from paper_2307_04886_amd.binding import from_problem
    g.library()
    hs, Bs = [], []
    for i, (name, minc, nrhs) in enumerate(GROUP):
        prob = problem(name)
        h, _ = from_problem(prob, g.default_options(min_coarse_points=minc))
        B = rhs_block(prob, nrhs, seed=seed + i) if nrhs else np.zeros((0, prob.n))
        if name == "pc4k":
            B[2] = 0.0                                   # a zero right-hand side inside a member
        hs.append(h)
        Bs.append(torch.from_numpy(np.ascontiguousarray(B)).cuda())
    return hs, Bs


@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_grouped_solve_equals_batched_solves(precision):
    """One grouped CG over 8 hierarchies (block-ordered levels, hubs, point clouds,
    1 to 8 right-hand sides, a member without any, a zero right-hand side): every
    member's solutions, iteration counts and residuals equal gmg_solve_pcg_batched
    on that hierarchy alone, bit for bit."""
    _say(f"[gpu] grouped CG {precision} over {len(GROUP)} hierarchies")
    from paper_2307_04886_amd.binding import solve_pcg_grouped
    hs, Bs = _group()
    Xs, infos, sts, st = solve_pcg_grouped(hs, Bs, tol=1e-8, precision=precision)
    assert st == 0 and all(v == 0 for v in sts)
    for h, B, X, inf, (name, _, nrhs) in zip(hs, Bs, Xs, infos, GROUP):
        if nrhs == 0:
            assert X.shape[0] == 0 and inf == []
            continue
        Xr, infr, str_ = h.solve_pcg_batched(B, tol=1e-8, precision=precision)
        assert str_ == 0
        assert torch.equal(X, Xr), name
        for a, b in zip(inf, infr):
            assert (a.iterations, a.converged, a.rel_residual) == (b.iterations, b.converged, b.rel_residual), name
        _say(f"[gpu]   {name}: {nrhs} rhs, iterations {[a.iterations for a in inf]}")


def test_grouped_solve_cap_and_guesses():
    """Iteration cap: members that stop unconverged report it and match the
    per-hierarchy call with the same cap; initial guesses are honoured."""
    _say("[gpu] grouped CG with a cap and initial guesses")
    from paper_2307_04886_amd.binding import solve_pcg_grouped
    hs, Bs = _group(seed=9)
    X0 = [torch.from_numpy(np.random.default_rng(i).uniform(-1, 1, tuple(B.shape))).cuda() for i, B in enumerate(Bs)]
    Xs, infos, sts, st = solve_pcg_grouped(hs, Bs, [x.clone() for x in X0], tol=1e-12, max_iters=3, precision="f32")
    assert st == 1
    for h, B, x0, X, inf, s_m, (name, _, nrhs) in zip(hs, Bs, X0, Xs, infos, sts, GROUP):
        if nrhs == 0:
            continue
        Xr, infr, str_ = h.solve_pcg_batched(B, x0.clone(), tol=1e-12, max_iters=3, precision="f32")
        assert s_m == str_ and torch.equal(X, Xr), name
        assert [a.iterations for a in inf] == [b.iterations for b in infr]


def test_grouped_solve_errors():
    _say("[gpu] grouped CG errors")
    import paper_2307_04886_amd as g
    from paper_2307_04886_amd.binding import solve_pcg_grouped
    hs, Bs = _group()
    with pytest.raises(g.GMGError) as e:                  # the same hierarchy twice
        solve_pcg_grouped([hs[0], hs[0]], [Bs[0], Bs[0]])
    assert e.value.status == -1
    with pytest.raises(g.GMGError) as e:                  # more than 8 right-hand sides
        solve_pcg_grouped([hs[0]], [torch.cat([Bs[0], Bs[0]])])
    assert e.value.status == -1
    bad = Bs[1].clone()
    bad[0, 3] = float("nan")
    with pytest.raises(g.GMGError) as e:
        solve_pcg_grouped(hs[:2], [Bs[0], bad])
    assert e.value.status == -1
    assert solve_pcg_grouped([], [])[3] == 0


def test_many_meshes_grouped_form():
    """The many-mesh driver's grouped form gives the bits of its per-mesh form."""
    _say("[gpu] many meshes, grouped form")
    import paper_2307_04886_amd as g
    from paper_2307_04886_amd.batch import solve_many
    g.library()
    batch = synth.config_batched(count=6, hi=40_000)
    systems = []
    for prob, B in batch:
        t = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in
             (prob.points, prob.edges, prob.indptr, prob.indices, prob.data)]
        systems.append(tuple(t) + (torch.from_numpy(B).cuda(),))
    per = solve_many(systems, streams=4)
    grp = solve_many(systems, streams=4, form="grouped")
    for (xa, ia, sa), (xb, ib, sb) in zip(per, grp):
        assert sa == sb == 0
        assert torch.equal(xa, xb)
        assert [i.iterations for i in ia] == [i.iterations for i in ib]


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("name,opt", [("ico4", dict(min_coarse_points=40, block_min_rows=20)),
                                      ("pc4k", dict(min_coarse_points=100, block_min_rows=100)),
                                      ("torus96", dict(min_coarse_points=200, block_min_rows=100, nu_pre=1)),
                                      ("pc20k", dict(min_coarse_points=600, block_min_rows=600)),
                                      ("pc100k", {})])
def test_batched_block_sweeps(name, opt, precision):
    """The block sweeps of 8 right-hand sides (small and large blocks, one and two
    rows per lane group) and the batched coarsest solve, bit for bit against the
    single-vector cycle, alone and grouped."""
    _say(f"[gpu] batched block sweeps {name} {opt} {precision}")
    from paper_2307_04886_amd.binding import from_problem, default_options, solve_pcg_grouped
    prob = problem(name)
    gpu, _ = from_problem(prob, default_options(**opt))
    assert any(gpu.sizes(l)["blocks"] for l in range(gpu.num_levels))
    R = np.random.default_rng(21).uniform(-1, 1, (8, prob.n))
    Z = gpu.precondition_batched(torch.from_numpy(R).cuda(), precision=precision).cpu().numpy()
    for q in range(8):
        z = gpu.precondition(torch.from_numpy(R[q].copy()).cuda(), precision=precision).cpu().numpy()
        assert_same_bits(z, Z[q], f"{name} {precision} right-hand side {q}")
    B = torch.from_numpy(rhs_block(prob, 8)).cuda()
    X, infos, st = gpu.solve_pcg_batched(B, precision=precision)
    other, _ = from_problem(problem("ico4"), default_options())
    Xs, ginfos, sts, _ = solve_pcg_grouped([other, gpu], [torch.from_numpy(rhs_block(problem("ico4"), 3)).cuda(), B],
                                           precision=precision)
    assert st == 0 and sts == [0, 0]
    assert_same_bits(X.cpu().numpy(), Xs[1].cpu().numpy(), f"{name} {precision} grouped")
    assert [i.iterations for i in infos] == [i.iterations for i in ginfos[1]]
