"""GPU parity of the rows beyond one iteration: worst-W signal set (Algorithm 2 step 3),
base initialisation (eq. (5)), new-base training on a signal set (Algorithm 2 steps 1, 3),
squared-error total (Section 4), and the growth step composed from them."""
import numpy as np
import pytest

import paper_1412_4944_amd as sbo
import sbo_synth as synth
from oracle import sbo_oracle as orc
from gpu_util import Sbo, compare_assigned_code, compare_Q, ORTHO_TOL

pytestmark = pytest.mark.gpu


def _problem(name, m=None, **kw):
    if name in synth.CONFIGS:
        return synth.generate(synth.CONFIGS[name], m=m)
    return synth.generate(synth.custom(name, m=m, **kw))


# ------------------------------------------------------------------ worst-W set
@pytest.mark.parametrize("m", [1, 63, 2048, 2049, 5000, 70001])
def test_worst_set_bit_exact(m):
    rng = np.random.default_rng(41 + m)
    err = (rng.random(m) ** 4).astype(np.float32)
    if m >= 63:
        err[rng.integers(0, m, m // 7)] = err[3]          # many exact ties at one value
        err[rng.integers(0, m, m // 9)] = 0.0             # and at zero
    print(f"case m={m}", flush=True)
    with Sbo(16, 2, 2, max(m, 16)) as g:
        for W in sorted({1, min(m, 2), min(m, 17), max(1, m // 3), max(1, m - 1), m}):
            ids = g.worst(err, W)
            ref = orc.o_worst(err, W)
            assert np.array_equal(ids, ref), f"m={m} W={W}: {np.sum(ids != ref)} ids differ"
        total = g.sqerr(err)
    assert abs(total - err.astype(np.float64).sum()) <= 1e-12 * max(total, 1e-300)


@pytest.mark.parametrize("m", [2, 8191, 8192, 8193, 16384, 16385, 32768, 32769])
def test_worst_set_at_the_sizes_of_its_kernels(m):
    """One workgroup up to 32768 entries, 8, 16 or 32 of them to a lane; infinities, both zeros and runs of ties.  And the
    error total, by one workgroup up to 16384."""
    rng = np.random.default_rng(43 + m)
    err = rng.standard_normal(m).astype(np.float32) ** 2
    err[rng.integers(0, m, m // 3)] = err[m // 2]
    err[::97] = 0.0
    err[1::97] = -0.0
    err[m - 1] = np.inf
    # descending by the order of the bits (-0 below +0), ascending index among equals
    bits = err.view(np.uint32).astype(np.int64)
    order = np.argsort(-np.where(bits >> 31, 0xffffffff - bits, bits + 0x80000000), kind="stable")
    print(f"case m={m}", flush=True)
    with Sbo(16, 2, 2, max(m, 16)) as g:
        for W in sorted({1, m // 2, m // 2 + 1, m - 1, m}):
            assert np.array_equal(g.worst(err, W), np.sort(order[:W])), f"m={m} W={W}"
        err[m - 1] = 1.0
        assert abs(g.sqerr(err) - err.astype(np.float64).sum()) <= 1e-12 * err.astype(np.float64).sum()


@pytest.mark.parametrize("n", [1, 4096, 4097])
def test_new_base_error_total_at_the_sizes_of_its_kernels(n):
    """The error total of a round over a listed set, by one workgroup up to 4096 signals: the sum of the set's errors."""
    pr = synth.generate(synth.custom("sq", p=16, K=2, m=6000, s0=3, snr_db=20.0))
    ids = np.random.default_rng(71).permutation(6000)[:n].astype(np.int32)
    with Sbo(16, 2, 3, 6000) as g:
        Q, supp, coef, err, sq = g.new_base(pr.Y, ids, 1)
        total = err[ids].astype(np.float64).sum()
    assert abs(sq[0] - total) <= 1e-12 * max(total, 1e-300)


def test_worst_set_all_equal_and_real_residuals():
    pr = _problem("patch8", m=9000)
    cfg = pr.cfg
    _b, _s, _c, err, _E = orc.o_code(pr.Y, pr.D_init, cfg.s0)
    err32 = err.astype(np.float32)
    with Sbo(cfg.p, cfg.K, cfg.s0, 9000) as g:
        for W in (1, 256, 4500):
            assert np.array_equal(g.worst(err32, W), orc.o_worst(err32, W))
        flat = np.full(9000, 0.25, np.float32)            # every entry ties: the first W indices
        assert np.array_equal(g.worst(flat, 1000), np.arange(1000))
        neg = err32.copy()
        neg[::5] = -neg[::5]                              # negative values order below every positive one
        assert np.array_equal(g.worst(neg, 3000), orc.o_worst(neg, 3000))


# ------------------------------------------------------------- base initialisation
def _check_init_base(Y, ids, Qg, svg):
    """Gap-aware comparison with the oracle: an eigenvector of the Gram matrix computed in
    fp32 moves by about (rounding of G) / (gap to the nearest other eigenvalue)."""
    p = Y.shape[1]
    Qo, svo = orc.o_init_base(Y, ids)
    lam_o, lam_g = svo ** 2, svg.astype(np.float64) ** 2
    lmax = lam_o[0]
    assert np.abs(lam_g - lam_o).max() <= 2e-5 * lmax, f"eigenvalues off by {np.abs(lam_g - lam_o).max() / lmax:.2e}"
    assert (np.diff(svg) <= 0).all(), "singular values not descending"
    Q = Qg.astype(np.float64)
    assert np.abs(Q @ Q.T - np.eye(p)).max() <= ORTHO_TOL
    sub = np.asarray(Y, np.float64)[ids].T
    G = sub @ sub.T
    H = Q @ G @ Q.T                                       # must be diag(lambda)
    assert np.abs(H - np.diag(np.diag(H))).max() <= 2e-5 * lmax, "atoms do not diagonalise the Gram matrix"
    checked, worst = 0, 0.0
    for k in range(p):
        gap = np.min(np.abs(np.delete(lam_o, k) - lam_o[k])) / lmax
        tol = 2e-5 / max(gap, 1e-30)
        if tol > 1e-2:
            continue                                      # direction not determined at fp32 (valid by the checks above)
        d = min(np.abs(Q[k] - Qo[k]).max(), np.abs(Q[k] + Qo[k]).max())
        assert d <= tol, f"atom {k}: off by {d:.2e}, gap {gap:.2e}"
        worst = max(worst, d)
        checked += 1
    return checked, worst


@pytest.mark.parametrize("name,kw,n", [("tiny", dict(), 300), ("patch8", dict(m=6000), 2500),
                                       ("patch8", dict(m=3000), 40), ("p32", dict(p=32, K=3, m=900, s0=4), 777),
                                       ("p256", dict(p=256, K=2, m=2600, s0=12, snr_db=25.0), 2300)])
def test_init_base_matches_oracle(name, kw, n):
    pr = _problem(name, **kw)
    cfg = pr.cfg
    m = pr.Y.shape[0]
    rng = np.random.default_rng(43)
    ids = np.sort(rng.choice(m, n, replace=False)).astype(np.int32)
    # give the set a decaying spectrum (as image patches have) so that the gaps are resolvable
    Y = pr.Y.astype(np.float64) * np.linspace(2.0, 0.3, cfg.p)[None, :]
    Y = Y.astype(np.float32)
    print(f"case {name}: p={cfg.p} m={m} n={n}", flush=True)
    with Sbo(cfg.p, cfg.K, cfg.s0, m) as g:
        Qg, svg = g.init_base(Y, ids)
        Q2, sv2 = g.init_base(Y, ids)
    assert np.array_equal(Qg, Q2) and np.array_equal(svg, sv2), "not bitwise repeatable"
    checked, worst = _check_init_base(Y, ids, Qg, svg)
    print(f"  {checked}/{cfg.p} atoms compared, worst {worst:.2e}", flush=True)
    if n >= cfg.p:
        assert checked >= cfg.p // 4


@pytest.mark.parametrize("p", [16, 32, 64, 256])
@pytest.mark.parametrize("kind", ["noise", "equal", "pairs", "zero", "scaled"])
def test_init_base_spectra(p, kind):
    """Spectra at both ends of what the tridiagonal eigenvectors take: well separated ones (noise, also far from
    unit scale), and equal, pairwise equal and vanishing eigenvalues, which the Jacobi kernels have to finish."""
    rng = np.random.default_rng(47 + p)
    n = p if kind in ("equal", "pairs") else 3 * p
    if kind in ("noise", "scaled"):
        Y = rng.standard_normal((n, p)) * (1e9 if kind == "scaled" else 1.0)
    else:
        Y = np.zeros((n, p))
        if kind != "zero":
            Y[np.arange(p), np.arange(p)] = 1.0 if kind == "equal" else 1.0 + np.arange(p) // 2
    Y = Y.astype(np.float32)
    ids = np.arange(n, dtype=np.int32)
    print(f"case p={p} {kind}", flush=True)
    with Sbo(p, 2, 4, n) as g:
        Qg, svg = g.init_base(Y, ids)
        if kind == "zero":
            assert (svg == 0).all() and np.abs(Qg @ Qg.T - np.eye(p)).max() <= ORTHO_TOL
            return
        _check_init_base(Y, ids, Qg, svg)


@pytest.mark.parametrize("p", [16, 32, 64, 256])
@pytest.mark.parametrize("decades", [1, 2, 3, 4])
@pytest.mark.parametrize("across", [False, True], ids=["along", "across"])
def test_init_base_falling_spectra(p, decades, across):
    """Amplitudes that fall, as those of image patches do.  Along the coordinates every entry of the Gram matrix is
    known to a rounding of sqrt(G_ii G_jj), and the eigenvectors have to be that good: Q G Q^T off its diagonal by
    that much of sqrt(lambda_i lambda_j); across them, of the largest eigenvalue.  Bounds: a rounding for each of the
    two vectors and some more for the fp32 sums of the Gram matrix, 8 * 2^-24 in all; where the matrix was left to the
    Jacobi kernels, what their sweeps add up to, up to fourteen of p rotations, which round the columns of two matrices:
    2 * 2^-24 sqrt(14 p)."""
    rng = np.random.default_rng(73 + p + decades)
    n = 4 * p
    Y = rng.standard_normal((n, p)) * np.logspace(0, -decades, p)
    if across:
        Y = Y @ synth.random_onb(rng, p)
    Y = Y.astype(np.float32)
    ids = np.arange(n, dtype=np.int32)
    print(f"case p={p} decades={decades} across={across}", flush=True)
    with Sbo(p, 2, 4, n) as g:
        Qg, svg = g.init_base(Y, ids)
        sweeps = sbo.sbo_svd_sweeps(g.ctx, 2)[0]
    _check_init_base(Y, ids, Qg, svg)
    G = Y.astype(np.float64).T @ Y.astype(np.float64)
    Q = Qg.astype(np.float64)
    H = Q @ G @ Q.T
    lam = np.linalg.eigvalsh(G)[::-1]
    off = np.abs(H - np.diag(np.diag(H))) / (lam[0] if across else np.sqrt(np.outer(lam, lam)))
    print(f"  off the diagonal {off.max():.1e}, sweeps {sweeps}", flush=True)
    assert off.max() <= (8 * 2.0 ** -24 if sweeps == 0 else 2 * 2.0 ** -24 * np.sqrt(14 * p))
    assert decades > 2 or sweeps == 0, "left to the Jacobi kernels"


# ------------------------------------------------------------------- new base
@pytest.mark.parametrize("name,kw,n,R", [("tiny", dict(), 400, 3), ("patch8", dict(m=5000), 1800, 3),
                                         ("p256", dict(p=256, K=2, m=1200, s0=12, snr_db=25.0), 700, 2)])
def test_new_base_rounds_teacher_forced(name, kw, n, R):
    """Each round from the oracle's orthobase (rounded to fp32): codes of the set's signals
    against the oracle's, the updated orthobase against the oracle's update from the GPU's
    own codes; rows outside the set untouched."""
    pr = _problem(name, **kw)
    cfg = pr.cfg
    m = pr.Y.shape[0]
    rng = np.random.default_rng(44)
    ids = np.sort(rng.choice(m, n, replace=False)).astype(np.int32)
    sub = pr.Y[ids]
    zeros = np.zeros(n, np.int32)
    print(f"case {name}: p={cfg.p} m={m} n={n} R={R}", flush=True)
    Q = orc.o_init_base(pr.Y, ids)[0]
    with Sbo(cfg.p, cfg.K, cfg.s0, m) as g:
        for r in range(R):
            Q32 = Q.astype(np.float32)
            so, co, eo = orc.o_train_rounds(sub, zeros, Q32[None], cfg.s0, 1)[1]
            Qg, sg, cg, eg, sq = g.new_base(pr.Y, ids, 1, Q0=Q32)
            outside = np.setdiff1d(np.arange(m), ids)
            assert (sg[outside] == -7).all() and np.isnan(eg[outside]).all(), "rows outside the set written"
            sg, cg, eg = sg[ids], cg[ids], eg[ids]
            # supports bit-exact except below the near-tie gap, exempt codes valid in fp64
            frac = compare_assigned_code(sub, Q32[None], zeros, cfg.s0, (so, co, eo), (sg, cg, eg))
            assert abs(sq[0] - eg.astype(np.float64).sum()) <= 1e-9 * sq[0] + 1e-30
            Dn, M = orc.o_update(sub, zeros, sg, cg, Q32[None])
            w = compare_Q(Qg[None], Dn, M, np.array([True]))
            print(f"  round {r}: exempt fraction {frac:.5f}, worst dQ {w:.2e}", flush=True)
            Q = orc.o_train_rounds(sub, zeros, Q32[None], cfg.s0, 1)[0][0]


@pytest.mark.parametrize("name,kw,n,R", [("patch8", dict(m=5000), 2000, 5),
                                         ("p256", dict(p=256, K=2, m=1500, s0=12, snr_db=25.0), 900, 3)])
def test_new_base_free_running(name, kw, n, R):
    """Initialisation + R rounds in one call: orthonormal result, error of the rounds never
    increasing and close to the oracle's own run (near-tie choices may differ)."""
    pr = _problem(name, **kw)
    cfg = pr.cfg
    m = pr.Y.shape[0]
    ids = np.sort(np.random.default_rng(45).choice(m, n, replace=False)).astype(np.int32)
    with Sbo(cfg.p, cfg.K, cfg.s0, m) as g:
        Qg, _s, _c, _e, sq = g.new_base(pr.Y, ids, R)
        Q2, *_rest = g.new_base(pr.Y, ids, R)
    assert np.array_equal(Qg, Q2), "not bitwise repeatable"
    Q = Qg.astype(np.float64)
    assert np.abs(Q @ Q.T - np.eye(cfg.p)).max() <= ORTHO_TOL
    assert (np.diff(sq) <= 1e-6 * sq[0]).all(), f"error increased over the rounds: {sq}"
    _Qo, sqo = orc.o_new_base(pr.Y, ids, cfg.s0, R)
    print(f"  gpu {sq}\n  oracle {sqo}", flush=True)
    assert np.abs(sq - sqo).max() <= 2e-3 * sqo[0]


@pytest.mark.parametrize("p,m,P0,arith", [(16, 900, 300, "f16x2"), (64, 1500, 500, "f16x2"), (256, 2100, 700, "f16x2"),
                                          (256, 2100, 700, "f32"), (256, 1000, 400, "f16x2")])
def test_learn_initial_sets_as_one_batch(p, m, P0, arith):
    """sbo_learn trains its initial orthobases as one batch (at p = 256 with the codes by position, and one after the
    other where 3 P0 > m): the same as sbo_new_base on each set, also where the sets share signals."""
    pr = synth.generate(synth.custom(f"batch_p{p}", p=p, K=3, m=m, s0=4, snr_db=20.0))
    rng = np.random.default_rng(61)
    sets = np.stack([np.sort(rng.choice(m, P0, replace=False)) for _ in range(3)]).astype(np.int32)
    sets[2] = sets[0]
    with Sbo(p, 3, 4, m, arith=arith) as g:
        t = g.torch
        D = t.zeros((3, p, p), dtype=t.float32, device=g.dev)
        sbo.sbo_learn(g.ctx, g.dev_f32(pr.Y), D, g.dev_i32(sets), 3, 100, 3, 0.0, *g.outputs(m))
        t.cuda.synchronize()
        D = D.cpu().numpy()
        assert np.array_equal(D[0], D[2])
        for j in range(3):
            Q = g.new_base(pr.Y, sets[j], 3)[0]
            np.testing.assert_allclose(D[j], Q, atol=2e-5)


@pytest.mark.parametrize("p", [16, 32, 64, 256])
def test_learn_more_initial_sets_than_the_eigenvectors_have_room_for(p):
    """The scratch of the eigenvectors is that of the accumulation's pieces, which small sets have few of: the initial
    orthobases of sbo_learn in several goes, each as sbo_new_base makes it."""
    K0 = 7 if p == 256 else 19
    P0 = min(2 * p, 300)
    m = K0 * P0
    pr = synth.generate(synth.custom(f"room_p{p}", p=p, K=2, m=m, s0=4, snr_db=20.0))
    sets = np.random.default_rng(67).permutation(m).reshape(K0, P0).astype(np.int32)
    with Sbo(p, K0, 4, m) as g:
        t = g.torch
        D = t.zeros((K0, p, p), dtype=t.float32, device=g.dev)
        sbo.sbo_learn(g.ctx, g.dev_f32(pr.Y), D, g.dev_i32(sets), 1, 100, K0, 0.0, *g.outputs(m))
        t.cuda.synchronize()
        D = D.cpu().numpy()
        for j in range(K0):
            np.testing.assert_allclose(D[j], g.new_base(pr.Y, sets[j], 1)[0], atol=2e-5)


@pytest.mark.parametrize("p,m", [(16, 700), (256, 1200)])
def test_learn_stops_on_the_error(p, m):
    """The worst-W set is prepared before the host knows whether it is wanted: a run that stops on the error returns
    what one without room to grow does, and the context's next run is a first one."""
    pr = synth.generate(synth.custom(f"stop_p{p}", p=p, K=3, m=m, s0=4, snr_db=20.0))
    sets = np.arange(2 * 300, dtype=np.int32).reshape(2, 300)
    with Sbo(p, 4, 4, m) as g:
        t = g.torch
        Y, ids = g.dev_f32(pr.Y), g.dev_i32(sets)

        def run(K_max, target):
            D, out = t.zeros((K_max, p, p), dtype=t.float32, device=g.dev), g.outputs(m)
            K, hist = sbo.sbo_learn(g.ctx, Y, D, ids, 2, 200, K_max, target, *out)
            return [K, np.asarray(hist), D[:K].cpu().numpy()] + [o.cpu().numpy() for o in out]

        want, free = run(2, 0.0), run(4, 0.0)
        assert (want[0], len(want[1]), free[0], len(free[1])) == (2, 1, 4, 3)
        for K, target in ((2, 1e9), (3, float(free[1][:2].mean())), (4, 0.0)):
            got = run(4, target)
            assert got[0] == K and len(got[1]) == K - 1
            np.testing.assert_allclose(got[1], free[1][:K - 1], rtol=1e-6)
            if K != 3:
                for a, b in zip(got, want if K == 2 else free):
                    np.testing.assert_allclose(a, b, atol=2e-5)


def test_learn_is_refused_under_capture():
    """The host decides inside sbo_learn: a capturing stream gets an error and nothing in its graph, and the context
    works as before."""
    p, m = 16, 600
    pr = synth.generate(synth.custom("capture", p=p, K=3, m=m, s0=3, snr_db=20.0))
    import torch
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream), Sbo(p, 3, 3, m) as g:
        Y, D, out = g.dev_f32(pr.Y), torch.zeros((3, p, p), device=g.dev), g.outputs(m)
        sets = g.dev_i32(np.arange(400).reshape(2, 200))
        args = (g.ctx, Y, D, sets, 2, 100, 3, 0.0, *out)
        K, hist = sbo.sbo_learn(*args)
        torch.cuda.synchronize()
        D1 = D.clone()
        D.zero_()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            D.add_(1.0)                                  # (something for the graph to hold)
            with pytest.raises(sbo.SboError) as e:
                sbo.sbo_learn(*args)
        assert e.value.code == sbo.binding.SBO_EHIP
        for n in (1, 2):
            graph.replay()
            torch.cuda.synchronize()
            assert (D == n).all()
        assert sbo.sbo_learn(*args) == (K, hist)
        torch.cuda.synchronize()
        assert torch.equal(D, D1)


@pytest.mark.parametrize("m", [32768, 32769])
def test_learn_grows_by_the_worst_set(m):
    """One growth step of sbo_learn on both sides of the line up to which its worst-W set comes from one workgroup:
    what sbo_code, sbo_worst, sbo_new_base, sbo_code and sbo_train_rounds make of the same initial orthobases."""
    p, s0, W, R = 16, 3, 700, 2
    pr = synth.generate(synth.custom("grow", p=p, K=3, m=m, s0=s0, snr_db=20.0))
    sets = np.random.default_rng(79).permutation(m)[:2 * 400].reshape(2, 400).astype(np.int32)
    with Sbo(p, 3, s0, m) as g:
        t = g.torch
        Y, D, out = g.dev_f32(pr.Y), t.zeros((3, p, p), dtype=t.float32, device=g.dev), g.outputs(m)
        _K, hist = sbo.sbo_learn(g.ctx, Y, D, g.dev_i32(sets), R, W, 2, 0.0, *out)
        D2 = D[:2].cpu().numpy()
        _K, hist = sbo.sbo_learn(g.ctx, Y, D, g.dev_i32(sets), R, W, 3, 0.0, *out)
        t.cuda.synchronize()
        D, err = D.cpu().numpy(), out[3].cpu().numpy()
        with Sbo(p, 2, s0, m) as g2:
            e2 = g2.code(pr.Y, D2)[3]
        Q = g.new_base(pr.Y, g.worst(e2, W), R)[0]
        D3 = np.concatenate([D2, Q[None]])
        Dr, _s, _c, er = g.train_rounds(pr.Y, g.code(pr.Y, D3)[0], D3, R)
    np.testing.assert_array_equal(D, Dr)
    np.testing.assert_array_equal(err, er)
    np.testing.assert_allclose(hist, [orc.rmse(e.astype(np.float64).sum(), p, m) for e in (e2, er)], rtol=1e-9)


def test_growth_step_reduces_error():
    """Algorithm 2 steps 3-4 composed from the entry points: worst-W set -> new orthobase ->
    appended to the dictionary -> recoding.  Every signal keeps its old blocks to choose
    from, so no residual may grow, and the worst set's total must drop."""
    pr = _problem("patch8", m=8000)
    cfg = pr.cfg
    m, W, R = 8000, 1024, 4
    with Sbo(cfg.p, cfg.K, cfg.s0, m) as g, Sbo(cfg.p, cfg.K + 1, cfg.s0, m) as g1:
        blk, supp, coef, err = g.code(pr.Y, pr.D_init)
        ids = g.worst(err, W)
        assert np.array_equal(ids, orc.o_worst(err, W))
        Qn, *_rest = g.new_base(pr.Y, ids, R)
        D1 = np.concatenate([pr.D_init, Qn[None]], axis=0)
        blk1, supp1, coef1, err1 = g1.code(pr.Y, D1)
    assert (err1 <= err * (1 + 1e-5) + 1e-6 * (pr.Y.astype(np.float64) ** 2).sum(1)).all()
    before, after = err[ids].astype(np.float64).sum(), err1[ids].astype(np.float64).sum()
    assert after < before
    assert (blk1[ids] == cfg.K).mean() > 0.2
    # the same step done by the oracle lands at the same error (near-tie choices may differ)
    eo = orc.o_code(pr.Y, pr.D_init, cfg.s0)[3]
    Qo, _sq = orc.o_new_base(pr.Y, orc.o_worst(eo.astype(np.float32), W), cfg.s0, R)
    e1o = orc.o_code(pr.Y, np.concatenate([pr.D_init.astype(np.float64), Qo[None]], axis=0), cfg.s0)[3]
    print(f"  worst-set error {before:.2f} -> {after:.2f} (oracle {e1o[ids].sum():.2f})", flush=True)
    assert abs(after - e1o[ids].sum()) <= 5e-3 * before
    # and the oracle agrees on the recoding with the grown dictionary
    from gpu_util import compare_code
    compare_code(pr.Y, D1, cfg.s0, orc.o_code(pr.Y, D1, cfg.s0), (blk1, supp1, coef1, err1))


# ------------------------------------------------------------- Algorithm 2 as a whole
@pytest.mark.parametrize("name,kw,K0,P0,R,W,K_max", [
    ("tiny", dict(), 2, 200, 2, 128, 5),
    ("patch8", dict(m=6000), 3, 600, 2, 512, 6),
])
def test_learn_against_oracle(name, kw, K0, P0, R, W, K_max):
    """The whole of Algorithm 2 free-running on both sides from the same signal sets: same
    number of orthobases, RMSE history never increasing and within 1 % of the oracle's
    (near-tie choices differ), orthonormal result; the final representation is re-derived
    by the oracle from the GPU's own dictionary; the stopping rule is honoured."""
    import torch
    import paper_1412_4944_amd as sbo
    pr = _problem(name, **kw)
    cfg = pr.cfg
    m, p, s0 = pr.Y.shape[0], cfg.p, cfg.s0
    rng = np.random.default_rng(46)
    sets = np.stack([np.sort(rng.choice(m, P0, replace=False)) for _ in range(K0)]).astype(np.int32)
    Do, blko, hist_o = orc.o_learn(pr.Y, s0, list(sets), R, W, K_max)
    print(f"case {name}: oracle history {hist_o}", flush=True)
    with Sbo(p, K_max, s0, m) as g:
        t, dev = g.torch, g.dev
        Yd = g.dev_f32(pr.Y)
        D = t.zeros((K_max, p, p), dtype=t.float32, device=dev)
        blk, supp, coef, err = g.outputs(m)
        Kf, hist = sbo.sbo_learn(g.ctx, Yd, D, g.dev_i32(sets), R, W, K_max, 0.0, blk, supp, coef, err)
        t.cuda.synchronize()
        Dg, blkg, errg = D.cpu().numpy(), blk.cpu().numpy(), err.cpu().numpy()
        hist = np.array(hist)
        print(f"  gpu history {hist}", flush=True)
        assert Kf == K_max == Do.shape[0] and hist.size == hist_o.size
        assert (np.diff(hist) <= 1e-6 * hist[0]).all()
        assert np.abs(hist - hist_o).max() <= 1e-2 * hist_o[0]
        for j in range(Kf):
            Q = Dg[j].astype(np.float64)
            assert np.abs(Q @ Q.T - np.eye(p)).max() <= ORTHO_TOL
        assert blkg.min() >= 0 and blkg.max() < Kf
        assert abs(hist[-1] - orc.rmse(errg.astype(np.float64).sum(), p, m)) <= 1e-9 * hist[0]
        # stopping rule: a target between two entries of the history stops right after the first below it
        D2 = t.zeros_like(D)
        target = 0.5 * (hist[1] + hist[2])
        Kf2, hist2 = sbo.sbo_learn(g.ctx, Yd, D2, g.dev_i32(sets), R, W, K_max, float(target), blk, supp, coef, err)
        t.cuda.synchronize()
        assert Kf2 == K0 + 2 and len(hist2) == 3 and np.array_equal(np.array(hist2), hist[:3])
        assert not t.isnan(D2[:Kf2]).any()
        # the context is back to its own block count and still works
        from gpu_util import compare_code
        frac = compare_code(pr.Y, Dg, s0, orc.o_code(pr.Y, Dg, s0), g.code(pr.Y, Dg))
        print(f"  coding with the learnt dictionary: exempt fraction {frac:.5f}", flush=True)


@pytest.mark.parametrize("name,kw,K0,P0,R,W,K_max", [
    ("patch8", dict(m=9000), 3, 700, 3, 600, 8),
    ("learn32", dict(p=32, K=6, m=7000, s0=4), 2, 500, 4, 400, 6),
    ("learn256", dict(p=256, K=3, m=4500, s0=12, snr_db=20.0), 2, 1200, 3, 800, 3),
])
def test_learn_quality(name, kw, K0, P0, R, W, K_max):
    """Algorithm 2 ends in another dictionary for every order of its sums, but in one as good: every entry of the
    RMSE history within 0.5 % of the oracle's (near-tie choices have been seen to move it by 0.1 %, another BLAS under
    the oracle by 0.01 %)."""
    import paper_1412_4944_amd as sbo
    pr = _problem(name, **kw)
    m, p, s0 = pr.Y.shape[0], pr.cfg.p, pr.cfg.s0
    rng = np.random.default_rng(47)
    sets = np.stack([np.sort(rng.choice(m, P0, replace=False)) for _ in range(K0)]).astype(np.int32)
    hist_o = orc.o_learn(pr.Y, s0, list(sets), R, W, K_max)[2]
    print(f"case {name}: oracle history {hist_o}", flush=True)
    with Sbo(p, K_max, s0, m) as g:
        D = g.torch.zeros((K_max, p, p), dtype=g.torch.float32, device=g.dev)
        blk, supp, coef, err = g.outputs(m)
        _K, hist = sbo.sbo_learn(g.ctx, g.dev_f32(pr.Y), D, g.dev_i32(sets), R, W, K_max, 0.0, blk, supp, coef, err)
        g.torch.cuda.synchronize()
    print(f"  gpu history {np.array(hist)}, off by {np.abs(np.array(hist) / hist_o - 1).max():.1e}", flush=True)
    np.testing.assert_allclose(hist, hist_o, rtol=5e-3)
