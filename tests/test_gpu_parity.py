"""GPU parity: the HIP path, called through the C-ABI, against the fp64 oracle on the
same seeded inputs.  Tolerances are the ones stated in tests/gpu_util.py."""
import numpy as np
import pytest

import sbo_synth as synth
from oracle import sbo_oracle as orc
from gpu_util import Sbo, compare_assigned_code, compare_code, compare_Q
import paper_1412_4944_amd as sbo

pytestmark = pytest.mark.gpu


def _problem(name, m=None, **kw):
    if name in synth.CONFIGS:
        return synth.generate(synth.CONFIGS[name], m=m)
    return synth.generate(synth.custom(name, m=m, **kw))


CODE_CASES = [
    ("tiny", dict()),
    ("patch8", dict(m=4096 + 77)),                       # several tiles + ragged tail
    ("headline", dict(m=3000)),
    ("p32", dict(p=32, K=6, m=1500, s0=4)),
    ("p32_oddK", dict(p=32, K=5, m=700, s0=16)),
    ("p16_oddK", dict(p=16, K=3, m=333, s0=2)),
    ("p16_full", dict(p=16, K=2, m=200, s0=16)),
    ("p16_s9", dict(p=16, K=4, m=257, s0=9)),
    ("p64_s1", dict(p=64, K=3, m=129, s0=1)),
    ("p64_s16", dict(p=64, K=4, m=640, s0=16)),
    ("p64_s5", dict(p=64, K=7, m=1000, s0=5)),
    ("K1", dict(p=64, K=1, m=100, s0=8)),
    ("m1", dict(p=64, K=4, m=1, s0=3)),
    ("p256", dict(p=256, K=3, m=333, s0=12, snr_db=25.0)),
    ("p256_s8", dict(p=256, K=2, m=150, s0=8, snr_db=25.0)),
    ("p256_s1", dict(p=256, K=2, m=70, s0=1, snr_db=25.0)),
]


ARITH = ["f32", "bf16x3", "screen", "f16x2"]     # the two ways the projection onto all K orthobases is multiplied out


@pytest.mark.parametrize("arith", ARITH)
@pytest.mark.parametrize("name,kw", CODE_CASES, ids=[c[0] for c in CODE_CASES])
def test_code_matches_oracle(name, kw, arith):
    pr = _problem(name, **kw)
    cfg = pr.cfg
    print(f"case {name} {arith}: p={cfg.p} K={cfg.K} m={pr.Y.shape[0]} s0={cfg.s0}", flush=True)
    with Sbo(cfg.p, cfg.K, cfg.s0, pr.Y.shape[0], arith=arith) as g:
        for D in (pr.D_init, pr.D_planted):
            o = orc.o_code(pr.Y, D, cfg.s0)
            out = g.code(pr.Y, D)
            # s0 = p keeps everything: all blocks tie exactly, so every signal is exempt
            frac = compare_code(pr.Y, D, cfg.s0, o, out,
                                max_exempt_frac=1.0 if cfg.s0 == cfg.p else 0.01)
            print(f"  exempt fraction {frac:.5f}", flush=True)


@pytest.mark.parametrize("p", [16, 64, 256])
@pytest.mark.parametrize("arith", ARITH)
def test_code_ties_zero_signal_and_duplicates(arith, p):
    # identical blocks (block tie -> lowest index), equal magnitudes (atom tie -> lowest
    # index), an all-zero signal; every expected value follows from the tie rules alone
    K, s0 = 4, 3
    rng = np.random.default_rng(3)
    Q = synth.random_onb(rng, p).T.astype(np.float32)
    D = np.stack([np.eye(p, dtype=np.float32), Q, np.eye(p, dtype=np.float32), Q])
    Y = np.zeros((70, p), np.float32)
    Y[0, [2, 5, 7, 9]] = [1.0, -1.0, 1.0, 1.0]          # four equal magnitudes, keep 2,5,7
    Y[1] = 0.0
    Y[2, [0, p - 1]] = [3.0, -3.0]                       # fewer non-zeros than s0
    Y[3:] = rng.standard_normal((67, p)).astype(np.float32)
    Y[40] = Y[39]                                        # duplicate signals
    o = orc.o_code(Y, D, s0)
    with Sbo(p, K, s0, 70, arith=arith) as g:
        blk, supp, coef, err = g.code(Y, D)
    assert blk[0] == 0 and supp[0].tolist() == [2, 5, 7] and coef[0].tolist() == [1.0, -1.0, 1.0]
    assert err[0] == 1.0
    assert blk[1] == 0 and supp[1].tolist() == [0, 1, 2] and (coef[1] == 0).all() and err[1] == 0
    assert blk[2] == 0 and supp[2].tolist() == [0, 1, p - 1] and coef[2].tolist() == [3.0, 0.0, -3.0]
    assert (blk[40], supp[40].tolist(), coef[40].tolist()) == (blk[39], supp[39].tolist(), coef[39].tolist())
    assert (blk < 2).all()                               # blocks 2,3 duplicate 0,1: lowest index wins
    compare_code(Y, D, s0, o, (blk, supp, coef, err), max_exempt_frac=0.05)


@pytest.mark.parametrize("s0", [1, 3, 8, 12, 16])
def test_code_p256_selection(s0):
    """p = 256 selects with 16 lanes to a signal: exact magnitude ties, zero signals and ragged blocks against the oracle,
    and the same signals as part of a larger set, where they share tiles with others."""
    p, K, m = 256, 4, 700
    rng = np.random.default_rng(53)
    D = np.stack([np.eye(p)] + [synth.random_onb(rng, p).T for _ in range(K - 1)]).astype(np.float32)
    Y = rng.standard_normal((2 * m, p)).astype(np.float32)
    Y[0] = 0.0
    Y[1:40] = rng.integers(-2, 3, size=(39, p))           # many ties in the first block
    Y[40] = 1.0
    print(f"case s0={s0}", flush=True)
    out = []
    for n in (m, 2 * m):
        with Sbo(p, K, s0, n) as g:
            out.append(g.code(Y[:n], D))
    a, b = out[0], [v[:m] for v in out[1]]
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    o = orc.o_code(Y[:m], D, s0)
    compare_code(Y[:m], D, s0, o, a)
    if a[0][40] == 0:
        assert a[1][40].tolist() == list(range(s0)) and (a[2][40] == 1.0).all()


@pytest.mark.parametrize("p,K,s0,m", [(64, 3, 5, 32768), (64, 8, 1, 33001), (64, 4, 8, 100003), (64, 1024, 12, 100003),
                                      (32, 5, 16, 32768), (32, 3, 2, 150001)])
def test_code_larger_sets_selection(p, K, s0, m):
    """From 32768 signals on the support is selected by workgroups that share a block, one to four tiles to a wavefront:
    601 signals (zero ones, exact ties) over and over, each copy the same and the first as the oracle has it."""
    n = 601
    rng = np.random.default_rng(57)
    D = np.stack([np.eye(p)] + [synth.random_onb(rng, p).T for _ in range(K - 1)]).astype(np.float32)
    base = rng.standard_normal((n, p)).astype(np.float32)
    base[0] = 0.0
    base[1:40] = rng.integers(-2, 3, size=(39, p))        # many ties in the first block
    base[40] = 1.0
    base[41:60] *= np.float32(1e-12)
    idx = np.arange(m) % n
    print(f"case p={p} K={K} s0={s0} m={m}", flush=True)
    with Sbo(p, K, s0, m) as g:
        out = g.code(base[idx], D)
        Y = base[idx]
        Y[70, p - 1] = np.inf
        inf = g.code(Y, D)
    first = [v[:n] for v in out]
    for x, y in zip(out[:3], first):
        assert np.array_equal(x, y[idx])
    # an infinite entry: all products of that signal are infinite (the identity's others 0 * inf), the others as before
    assert all(np.array_equal(np.delete(x, 70, 0), np.delete(y, 70, 0)) for x, y in zip(inf[:3], out))
    if inf[0][70] != 0:
        assert inf[1][70].tolist() == list(range(s0)) and np.isinf(inf[2][70]).all() and (p == s0 or np.isinf(inf[3][70]))
    # (a tile with a tie adds the up to p squares up in another order: each sum is off by at most p 2^-24 of itself)
    np.testing.assert_allclose(out[3], first[3][idx], rtol=2 * p * 2.0 ** -24)
    compare_code(base, D, s0, orc.o_code(base, D, s0), first)


@pytest.mark.parametrize("p,K,s0", [(64, 5, 8), (16, 3, 4), (256, 2, 12)])
@pytest.mark.parametrize("arith", ARITH)
def test_code_over_signal_scales_and_dynamic_range(arith, p, K, s0):
    """Coding does not depend on the scale of a signal (the fp16 arithmetic rescales every signal by
    a power of two, the others work on the values as they are): signals scaled by 1e-12 .. 1e12
    (squares stay inside the fp32 range), signals with one dimension 1e4 times the others, and a
    signal of a single non-zero entry."""
    rng = np.random.default_rng(91 + p)
    pr = _problem(f"scales_p{p}", p=p, K=K, m=700, s0=s0, snr_db=25.0)
    Y = pr.Y.copy()
    m = Y.shape[0]
    Y *= (10.0 ** rng.uniform(-12, 12, size=(m, 1))).astype(np.float32)
    Y[5::50, 3] *= 1e4
    Y[7] = 0.0
    Y[7, p - 2] = -2.5e-9
    D = pr.D_planted
    print(f"case {arith}: p={p} K={K} m={m} s0={s0}", flush=True)
    o = orc.o_code(Y, D, s0)
    with Sbo(p, K, s0, m, arith=arith) as g:
        out = g.code(Y, D)
    frac = compare_code(Y, D, s0, o, out, max_exempt_frac=0.01)
    print(f"  exempt fraction {frac:.5f}", flush=True)


SCREEN_EDGES = [                                         # both shapes, their borders and remainders; a table
                                                         # too large for 512 signals (the last two)
    (64, 1, 8, 1), (64, 9, 16, 65), (32, 5, 16, 193), (16, 7, 8, 63), (16, 1, 1, 64), (256, 3, 16, 129),
    (64, 3, 4, 52428), (64, 2, 6, 52429), (64, 119, 8, 85196), (64, 3, 8, 85197), (32, 7, 3, 86000 + 513), (16, 5, 8, 86016 + 31), (256, 2, 12, 86016 + 1),
    (64, 4, 3, 131072), (32, 5, 5, 131073), (16, 160, 3, 90001), (64, 130, 2, 86081),
]


@pytest.mark.parametrize("p,K,s0,m", SCREEN_EDGES)
@pytest.mark.parametrize("close", [False, True], ids=["apart", "close"])
def test_screened_block_choice(p, K, s0, m, close):
    """The screened choice at the edges of its shapes; with blocks that differ from one another by
    about 1e-5, nearly every signal has several candidates left to be resolved in full precision."""
    rng = np.random.default_rng(17 + p + K)
    if close:
        Q = synth.random_onb(rng, p)
        D = np.stack([np.linalg.qr(Q + 1e-5 * rng.standard_normal((p, p)))[0] for _ in range(K)])
        D *= np.sign(np.einsum("kij,ij->kj", D, Q))[:, None, :]
        D = np.ascontiguousarray(D.transpose(0, 2, 1)).astype(np.float32)
    else:
        D = np.stack([synth.random_onb(rng, p).T for _ in range(K)]).astype(np.float32)
    Y = rng.standard_normal((m, p)).astype(np.float32)
    Y[m // 2] = 0.0
    rows = np.unique(np.r_[0:min(m, 300), max(0, m - 600):m])
    o = orc.o_code(Y[rows], D, s0)
    outs = []
    for arith in ["f16x2"] if p == 256 else ["f32", "bf16x3", "f16x2"]:
        print(f"case {arith}: p={p} K={K} m={m} s0={s0} close={close}", flush=True)
        with Sbo(p, K, s0, m, arith=arith) as g:
            out = g.code(Y, D)
        compare_code(Y[rows], D, s0, o, tuple(a[rows] for a in out), max_exempt_frac=1.0 if close else 0.01)
        outs.append(out[0])
    for blk in outs:
        assert blk[m // 2] == 0 and blk.min() >= 0 and blk.max() < K
        assert close or (blk != outs[0]).mean() < 0.01


@pytest.mark.parametrize("K,m", [(256, 3000), (200, 20001), (257, 3000), (32, 131072), (32, 131073), (1, 262145)])
def test_group_scan_inside_scatter(K, m):
    """Both sides of the rule by which the scan over the chunks is part of the scatter; twice on one
    context (the histograms are set back)."""
    rng = np.random.default_rng(K + m)
    with Sbo(16, K, 2, m) as g:
        for _ in range(2):
            blk = rng.integers(0, K, m).astype(np.int32)
            counts, offsets, perm = g.group(blk)
            assert np.array_equal(counts, np.bincount(blk, minlength=K))
            assert np.array_equal(offsets, np.r_[0, np.cumsum(counts)])
            assert np.array_equal(perm, np.argsort(blk, kind="stable"))


@pytest.mark.parametrize("K,m", [(4, 1024), (32, 5000), (128, 70001), (1, 100), (1000, 3000), (7, 1)])
def test_group_matches_oracle(K, m):
    rng = np.random.default_rng(K * 1000 + m)
    w = (np.arange(K) + 1.0) ** -1.1
    blk = rng.choice(K, size=m, p=w / w.sum()).astype(np.int32)
    if K > 3:
        blk[blk == 2] = 1                                # an empty block
    print(f"case K={K} m={m}", flush=True)
    with Sbo(64, K, 4, m) as g:
        counts, offsets, perm = g.group(blk)
    oc, oo, op = orc.o_group(blk, K)
    np.testing.assert_array_equal(counts, oc)
    np.testing.assert_array_equal(offsets, oo)
    np.testing.assert_array_equal(perm, op)


@pytest.mark.parametrize("p", [16, 32, 64])
@pytest.mark.parametrize("K,m", [(256, 1024), (256, 1025), (257, 1024), (1, 1024), (256, 1), (5, 513)])
def test_code_groups_small_sets_in_the_select_kernel(p, K, m):
    """Both sides of the rule by which sbo_code leaves the grouping of a small set to the select kernel (m <= 1024,
    K <= 256: at (256, 1024) its lists and the tiles fill LDS), on one context in turn with calls that group by a
    launch: what either leaves in the workspace is what the other needs."""
    pr = synth.generate(synth.custom(f"small_p{p}", p=p, K=K, m=max(m, 1100), s0=4, snr_db=20.0))
    Y, D = pr.Y[:m], pr.D_planted
    with Sbo(p, K, 4, pr.Y.shape[0]) as g:
        sbo.sbo_set_timing(g.ctx, 1)
        for n in (m, pr.Y.shape[0], m):
            out = g.code(pr.Y[:n], D)
            ms = sbo.sbo_stage_ms(g.ctx)
            assert (ms["group"] > 0) == (n > 1024 or K > 256)
            compare_code(pr.Y[:n], D, 4, orc.o_code(pr.Y[:n], D, 4), out)
        sbo.sbo_set_timing(g.ctx, 0)
        # the histograms of the choice are zero again: a grouping that adds to them, and one that counts itself
        D1, blk, supp, coef, err, sq = g.iterate(Y, D, 1)
        np.testing.assert_array_equal(blk, out[0])
        np.testing.assert_array_equal(supp, out[1])
        counts, offsets, perm = g.group(blk)
        oc, oo, op = orc.o_group(blk, K)
        np.testing.assert_array_equal(counts, oc)
        np.testing.assert_array_equal(perm, op)


@pytest.mark.parametrize("p,K,m,s0", [(64, 64, 1024, 8), (64, 65, 1024, 8), (64, 64, 512, 8), (64, 64, 513, 8), (64, 65, 500, 8),
                                      (32, 32, 1024, 4), (32, 33, 993, 4), (64, 32, 225, 8), (64, 3, 33, 16), (32, 64, 1000, 1),
                                      (32, 7, 500, 16), (16, 63, 1024, 8), (16, 5, 31, 3), (16, 1, 1, 2)])
@pytest.mark.parametrize("arith", ARITH)
def test_code_small_sets_without_screening(p, K, m, s0, arith):
    """Small sets (K <= 64, m <= 1024 and K m <= 32768) compare full-precision energies in the select kernel; in a larger set the same
    signals go through the screened choice.  Blocks and codes are the same, bit by bit; zero signals, ties between equal
    blocks and a near-random dictionary among them."""
    rng = np.random.default_rng(59 + p + K)
    pr = synth.generate(synth.custom(f"direct_p{p}", p=p, K=K, m=m, s0=s0, snr_db=15.0))
    Y, D = pr.Y.copy(), (pr.D_planted if K % 2 else pr.D_init).astype(np.float32)
    if K > 4:
        D[K - 1] = D[2]                                    # ties go to the lower block
    Y[m // 2] = 0.0
    Y[m // 3] *= 1e-20                                     # (squares underflow in fp32: not for the oracle)
    full = np.concatenate([Y, rng.standard_normal((1025 - m, p)).astype(np.float32)])
    print(f"case {arith}: p={p} K={K} m={m} s0={s0}", flush=True)
    with Sbo(p, K, s0, 1025, arith=arith) as g:
        for _ in range(2):
            a = g.code(Y, D)
            b = g.code(full, D)
            for x, y in zip(a, b):
                np.testing.assert_array_equal(x, y[:m])
    keep = np.arange(m) != (m // 3 if m > 1 else -1)
    compare_code(Y[keep], D, s0, orc.o_code(Y[keep], D, s0), tuple(x[keep] for x in a))


@pytest.mark.parametrize("p,K,m", [(16, 4, 1024), (32, 3, 1024), (64, 2, 1024), (64, 5, 257), (16, 2, 1)])
def test_iterate_groups_small_sets_in_the_select_kernel(p, K, m):
    """sbo_iterate on both sides of the rule (m <= 1024): filled up with zero signals, which go to the end of block 0 and
    add nothing, a set is grouped by a launch; codes and dictionary have to be the same, and what either leaves behind
    is what the other needs."""
    pr = synth.generate(synth.custom(f"small_it_p{p}", p=p, K=K, m=m, s0=4, snr_db=20.0))
    full = np.concatenate([pr.Y, np.zeros((1025 - m, p), np.float32)])
    with Sbo(p, K, 4, 1025) as g:
        for _ in range(2):
            a = g.iterate(pr.Y, pr.D_init, 3)
            b = g.iterate(full, pr.D_init, 3)
            np.testing.assert_array_equal(a[1], b[1][:m])
            np.testing.assert_array_equal(a[2], b[2][:m])
            np.testing.assert_allclose(a[3], b[3][:m], atol=2e-5 * np.abs(pr.Y).max())
            if m > 100:                                    # (every block of full rank)
                np.testing.assert_allclose(a[0], b[0], atol=2e-5)
            np.testing.assert_allclose(a[5], b[5], rtol=1e-5)
            counts, offsets, perm = g.group(a[1])
            np.testing.assert_array_equal(perm, orc.o_group(a[1], K)[2])


@pytest.mark.parametrize("p,K,m,s0", [(64, 16, 2049, 6), (64, 128, 32500, 5), (64, 129, 32500, 5), (64, 64, 69632, 8), (64, 65, 69632, 8),
                                      (64, 3, 131072, 1), (64, 3, 131073, 1), (64, 5, 81920, 3), (64, 5, 81921, 3), (32, 8, 131072, 2), (32, 9, 81921, 2), (16, 51, 81920, 2),
                                      (32, 7, 32767, 4), (32, 24, 32768, 7), (16, 5, 100003, 3),
                                      (16, 128, 2100, 16), (256, 16, 5041, 12), (256, 2, 65536, 16), (256, 2, 65537, 16),
                                      (256, 97, 4100, 3)])
@pytest.mark.parametrize("arith", ["f16x2", "f32"])
def test_code_lists_the_signals_of_a_tile_from_the_histograms(p, K, m, s0, arith):
    """sbo_code on both sides of its rule (2049 to 81920 signals, up to 8 blocks 131072, p = 256 65536, K <= 128, 9216 histogram entries), in turn
    with calls that group; filled up with zero signals, which all go to block 0, to a set that is grouped, the codes are the same."""
    if arith == "f32" and m > 40000:
        pytest.skip("one arithmetic is enough at these sizes")
    pr = synth.generate(synth.custom(f"clists_p{p}_K{K}", p=p, K=K, m=m, s0=s0, snr_db=20.0, zipf_s=1.2 if K > 20 else None))
    more = 140000 if p <= 64 else 70000
    full = np.concatenate([pr.Y, np.zeros((more - m, p), np.float32)])
    with Sbo(p, K, s0, more, arith=arith) as g:
        for _ in range(2):
            blk, supp, coef, err = g.code(pr.Y, pr.D_planted)
            blk2, supp2, coef2, err2 = (a[:m] for a in g.code(full, pr.D_planted))
            np.testing.assert_array_equal(blk, blk2)
            # (other sizes take other select kernels: the last bits of a coefficient may differ, and with them a tie)
            same = (supp == supp2).all(1)
            assert same.mean() > 0.999
            tol = 2e-6 * np.linalg.norm(pr.Y, axis=1)
            assert (np.abs(coef - coef2).max(1) <= tol)[same].all()
            assert (np.abs(err - err2) <= tol * np.linalg.norm(pr.Y, axis=1)).all()
        counts, _off, perm = g.group(blk)
        np.testing.assert_array_equal(perm, orc.o_group(blk, K)[2])
        np.testing.assert_array_equal(g.iterate(pr.Y, pr.D_planted, 1)[1], blk)    # (its histograms start from zero)


@pytest.mark.parametrize("p,K,m,s0", [(64, 16, 16384, 6), (64, 56, 32768, 8), (64, 57, 32768, 8), (64, 3, 32769, 5), (64, 2, 32767, 4),
                                      (32, 24, 511, 4), (32, 7, 513, 3), (32, 70, 20001, 4), (16, 4, 1024, 3), (16, 256, 4096, 2),
                                      (16, 257, 4000, 2), (16, 400, 1000, 2), (64, 1, 1, 8), (16, 5, 33, 3),
                                      (64, 32, 52428, 6), (64, 32, 52429, 6), (64, 128, 32768, 16), (32, 34, 131072, 4), (32, 34, 131073, 4),
                                      (16, 128, 32768, 3), (16, 129, 32767, 2), (16, 241, 4500, 2), (32, 5, 81920, 3), (16, 54, 81921, 3), (16, 8, 131072, 3), (32, 8, 131073, 4), (32, 9, 81920, 4)])
@pytest.mark.parametrize("skewed", [False, True], ids=["even", "skewed"])
def test_iterate_lists_the_signals_of_a_piece_from_the_histograms(p, K, m, s0, skewed):
    """Sets with few histogram entries, whose block choice does not need the lists, are not grouped in sbo_iterate.  A round on the blocks that it chose,
    which groups them, has the same sums in the same order, so every bit is the same; and the histograms are left zero."""
    pr = synth.generate(synth.custom(f"lists_p{p}_K{K}", p=p, K=K, m=m, s0=s0, snr_db=20.0, zipf_s=2.0 if skewed else None))
    with Sbo(p, K, s0, m) as g:
        for _ in range(2):
            Q, blk, supp, coef, err, _sq = g.iterate(pr.Y, pr.D_init, 1)[:6]
            Q2, supp2, coef2, err2 = g.train_rounds(pr.Y, blk, pr.D_init, 1)
            for a, b in ((Q, Q2), (supp, supp2), (coef, coef2), (err, err2)):
                np.testing.assert_array_equal(a, b)
        np.testing.assert_array_equal(g.code(pr.Y, pr.D_init)[0], blk)
        counts, _off, perm = g.group(blk)
        np.testing.assert_array_equal(counts, np.bincount(blk, minlength=K))
        np.testing.assert_array_equal(perm, orc.o_group(blk, K)[2])


UPDATE_CASES = [
    ("tiny", dict()),
    ("patch8", dict(m=4096 + 77)),
    ("headline", dict(m=20000)),
    ("p32", dict(p=32, K=6, m=3000, s0=4)),
    ("p16_oddK", dict(p=16, K=3, m=999, s0=2)),
    ("p256", dict(p=256, K=2, m=2500, s0=12, snr_db=25.0)),
]


@pytest.mark.parametrize("name,kw", UPDATE_CASES, ids=[c[0] for c in UPDATE_CASES])
def test_update_stages_match_oracle_teacher_forced(name, kw):
    pr = _problem(name, **kw)
    cfg = pr.cfg
    print(f"case {name}: p={cfg.p} K={cfg.K} m={pr.Y.shape[0]} s0={cfg.s0}", flush=True)
    blk, supp, coef, err, E = orc.o_code(pr.Y, pr.D_init, cfg.s0)
    coef32 = coef.astype(np.float32)
    Dn, M = orc.o_update(pr.Y, blk, supp, coef32, pr.D_init)
    counts = np.bincount(blk, minlength=cfg.K)
    with Sbo(cfg.p, cfg.K, cfg.s0, pr.Y.shape[0]) as g:
        Mg = g.accumulate(pr.Y, blk, supp, coef32)
        Mg2 = g.accumulate(pr.Y, blk, supp, coef32)
        assert np.array_equal(Mg, Mg2), "accumulation not bitwise repeatable"
        for j in range(cfg.K):
            scale = np.abs(M[j]).max() + 1e-30
            assert np.abs(Mg[j] - M[j]).max() <= 2e-5 * scale * max(1.0, np.sqrt(counts[j] / 64.0)), \
                f"M[{j}] off by {np.abs(Mg[j] - M[j]).max() / scale} rel"
        Dp = g.polar(M.astype(np.float32), pr.D_init, counts.astype(np.int32))
        w1 = compare_Q(Dp, Dn, M, counts > 0)
        Dg, cg = g.update(pr.Y, blk, supp, coef32, pr.D_init)
        np.testing.assert_array_equal(cg, counts)
        w2 = compare_Q(Dg, Dn, M, counts > 0)
        Dg2, _ = g.update(pr.Y, blk, supp, coef32, pr.D_init)
        assert np.array_equal(Dg, Dg2), "update not bitwise repeatable"
        print(f"  worst |Q - Q_oracle|: polar {w1:.2e}, update {w2:.2e}", flush=True)


def test_polar_rank_deficient_and_empty_blocks():
    p, K = 64, 5
    rng = np.random.default_rng(17)
    M = rng.standard_normal((K, p, p))
    M[1][:, :] = 0.0
    M[1][:5] = rng.standard_normal((5, p))               # rank 5: most atoms never used
    M[2][7] = 0.0                                        # one unused atom
    M[3] = 0.0                                           # all-zero but counted as non-empty
    u, s, vt = np.linalg.svd(M[4])
    M[4] = (u * np.geomspace(1, 1e-6, p)) @ vt           # ill-conditioned but full rank
    D_old = synth.random_dictionary(rng, K, p).astype(np.float32)
    counts = np.array([10, 10, 10, 10, 10], np.int32)
    counts0 = counts.copy()
    counts0[0] = 0
    with Sbo(p, K, 4, 16) as g:
        Dg = g.polar(M.astype(np.float32), D_old, counts0)
        np.testing.assert_array_equal(Dg[0], D_old[0])   # empty block keeps its basis
        Dg = g.polar(M.astype(np.float32), D_old, None)
    M32 = M.astype(np.float32).astype(np.float64)
    Dn = np.stack([orc.o_polar(M32[j]) for j in range(K)])
    compare_Q(Dg, Dn, M32, np.ones(K, bool))


@pytest.mark.parametrize("name,kw,iters", [("tiny", dict(), 5), ("patch8", dict(m=8192), 6),
                                           ("p32", dict(p=32, K=6, m=3000, s0=4), 4),
                                           ("p256", dict(p=256, K=2, m=2500, s0=12, snr_db=25.0), 3)])
@pytest.mark.parametrize("arith", ARITH)
def test_iterate_free_running(name, kw, iters, arith):
    pr = _problem(name, **kw)
    cfg = pr.cfg
    print(f"case {name} {arith}: p={cfg.p} K={cfg.K} m={pr.Y.shape[0]} s0={cfg.s0}", flush=True)
    Do, last, sq_o = orc.o_iterate(pr.Y, pr.D_init, cfg.s0, iters)
    with Sbo(cfg.p, cfg.K, cfg.s0, pr.Y.shape[0], arith=arith) as g:
        Dg, blk, supp, coef, err, sq = g.iterate(pr.Y, pr.D_init, iters)
        Dg2, *_rest, sq2 = g.iterate(pr.Y, pr.D_init, iters)
    assert np.array_equal(Dg, Dg2) and np.array_equal(sq, sq2), "iteration not bitwise repeatable"
    print("  oracle sqerr", sq_o, "\n  gpu    sqerr", sq, flush=True)
    assert (np.diff(sq) <= 1e-6 * sq[0]).all(), "error increased"
    np.testing.assert_allclose(sq, sq_o, rtol=1e-3)
    assert abs(sq[-1] - err.astype(np.float64).sum()) <= 1e-6 * sq[-1] + 1e-12
    for j in range(cfg.K):
        Q = Dg[j].astype(np.float64)
        assert np.abs(Q @ Q.T - np.eye(cfg.p)).max() <= 1e-5


def _home_case(p, K, s0, m, kind):
    """Signals planted in K orthobases at 20 dB, the dictionary 8 % off; or what takes the shortcuts of later iterations away."""
    rng = np.random.default_rng(p * 1000 + K * 10 + s0)
    base = np.linalg.qr(rng.standard_normal((K, p, p)))[0].transpose(0, 2, 1)
    if kind == "close":                        # every orthobase has a near twin: contenders for every signal
        twin = base[0::2][: (K + 1) // 2] + rng.standard_normal(((K + 1) // 2, p, p)) * (0.02 / np.sqrt(p))
        base = np.concatenate([base[0::2], np.linalg.qr(twin.transpose(0, 2, 1))[0].transpose(0, 2, 1)])[:K]
    blk = rng.integers(0, K, m)
    atoms = rng.random((m, p), dtype=np.float32).argpartition(s0, axis=1)[:, :s0]
    x = rng.uniform(0.5, 2.0, (m, s0)) * rng.choice([-1.0, 1.0], (m, s0))
    Y = np.zeros((m, p))
    for t in range(s0):
        Y += base[blk, atoms[:, t]] * x[:, t:t + 1]
    Y += rng.standard_normal((m, p)) * (0.1 * np.sqrt((Y ** 2).mean(1, keepdims=True)))
    Y *= np.exp(0.6 * rng.standard_normal((m, 1)))
    D = base + rng.standard_normal((K, p, p)) * (0.08 / np.sqrt(p))
    D = np.linalg.qr(D.transpose(0, 2, 1))[0].transpose(0, 2, 1)
    D *= np.sign((D * base).sum(2, keepdims=True))
    if kind == "odd signals":                  # too small to be screened, zero, unlike any orthobase
        Y[::401] = rng.standard_normal(Y[::401].shape)
        Y[7::5003] = 0.0
        Y[11::5003] *= 1e-21
    elif kind.startswith("noise"):             # every so many signals
        Y[::int(kind[5:])] = rng.standard_normal(Y[::int(kind[5:])].shape)
    elif kind == "random":
        D = np.linalg.qr(rng.standard_normal((K, p, p)))[0]
    elif kind == "unused":                     # a block that nobody takes and that is no orthobase
        D[K - 1] *= 0.25
    return Y.astype(np.float32), D.astype(np.float32)


HOME_CASES = [(64, 5, 8, 60001, "planted", "f16x2"), (64, 32, 6, 100003, "planted", "f16x2"), (64, 1, 3, 90000, "planted", "f16x2"),
              (64, 9, 4, 131149, "odd signals", "f32"), (64, 6, 8, 100003, "odd signals", "bf16x3"),
              (64, 8, 8, 100003, "random", "f16x2"), (64, 8, 5, 70001, "close", "f16x2"), (64, 40, 8, 100003, "close", "bf16x3"),
              (64, 7, 6, 90001, "unused", "f16x2"), (64, 70, 9, 53001, "planted", "f16x2"), (64, 6, 10, 60001, "planted", "f16x2"), (256, 5, 12, 90001, "planted", "f16x2"),
              (64, 33, 5, 100003, "noise40", "f16x2"), (64, 32, 8, 66001, "noise9", "bf16x3"), (64, 70, 3, 53001, "noise15", "f32"),
              (256, 4, 16, 86017, "close", "f16x2"), (256, 3, 5, 131072, "odd signals", "f16x2")]


@pytest.mark.parametrize("p,K,s0,m,kind,arith", HOME_CASES)
def test_iterations_in_one_call_are_iterations_in_calls_of_their_own(p, K, s0, m, kind, arith):
    """From the second iteration of a call on, large sets are coded in the order of the last grouping, starting from the
    block that a signal came from; every bit of the results is that of calls of one iteration, which know no such block."""
    Y, D = _home_case(p, K, s0, m, kind)
    n = 3
    with Sbo(p, K, s0, m, arith=arith) as g:
        t = g.torch
        Yd = g.dev_f32(Y)
        got = []
        for per_call in (n, 1):
            Dd, out = g.dev_f32(D), g.outputs(m)
            sq = t.zeros(n, dtype=t.float64, device=g.dev)
            for it in range(0, n, per_call):
                sbo.sbo_iterate(g.ctx, Yd, Dd, per_call, *out, sq[it:it + per_call])
            t.cuda.synchronize()
            got.append([a.cpu().numpy() for a in (*out, Dd, sq)])
        for name, a, b in zip(("blk", "supp", "coef", "err", "D", "sq"), *got):
            assert np.array_equal(a, b), (name, int((a != b).sum()))
        again = [a.cpu().numpy() for a in out]                     # and the context is as it was: the same once more
        Dd = g.dev_f32(D)
        sbo.sbo_iterate(g.ctx, Yd, Dd, n, *out, sq)
        t.cuda.synchronize()
        assert all(np.array_equal(a, b.cpu().numpy()) for a, b in zip(again, out))


@pytest.mark.parametrize("op,p,K,s0,m,kind,taken", [
    ("code", 64, 32, 8, 65537, "planted", "most"), ("code", 64, 64, 5, 100003, "planted", "most"), ("code", 64, 127, 8, 100003, "planted", "most"),
    ("code", 64, 33, 7, 66000, "random", "none"), ("code", 64, 64, 5, 100003, "noise10", "none"), ("code", 64, 64, 5, 100003, "noise33", "most"),
    ("iterate", 64, 32, 6, 100003, "noise12", "most"), ("code", 64, 32, 8, 53001, "planted", "no kernel"),
    ("iterate", 64, 32, 6, 100003, "planted", "most"), ("iterate", 64, 70, 9, 53001, "planted", "most"), ("iterate", 64, 8, 8, 100003, "random", "none"),
    ("iterate", 64, 9, 6, 90001, "unused", "none"), ("iterate", 64, 6, 10, 60001, "planted", "no kernel"),
    ("iterate", 64, 8, 6, 90001, "planted", "most"), ("iterate", 64, 7, 6, 90001, "planted", "no kernel"), ("iterate", 256, 2, 5, 90001, "planted", "most"), ("iterate", 256, 5, 12, 90001, "planted", "most")])
def test_short_cuts_of_the_block_choice_are_taken(op, p, K, s0, m, kind, taken):
    """Whether the workgroups decide by guessed blocks (sbo_code) and home blocks (the last iteration), which no result shows."""
    Y, D = _home_case(p, K, s0, m, kind)
    with Sbo(p, K, s0, m) as g:
        _out, n, n_taken = g.short_cuts(m, (lambda: g.code(Y, D)) if op == "code" else (lambda: g.iterate(Y, D, 3)))
    print(n, n_taken)
    assert (n == 0) == (taken == "no kernel")
    assert n_taken >= 0.9 * n if taken == "most" else n_taken == 0


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.nan])
def test_a_block_that_is_not_finite_is_no_orthobase(bad):
    """Which block a signal gets is then anybody's guess, but not by bounds that hold for orthobases only."""
    K, s0, m = 33, 5, 100003
    Y, D = _home_case(64, K, s0, m, "planted")
    D[7, 40, 3] = bad
    with Sbo(64, K, s0, m) as g:
        out, n, n_taken = g.short_cuts(m, lambda: g.code(Y, D))
    assert n > 0 and n_taken == 0
    assert (out[0] >= 0).all() and (out[0] < K).all()


@pytest.mark.parametrize("p,K,s0,m", [(16, 4, 3, 513), (16, 60, 2, 70001), (32, 16, 4, 131072), (64, 5, 8, 1), (64, 33, 8, 65537),
                                      (64, 128, 3, 32768)])
def test_update_lists_the_signals_of_a_piece_from_the_histograms(p, K, s0, m):
    """sbo_update without a grouping: blocks that nobody takes, one that takes half of the signals, choices that are no block
    (dropped).  The same bits as by the calls that group first."""
    rng = np.random.default_rng(m + K)
    Y = rng.standard_normal((m, p)).astype(np.float32)
    blk = np.where(rng.random(m) < 0.5, 1, rng.integers(-1, K, m)).astype(np.int32)
    blk[blk == 2] = 3
    supp = np.sort(rng.random((m, p), dtype=np.float32).argpartition(s0, axis=1)[:, :s0], axis=1).astype(np.int32)
    coef = rng.standard_normal((m, s0)).astype(np.float32)
    D = np.linalg.qr(rng.standard_normal((K, p, p)))[0].astype(np.float32)
    with Sbo(p, K, s0, m) as g:
        got, counts = g.update(Y, blk, supp, coef, D)
        again, _ = g.update(Y, blk, supp, coef, D)
        c, _offsets, _perm = g.group(blk)
        M = g.accumulate(Y, blk, supp, coef)
        want = g.polar(M, D, c)
    assert np.array_equal(counts, np.bincount(blk[blk >= 0], minlength=K)) and np.array_equal(counts, c)
    assert np.array_equal(got, again)
    # the same pieces, summed in the same order: the same bits
    assert np.array_equal(got, want), np.abs(got - want).max()


@pytest.mark.parametrize("p,K,m", [(16, 4, 81920), (32, 7, 66047), (64, 9, 51713), (64, 3, 33279), (16, 6, 515), (32, 5, 2559), (32, 8, 131071)])
@pytest.mark.parametrize("shift", [0, 1])
def test_pieces_of_rare_blocks_come_from_many_chunks(p, K, m, shift):
    """Blocks with a signal in every chunk, in every other one, in the last ones only or with three neighbours now and then, listed by
    chunks; the choices stand anywhere in memory.  The same bits as by the calls that group first."""
    rng = np.random.default_rng(m + K)
    blk = np.zeros(m, np.int32)
    blk[3::509] = 1
    blk[511::1024] = 2
    for j in range(3, K):
        blk[j * 40:: 300 + 213 * j] = j
        blk[j * 40 + 1:: 300 + 213 * j] = j
        blk[j * 40 + 2:: 300 + 213 * j] = j
    blk[m - 5:] = [K - 1, 0, 1, K - 1, 1]
    s0 = 4
    Y = rng.standard_normal((m, p)).astype(np.float32)
    supp = np.sort(rng.random((m, p), dtype=np.float32).argpartition(s0, axis=1)[:, :s0], axis=1).astype(np.int32)
    coef = rng.standard_normal((m, s0)).astype(np.float32)
    D = np.linalg.qr(rng.standard_normal((K, p, p)))[0].astype(np.float32)
    with Sbo(p, K, s0, m) as g:
        t = g.torch
        c, _offsets, _perm = g.group(blk)
        want = g.polar(g.accumulate(Y, blk, supp, coef), D, c)
        at = t.zeros(m + 4, dtype=t.int32, device=g.dev)[shift:shift + m]
        at.copy_(g.dev_i32(blk))
        Dd, counts = g.dev_f32(D), t.zeros(K, dtype=t.int32, device=g.dev)
        sbo.sbo_update(g.ctx, g.dev_f32(Y), at, g.dev_i32(supp), g.dev_f32(coef), Dd, counts)
        t.cuda.synchronize()
        assert np.array_equal(counts.cpu().numpy(), np.bincount(blk, minlength=K)) and np.array_equal(counts.cpu().numpy(), c)
        assert np.array_equal(Dd.cpu().numpy(), want)


@pytest.mark.parametrize("K,s0,m,kind,arith", [(32, 8, 65537, "planted", "bf16x3"), (16, 3, 70001, "planted", "f32"),
                                               (31, 6, 90001, "odd signals", "f16x2"), (100, 5, 53001, "close", "f16x2"),
                                               (64, 5, 131149, "close", "bf16x3"), (127, 8, 100003, "planted", "f16x2"),
                                               (40, 8, 270001, "odd signals", "f32"), (33, 7, 66000, "random", "f16x2"),
                                               (159, 4, 210007, "planted", "f16x2"), (64, 5, 100003, "noise33", "f16x2"),
                                               (97, 3, 70001, "noise40", "f32"), (32, 8, 66001, "noise130", "bf16x3"),
                                               (127, 7, 200003, "noise15", "f16x2")])
def test_code_starts_from_the_block_of_the_largest_bound(K, s0, m, kind, arith):
    """sbo_code on many signals guesses their block from bounds, where the dictionary consists of orthobases; with one more
    block that is none and that nobody takes it screens them all: the same bits."""
    Y, D = _home_case(64, K, s0, m, kind)
    got = []
    for Dk in (D, np.concatenate([D, 0.25 * D[:1]])):
        with Sbo(64, len(Dk), s0, m, arith=arith) as g:
            got.append(g.code(Y, Dk))
    for name, a, b in zip(("blk", "supp", "coef", "err"), *got):
        assert np.array_equal(a, b), (name, int((a != b).sum()))


@pytest.mark.parametrize("p,K,s0,kind,arith", [(256, 16, 12, "close", "f16x2"), (256, 31, 5, "planted", "f16x2"),
                                               (64, 33, 8, "close", "bf16x3"), (64, 130, 6, "odd signals", "f32"),
                                               (64, 256, 3, "planted", "f16x2")])
def test_code_of_few_signals_shares_out_the_blocks(p, K, s0, kind, arith):
    """Up to 8192 signals the block choice is split among workgroups; a signal gets the same bits as in a larger set
    (but for the last one of its error, which is rounded by where it stands in a tile of the selection)."""
    Y, D = _home_case(p, K, s0, 8256, kind)
    with Sbo(p, K, s0, len(Y), arith=arith) as g:
        want = g.code(Y, D)
        for m in (1100, 4097, 5041, 8192, 2111):
            for name, a, b in zip(("blk", "supp", "coef"), want, g.code(Y[:m], D)):
                assert np.array_equal(a[:m], b), (m, name, int((a[:m] != b).sum()))


@pytest.mark.parametrize("p,K_cap,K,s0", [(64, 257, 64, 6), (64, 512, 256, 4), (256, 260, 16, 12), (256, 300, 8, 5)])
def test_contexts_for_more_blocks_than_are_in_use_share_them_out(p, K_cap, K, s0):
    """A context made for more orthobases than the split choice takes, used with fewer: bit for bit what a context made for
    that many gives, also in the calls that follow."""
    Y, D = _home_case(p, K, s0, 8192, "planted")
    with Sbo(p, K_cap, s0, len(Y)) as big, Sbo(p, K, s0, len(Y)) as small:
        sbo.sbo_set_blocks(big.ctx, K)
        for m in (5041, 2111, 8192, 5041):
            print(f"case p={p} K={K} of {K_cap} m={m}", flush=True)
            for a, b in zip(big.code(Y[:m], D), small.code(Y[:m], D)):
                assert np.array_equal(a, b)
        for a, b in zip(big.iterate(Y[:5041], D, 3), small.iterate(Y[:5041], D, 3)):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("p,K_cap,K0,K_max", [(64, 300, 32, 34), (256, 300, 8, 9)])
def test_learn_on_a_context_for_more_blocks_than_it_ends_with(p, K_cap, K0, K_max):
    """Algorithm 2 with a number of orthobases whose block choice is split, on a context with room for many more."""
    m, s0, P0, W = 4097, 4, 3 * p, 4 * p
    Y, _D = _home_case(p, K_max, s0, m, "planted")
    rng = np.random.default_rng(p)
    sets = np.stack([np.sort(rng.permutation(m)[:P0]) for _ in range(K0)]).astype(np.int32)
    got = []
    for cap in (K_cap, K_max):
        with Sbo(p, cap, s0, m) as g:
            D = g.torch.zeros((K_max, p, p), dtype=g.torch.float32, device=g.dev)
            out = g.outputs(m)
            k, history = sbo.sbo_learn(g.ctx, g.dev_f32(Y), D, g.dev_i32(sets), 2, W, K_max, 0.0, *out)
            g.torch.cuda.synchronize()
            got.append([np.array([k]), np.array(history), D.cpu().numpy()] + [a.cpu().numpy() for a in out])
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("name,kw", [("tiny", dict()), ("patch8", dict(m=5000)), ("p32", dict(p=32, K=6, m=3000, s0=4)),
                                     ("p64_s5", dict(p=64, K=7, m=2100, s0=5)),
                                     ("p256", dict(p=256, K=2, m=1500, s0=12, snr_db=25.0))])
@pytest.mark.parametrize("arith", ARITH)
def test_iterate_one_step_matches_oracle(name, kw, arith):
    """sbo_iterate(1) (which fuses select and accumulate for p <= 64) against the oracle:
    the coding outputs element by element, the updated dictionary teacher-forced."""
    pr = _problem(name, **kw)
    cfg = pr.cfg
    print(f"case {name} {arith}: p={cfg.p} K={cfg.K} m={pr.Y.shape[0]} s0={cfg.s0}", flush=True)
    o = orc.o_code(pr.Y, pr.D_init, cfg.s0)
    with Sbo(cfg.p, cfg.K, cfg.s0, pr.Y.shape[0], arith=arith) as g:
        Dg, blk, supp, coef, err, sq = g.iterate(pr.Y, pr.D_init, 1)
        frac = compare_code(pr.Y, pr.D_init, cfg.s0, o, (blk, supp, coef, err))
        # the update the GPU made from ITS code, against the oracle's update from the same code
        Dn, M = orc.o_update(pr.Y, blk, supp, coef, pr.D_init)
        w = compare_Q(Dg, Dn, M, np.bincount(blk, minlength=cfg.K) > 0)
        b2, s2, c2, e2 = g.code(pr.Y, pr.D_init)
    assert np.array_equal(blk, b2) and np.array_equal(supp, s2)
    np.testing.assert_allclose(coef, c2, rtol=0, atol=1e-6 * np.abs(c2).max())
    assert abs(sq[0] - err.astype(np.float64).sum()) <= 1e-6 * sq[0] + 1e-12
    print(f"  exempt {frac:.5f}, worst dQ {w:.2e}", flush=True)


@pytest.mark.parametrize("name,kw,R", [("tiny", dict(), 4), ("patch8", dict(m=6000), 3),
                                       ("p256", dict(p=256, K=2, m=1500, s0=12, snr_db=25.0), 2)])
def test_train_rounds_frozen_assignment(name, kw, R):
    """R rounds of 1ONB per block with the assignment frozen.  Every round is compared with
    the oracle teacher-forced (the GPU starts the round from the oracle's dictionary, so a
    near-tie support flip cannot compound); the R-round call is then compared with the
    chain of single-round calls."""
    pr = _problem(name, **kw)
    cfg = pr.cfg
    m = pr.Y.shape[0]
    print(f"case {name}: p={cfg.p} K={cfg.K} m={m} s0={cfg.s0} R={R}", flush=True)
    blk = orc.o_code(pr.Y, pr.D_init, cfg.s0)[0]
    counts = np.bincount(blk, minlength=cfg.K)
    D = pr.D_init.astype(np.float64)
    with Sbo(cfg.p, cfg.K, cfg.s0, m) as g:
        chain = pr.D_init
        for r in range(R):
            D32 = D.astype(np.float32)
            # oracle round from D32: SELECT in the assigned block, then the update
            so, co, eo = orc.o_train_rounds(pr.Y, blk, D32, cfg.s0, 1)[1]
            Dg, sg, cg, eg = g.train_rounds(pr.Y, blk, D32, 1)
            # supports bit-exact except below the near-tie gap, exempt codes valid in fp64
            frac = compare_assigned_code(pr.Y, D32, blk, cfg.s0, (so, co, eo), (sg, cg, eg))
            Dn, M = orc.o_update(pr.Y, blk, sg, cg, D32)       # from the GPU's own code
            w = compare_Q(Dg, Dn, M, counts > 0)
            print(f"  round {r}: exempt fraction {frac:.5f}, worst dQ {w:.2e}, sqerr {eg.astype(np.float64).sum():.6f}",
                  flush=True)
            D = orc.o_train_rounds(pr.Y, blk, D32, cfg.s0, 1)[0]
            chain, s_ch, c_ch, e_ch = g.train_rounds(pr.Y, blk, chain, 1)
        DR, sR, cR, eR = g.train_rounds(pr.Y, blk, pr.D_init, R)
        DR2, *_ = g.train_rounds(pr.Y, blk, pr.D_init, R)
        D1, s1, c1, e1 = g.train_rounds(pr.Y, blk, pr.D_init, 1)
    assert np.array_equal(DR, DR2), "rounds not bitwise repeatable"
    # one call with R rounds = R calls with one round, bit for bit
    assert np.array_equal(DR, chain) and np.array_equal(sR, s_ch)
    assert np.array_equal(cR, c_ch) and np.array_equal(eR, e_ch)
    assert eR.astype(np.float64).sum() <= e1.astype(np.float64).sum() * (1 + 1e-6), "error increased over rounds"
    for j in range(cfg.K):
        Q = DR[j].astype(np.float64)
        assert np.abs(Q @ Q.T - np.eye(cfg.p)).max() <= 1e-5


def test_teacher_forced_iterations_patch8():
    """Each iteration: the GPU codes with the oracle's dictionary (rounded to fp32) and
    updates from the oracle's code, so chaotic block flips do not compound."""
    pr = _problem("patch8", m=4096)
    cfg = pr.cfg
    D = pr.D_init.astype(np.float64)
    with Sbo(cfg.p, cfg.K, cfg.s0, pr.Y.shape[0]) as g:
        for it in range(4):
            D32 = D.astype(np.float32)
            o = orc.o_code(pr.Y, D32, cfg.s0)
            frac = compare_code(pr.Y, D32, cfg.s0, o, g.code(pr.Y, D32))
            blk, supp, coef, err, E = o
            coef32 = coef.astype(np.float32)
            Dn, M = orc.o_update(pr.Y, blk, supp, coef32, D32)
            Dg, _ = g.update(pr.Y, blk, supp, coef32, D32)
            w = compare_Q(Dg, Dn, M, np.bincount(blk, minlength=cfg.K) > 0)
            print(f"  iter {it}: exempt {frac:.5f}, worst dQ {w:.2e}", flush=True)
            D = Dn


def test_errors_are_reported_not_faulted():
    import paper_1412_4944_amd as sbo
    import torch
    with Sbo(64, 4, 3, 128) as g:
        Y = g.dev_f32(np.zeros((256, 64)))
        D = g.dev_f32(np.zeros((4, 64, 64)))
        blk, supp, coef, err = g.outputs(256)
        with pytest.raises(sbo.SboError) as e:
            sbo.sbo_code(g.ctx, Y, D, blk, supp, coef, err)      # m > m_max
        assert e.value.code == sbo.binding.SBO_EINVAL
        # out-of-range block ids are dropped by grouping, not dereferenced
        b = np.array([0, 1, 99, -5, 3] + [2] * 100, np.int32)
        counts, offsets, perm = g.group(b)
        assert counts.tolist() == [1, 1, 100, 1] and offsets[-1] == 103
        torch.cuda.synchronize()


@pytest.mark.parametrize("arith", ARITH)
def test_largest_K_and_context_reuse(arith):
    """K = 1024 orthobases (the largest the boundary accepts), most of them empty after
    coding; and one context (sized for m_max) used for calls with smaller and changing m."""
    pr = synth.generate(synth.custom("bigK", p=16, K=1024, m=3000, s0=2, snr_db=20.0))
    cfg = pr.cfg
    with Sbo(16, 1024, 2, 4000, arith=arith) as g:        # m_max > every m used below
        for m in (3000, 777, 2500):
            Y = pr.Y[:m]
            o = orc.o_code(Y, pr.D_init, 2)
            out = g.code(Y, pr.D_init)
            compare_code(Y, pr.D_init, 2, o, out)
            blk, supp, coef, _err = out
            Dg, counts = g.update(Y, blk, supp, coef, pr.D_init)
            assert np.array_equal(counts, np.bincount(blk, minlength=1024))
            Dn, M = orc.o_update(Y, blk, supp, coef, pr.D_init)
            compare_Q(Dg, Dn, M, counts > 0)
            assert np.array_equal(Dg[counts == 0], pr.D_init[counts == 0]), "an empty block changed"
        # iterate in the same context, then code again: the fused path must leave the
        # workspace invariants intact for the call after it
        Y = pr.Y[:1500]
        Dg, blk, supp, coef, err, sq = g.iterate(Y, pr.D_init, 2)
        assert sq[1] <= sq[0] * (1 + 1e-6)
        compare_code(Y, Dg, 2, orc.o_code(Y, Dg, 2), g.code(Y, Dg))


@pytest.mark.parametrize("K", [1013, 1014, 1024])
def test_largest_K_at_p256(K):
    """Both sides of the line up to which the table of the screening kernel holds all blocks, and the largest K:
    coding against the oracle; beyond the line it is the coding in three bf16 parts, bit for bit, also inside
    sbo_iterate (which rereads the operand orders that the SVD kernel leaves)."""
    p, s0, m = 256, 12, 70
    rng = np.random.default_rng(K)
    Q = synth.random_onb(rng, p).T
    v = rng.standard_normal((K, p))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    D = (Q - 2 * (v @ Q.T)[:, :, None] * v[:, None, :]).astype(np.float32)       # atoms reflected at K hyperplanes
    Y = np.einsum("ik,ikd->id", rng.standard_normal((m, s0)), D[rng.integers(0, K, m)][:, :s0].astype(np.float64))
    Y = (Y + 0.05 * rng.standard_normal(Y.shape)).astype(np.float32)
    o = orc.o_code(Y, D, s0)
    codes, dicts = {}, {}
    for arith in ("f16x2", "bf16x3"):
        print(f"case {arith}: K={K}", flush=True)
        with Sbo(p, K, s0, m, arith=arith) as g:
            codes[arith] = g.code(Y, D)
            compare_code(Y, D, s0, o, codes[arith])
            dicts[arith] = g.iterate(Y[:24], D, 2)[:2] if K == 1014 else ()
    if K > 1013:
        for a, b in zip(codes["f16x2"] + tuple(dicts["f16x2"]), codes["bf16x3"] + tuple(dicts["bf16x3"])):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("K,m,s0", [(1, 1, 1), (1, 79, 16), (1, 16384, 12), (1, 16385, 12), (3, 8191, 1), (16, 5041, 12),
                                    (16, 16384, 16), (17, 5041, 12)])
def test_accumulate_p256_in_slices(K, m, s0):
    """p = 256, small sets: the dims of a piece in slices, at the edges of that rule and of pieces and steps; an empty block, ids
    out of range (ignored) and the sum over the pieces.  Bound: the fp32 sums of at most 64 products and of the pieces, each
    rounding 2^-24 of a partial sum, which random signs keep near the square root of their number."""
    p = 256
    rng = np.random.default_rng(71 + m + K)
    Y = rng.standard_normal((m, p)).astype(np.float32)
    blk = rng.integers(0, K, m).astype(np.int32)
    if K > 2:
        blk[blk == 1] = 0
    supp = np.sort(np.argsort(rng.random((m, p)), axis=1)[:, :s0], axis=1).astype(np.int32)
    coef = rng.standard_normal((m, s0)).astype(np.float32)
    x = np.zeros((m, p))
    np.put_along_axis(x, supp.astype(np.int64), coef.astype(np.float64), axis=1)
    if m > 10:
        x[3, supp[3, -1]] = 0.0
        supp[3, -1] = 256
    ref = np.stack([x[blk == j].T @ Y[blk == j].astype(np.float64) for j in range(K)])
    with Sbo(p, K, s0, m) as g:
        M = g.accumulate(Y, blk, supp, coef)
        np.testing.assert_array_equal(M, g.accumulate(Y, blk, supp, coef))
    for j in range(K):
        n = np.linalg.norm(ref[j])
        assert np.linalg.norm(M[j] - ref[j]) <= 4e-7 * n, j
        assert np.abs(M[j] - ref[j]).max() <= 4e-6 * max(np.abs(ref[j]).max(), 1e-30), j


@pytest.mark.parametrize("p", [16, 32, 64, 256])
def test_polar_condition_sweep_and_both_paths(p):
    """The SVD update over a range of condition numbers, once with the default path
    (Newton-Schulz, Jacobi for the blocks it flags) and once with the Jacobi SVD alone: each
    against the oracle, and the two against each other.  The last block is a symmetric positive
    definite matrix (polar factor = I) whose dominant eigenvectors are orthogonal to the vector of
    absolute row sums of its Gram matrix: a scale estimated by power iteration from that vector
    alone would be too small by a factor of 3.7 and send the dominant singular values to -1."""
    rng = np.random.default_rng(23 + p)
    conds = [1.0, 3.0, 30.0, 300.0, 900.0, 3e3, 3e4, 1e6, np.inf]
    K = len(conds) + 1
    M = np.empty((K, p, p))
    for j, c in enumerate(conds):
        u = synth.random_onb(rng, p)
        v = synth.random_onb(rng, p)
        s = np.geomspace(1.0, 1.0 / c, p) if np.isfinite(c) else np.r_[np.geomspace(1.0, 0.1, p - 3), 0, 0, 0]
        M[j] = (u * s) @ v.T * (10.0 ** rng.uniform(-3, 3))          # any overall scale
    # sqrt of kron(I, [[1, -0.6], [-0.6, 1]]): eigenvalues sqrt(1.6) on (1, -1)/sqrt2, sqrt(0.4) on (1, 1)/sqrt2
    a, b = (np.sqrt(1.6) + np.sqrt(0.4)) / 2, (np.sqrt(0.4) - np.sqrt(1.6)) / 2
    M[K - 1] = np.kron(np.eye(p // 2), np.array([[a, b], [b, a]]))
    M32 = M.astype(np.float32)
    D_old = synth.random_dictionary(rng, K, p).astype(np.float32)
    Dn = np.stack([orc.o_polar(M32[j].astype(np.float64)) for j in range(K)])
    assert np.abs(Dn[K - 1] - np.eye(p)).max() < 1e-6                # oracle agrees: polar factor = I
    out = {}
    with Sbo(p, K, min(4, p), 256) as g:
        for mode in ("default", "jacobi"):
            g.svd_jacobi(mode == "jacobi")
            out[mode] = g.polar(M32, D_old, None)
            sweeps = sbo.sbo_svd_sweeps(g.ctx, K)
            w = compare_Q(out[mode], Dn, M32.astype(np.float64), np.ones(K, bool))
            print(f"  p={p} {mode}: worst |Q - Q_oracle| {w:.2e}, per block {sweeps}", flush=True)
            if mode == "default":
                assert all(x < 0 for x in sweeps[:4]), "well-conditioned blocks should not need the fallback"
                assert sweeps[len(conds) - 1] > 0, "the rank-deficient block must go to the Jacobi SVD"
                assert sweeps[K - 1] < 0, "the symmetric block is well conditioned: Newton-Schulz"
            else:
                assert all(x > 0 for x in sweeps)
    good = [j for j, c in enumerate(conds) if c <= 900.0] + [K - 1]
    assert np.abs(out["default"][good] - out["jacobi"][good]).max() <= 1e-4


@pytest.mark.parametrize("p", [16, 32, 64, 256])
@pytest.mark.parametrize("cond", [3.0, 40.0, 150.0])
def test_polar_last_step_is_accurate(p, cond):
    """Signed permutations with random singular values: often one of them converges last, alone, and the error of
    the last step's polynomial and products all goes into one entry of size one.  Bound: two roundings of
    2^-24 (the Gram matrix, the result) and 2e-8 of the polynomial, with a margin of a quarter."""
    K = 16 if p == 256 else 96
    rng = np.random.default_rng(41 + p + int(cond))
    perm = np.stack([np.eye(p)[rng.permutation(p)] * rng.choice([-1.0, 1.0], p) for _ in range(K)])
    M = (perm * rng.uniform(1 / cond, 1, (K, 1, p)) * 10.0 ** rng.uniform(-3, 3, (K, 1, 1))).astype(np.float32)
    with Sbo(p, K, 4, 256) as g:
        D = g.polar(M, np.zeros_like(M), None)
        assert all(x < 0 for x in sbo.sbo_svd_sweeps(g.ctx, K))
    worst = np.abs(D.astype(np.float64) - perm).max()
    print(f"  p={p} cond={cond}: worst |Q - exact| {worst:.2e}", flush=True)
    assert worst <= 1.25 * (2 * 2.0 ** -24 + 2e-8)


@pytest.mark.parametrize("p", [16, 32, 64, 256])
@pytest.mark.parametrize("kind", ["spread", "one low", "one high"])
def test_polar_of_narrow_spectra_is_accurate(p, kind):
    """Singular values within 2 % (atoms used equally often): the iteration has nothing to do but to round twice, so
    the error per singular value is that of a sum of p terms in fp32, 2^-24 max(1, sqrt(p / 64)), with a margin
    of a half.  And on both sides of the line below which a spectrum counts as narrow, the same to 1e-6."""
    K = 16
    rng = np.random.default_rng(43 + p)
    def spectrum(low):
        if kind == "spread":
            return rng.uniform(low, 1, p)
        return np.r_[np.full(p - 1, low if kind == "one high" else 1.0), 1.0 if kind == "one high" else low]
    low = np.r_[np.full(8, 1 / 1.02), np.geomspace(1 / 1.1, 1 / 3, 8)]
    M32 = np.stack([(synth.random_onb(rng, p) * spectrum(l)) @ synth.random_onb(rng, p) * 10.0 ** rng.uniform(-3, 3)
                    for l in low]).astype(np.float32)
    with Sbo(p, K, 4, 256) as g:
        D = g.polar(M32, np.zeros_like(M32), None)
        steps = sbo.sbo_svd_sweeps(g.ctx, K)
    Q = np.stack([orc.o_polar(m.astype(np.float64)) for m in M32])
    err = np.sqrt(((D - Q) ** 2).sum((1, 2)) / p)
    print(f"  p={p} {kind}: worst {err[:8].max():.2e}, then {err[8:].max():.2e}, steps {steps}", flush=True)
    assert err[:8].max() <= 1.5 * 2.0 ** -24 * max(1.0, np.sqrt(p / 64))
    assert err.max() <= 1e-6


@pytest.mark.parametrize("m", [33, 2048, 2100])         # an unfinished tile; grouped; listed from the histograms
def test_select_p256_two_parts_over_magnitudes(m):
    """Signals of 1e-36 to 1e30, zeros among them: the two fp16 parts are those of a signal scaled by a power of two.
    Bound per coefficient: 3 * 2^-22 |y||q| for the parts, and sums of 48 products, 2^-24 each, of at most |y||q|."""
    p, s0 = 256, 12
    rng = np.random.default_rng(53 + m)
    D = synth.random_onb(rng, p)[None].astype(np.float32)
    scale = rng.choice([1e-36, 1e-30, 1e-18, 1e-3, 1.0, 1e18, 1e30, 0.0], m)
    x = np.zeros((m, p))
    np.put_along_axis(x, np.argsort(rng.random((m, p)), 1)[:, :s0], rng.uniform(0.5, 2, (m, s0)), 1)
    Y = ((x @ D[0] + 0.01 * rng.standard_normal((m, p))) * scale[:, None]).astype(np.float32)
    with Sbo(p, 1, s0, m) as g:
        _blk, supp, coef, _err = g.code(Y, D)
    c64 = Y.astype(np.float64) @ D[0].astype(np.float64).T
    norm = np.linalg.norm(Y.astype(np.float64), axis=1, keepdims=True)
    assert (np.abs(coef - np.take_along_axis(c64, supp, 1)) <= (3 * 2.0 ** -22 + 48 * 2.0 ** -24) * norm + 2.0 ** -149).all()
    some = scale > 0
    assert np.array_equal(supp[some], np.sort(np.argsort(-np.abs(c64[some]), 1)[:, :s0], 1))
    assert (coef[~some] == 0).all()


@pytest.mark.parametrize("p", [16, 32, 64, 256])
@pytest.mark.parametrize("s0", [1, 4])
@pytest.mark.parametrize("m", [100, 5000])
def test_code_with_dictionary_entries_up_to_8(p, s0, m):
    """The default arithmetic takes dictionary entries below 8: up to the next number below, where fp16 parts scaled by 2^13 end.
    Energies: 3 * 2^-22 |y||q| for the parts of a coefficient, and a rounding of 2^-24 |y||q| for each of its p products."""
    K = 4
    rng = np.random.default_rng(101 + p)
    D = np.stack([synth.random_onb(rng, p) for _ in range(K)])
    for j, largest in ((1, np.nextafter(np.float32(8), np.float32(0))), (3, 7.9985)):
        D[j] *= largest / np.abs(D[j]).max()
    D = D.astype(np.float32)
    D[1][np.unravel_index(np.abs(D[1]).argmax(), (p, p))] = np.nextafter(np.float32(8), np.float32(0))
    Y = rng.standard_normal((m, p)).astype(np.float32)
    with Sbo(p, K, s0, m) as g:
        blk, supp, coef, _err = g.code(Y, D)
    D64, Y64 = D.astype(np.float64), Y.astype(np.float64)
    c64 = np.einsum("mp,kap->mka", Y64, D64)
    E = np.sort(c64 ** 2, axis=2)[:, :, -s0:].sum(2)
    norm = np.linalg.norm(Y64, axis=1)
    rel = 3 * 2.0 ** -22 + p * 2.0 ** -24
    bound = rel * norm * np.linalg.norm(D64, axis=2).max()
    assert (E[np.arange(m), blk] >= E.max(1) - 4 * np.sqrt(s0 * E.max(1)) * bound).all()
    own = c64[np.arange(m), blk]
    assert (np.abs(coef - np.take_along_axis(own, supp, 1)) <= bound[:, None]).all()
    kept = np.zeros((m, p), bool)
    np.put_along_axis(kept, supp, True, 1)
    mag = np.abs(own)
    assert (np.where(kept, mag, np.inf).min(1) >= np.where(kept, 0, mag).max(1) - 2 * bound).all()


@pytest.mark.parametrize("m", [79, 2048, 2100])         # as above
@pytest.mark.parametrize("kind,size", [("scale", 1.01 / 16), ("scale", 0.99 / 16), ("scale", 1e-6), ("scale", 1e-8), ("scale", 1e-12),
                                       ("scale", 1e-20), ("atoms", 1e-3), ("atoms", 1e-8), ("atoms", 0.0), ("last", 5.0)])
def test_select_p256_takes_any_dictionary(m, kind, size):
    """sbo_code, one orthobase by any factor, or some of its atoms: the coefficient of an atom is as exact as its own norm allows (bound
    as above), on both sides of the line (1/16) from which on rows are read from D itself."""
    p, s0 = 256, 12
    rng = np.random.default_rng(89)
    D = synth.random_onb(rng, p)[None]
    at = {"scale": slice(None), "atoms": [0, 31, 32, 200], "last": [255]}[kind]
    D[0][at] *= size
    D = D.astype(np.float32)
    Y = rng.standard_normal((m, p)).astype(np.float32)
    with Sbo(p, 1, s0, m) as g:
        blk, supp, coef, _err = g.code(Y, D)
    assert (blk == 0).all()
    D64, Y64 = D[0].astype(np.float64), Y.astype(np.float64)
    c64 = Y64 @ D64.T
    bound = (3 * 2.0 ** -22 + 48 * 2.0 ** -24) * np.linalg.norm(Y64, axis=1)[:, None] * np.linalg.norm(D64, axis=1)
    assert (np.abs(coef - np.take_along_axis(c64, supp, 1)) <= np.take_along_axis(bound, supp, 1)).all()
    kept = np.zeros((m, p), bool)
    np.put_along_axis(kept, supp, True, 1)
    mag = np.abs(c64)
    assert (np.where(kept, mag + bound, np.inf).min(1) >= np.where(kept, 0, mag - bound).max(1)).all()


@pytest.mark.parametrize("m,s0", [(1500, 8), (6000, 5), (140000, 2)])      # a tile per wavefront; a few; many, grouped first
@pytest.mark.parametrize("order", ["rising", "falling", "mixed"])
def test_select_accum_two_parts_over_magnitudes(m, s0, order):
    """Signals of 1e-9 to 1, zeros among them, in one block and in every order: wherever parts of operands are scaled, no scale may fit
    the strong signals of a tile or piece alone.  Coefficients: 4 * 2^-22 |y||q| for the parts (two in fp16; three in bf16 leave less), and sums of 24 products, 2^-24 each, of at most |y||q|.  The update from the call's own codes."""
    p, K = 64, 2
    rng = np.random.default_rng(59 + m)
    D = np.stack([synth.random_onb(rng, p) for _ in range(K)]).astype(np.float32)
    scale = np.sort(np.r_[10.0 ** rng.uniform(-9, 0, m // 2), np.ones(m - m // 2 - 5), np.zeros(5)])
    scale = {"rising": scale, "falling": scale[::-1], "mixed": rng.permutation(scale)}[order]
    of, x = rng.integers(0, K, m), np.zeros((m, p))
    np.put_along_axis(x, np.argsort(rng.random((m, p)), 1)[:, :s0], rng.uniform(0.5, 2, (m, s0)), 1)
    Y = np.where(of[:, None] == 0, x @ D[0], x @ D[1]) + 0.01 * rng.standard_normal((m, p))
    Y = (Y * scale[:, None]).astype(np.float32)
    with Sbo(p, K, s0, m) as g:
        Dg, blk, supp, coef, err, _sq = g.iterate(Y, D, 1)
    Y64 = Y.astype(np.float64)
    c64 = np.where(blk[:, None] == 0, Y64 @ D[0].astype(np.float64).T, Y64 @ D[1].astype(np.float64).T)
    norm = np.linalg.norm(Y64, axis=1)
    kept = np.take_along_axis(c64, supp, 1)
    assert (np.abs(coef - kept) <= (4 * 2.0 ** -22 + 24 * 2.0 ** -24) * norm[:, None]).all()
    assert (np.abs(err - ((c64 ** 2).sum(1) - (kept ** 2).sum(1))) <= 1e-5 * norm ** 2).all()
    Dn, M = orc.o_update(Y, blk, supp, coef, D)
    print(f"  m={m} {order}: worst dQ {compare_Q(Dg, Dn, M, np.bincount(blk, minlength=K) > 0):.2e}", flush=True)


@pytest.mark.parametrize("largest", [7.9, 8.1, 3e4, 1e20])
def test_train_rounds_with_large_dictionary_entries(largest):
    """sbo_train_rounds takes any dictionary; entries of 8 and more are beyond fp16's range with the usual scale."""
    p, K, m, s0 = 64, 2, 3000, 6
    rng = np.random.default_rng(67)
    D = np.stack([synth.random_onb(rng, p) for _ in range(K)])
    D[1] *= largest / np.abs(D[1]).max()
    D = D.astype(np.float32)
    Y = rng.standard_normal((m, p)).astype(np.float32)
    blk = rng.integers(0, K, m).astype(np.int32)
    with Sbo(p, K, s0, m) as g:
        Q, supp, coef, _err = g.train_rounds(Y, blk, D, 1)
    c64 = np.where(blk[:, None] == 0, Y.astype(np.float64) @ D[0].astype(np.float64).T, Y.astype(np.float64) @ D[1].astype(np.float64).T)
    size = np.linalg.norm(Y, axis=1) * np.where(blk == 0, 1.0, np.linalg.norm(D[1].astype(np.float64), axis=1).max())
    assert (np.abs(coef - np.take_along_axis(c64, supp, 1)) <= (4 * 2.0 ** -22 + 24 * 2.0 ** -24) * size[:, None]).all()
    Dn, M = orc.o_update(Y, blk, supp, coef, D)
    compare_Q(Q, Dn, M, np.ones(K, bool))


@pytest.mark.parametrize("p", [16, 32, 64])
@pytest.mark.parametrize("kind,size", [("largest", 7.999), ("largest", 15.999), ("largest", 1.9999 * 2.0 ** 40), ("scale", 1e-6),
                                       ("scale", 1e-8), ("scale", 1e-12), ("atom", 1e6), ("atom", 1e8), ("atom", 1e-8)])
def test_train_rounds_with_any_dictionary(p, kind, size):
    """Orthobases by any factor, largest entries just below a power of two, and one atom of another size than the others: the
    coefficient of an atom is as exact as its own norm allows (bound as above)."""
    K, m, s0 = 2, 3000, 4
    rng = np.random.default_rng(71)
    D = np.stack([synth.random_onb(rng, p) for _ in range(K)])
    if kind == "largest":
        D[1] *= size / np.abs(D[1]).max()
    elif kind == "scale":
        D[1] *= size
    else:
        D[1][5] *= size
    D = D.astype(np.float32)
    Y = rng.standard_normal((m, p)).astype(np.float32)
    blk = rng.integers(0, K, m).astype(np.int32)
    with Sbo(p, K, s0, m) as g:
        Q, supp, coef, _err = g.train_rounds(Y, blk, D, 1)
    D64, Y64 = D.astype(np.float64), Y.astype(np.float64)
    c64 = np.where(blk[:, None] == 0, Y64 @ D64[0].T, Y64 @ D64[1].T)
    bound = (4 * 2.0 ** -22 + 24 * 2.0 ** -24) * np.linalg.norm(Y64, axis=1)[:, None] * np.linalg.norm(D64, axis=2)[blk]
    assert (np.abs(coef - np.take_along_axis(c64, supp, 1)) <= np.take_along_axis(bound, supp, 1)).all()
    kept = np.zeros((m, p), bool)
    np.put_along_axis(kept, supp, True, 1)
    mag = np.abs(c64)
    assert (np.where(kept, mag + bound, np.inf).min(1) >= np.where(kept, 0, mag - bound).max(1)).all()
    Dn, M = orc.o_update(Y, blk, supp, coef, D)
    compare_Q(Q, Dn, M, np.ones(K, bool))


@pytest.mark.parametrize("p", [16, 32, 64])
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_update_of_an_atom_that_only_weak_signals_use(p, seed):
    """Signals 2^-10 as strong as the others use the last atom, and nobody else does: its row of P_j, some 1e-5 of the largest one (from
    1e-6 on the SVD takes a row for zero), is a sum of its own, as exact as that row's size allows.  Bound: the sums of 16 products and
    the rotations of the SVD, a rounding of 2^-24 in each of some 100."""
    s0, weak, strong = 4, 16, 105 * p // 64
    rng = np.random.default_rng(73 + seed)
    D = synth.random_onb(rng, p)
    x = np.zeros((weak + strong, p))
    for i in range(weak + strong):
        x[i, rng.permutation(p - 1)[:s0]] = rng.uniform(0.5, 2, s0) * rng.choice([-1, 1], s0)
    x[:weak, p - 1] = rng.uniform(2, 3, weak)            # (the fifth: the smallest of the others goes)
    Y = x @ D + 0.02 * rng.standard_normal((weak + strong, p))
    Y[:weak] *= 2.0 ** -10
    Y = Y[rng.permutation(weak + strong)].astype(np.float32)
    blk = np.zeros(weak + strong, np.int32)
    with Sbo(p, 1, s0, weak + strong) as g:
        Q, supp, coef, _err = g.train_rounds(Y, blk, D[None].astype(np.float32), 1)
    used = (supp == p - 1).any(1)
    assert used.sum() == weak and np.abs(coef[used]).max() < 2.0 ** -7
    Dn, _M = orc.o_update(Y, blk, supp, coef, D[None])
    off = np.linalg.norm(Q[0, p - 1] - Dn[0, p - 1])
    print(f"  p={p}: last atom off by {off:.2e}", flush=True)
    assert off <= 100 * 2.0 ** -24


@pytest.mark.parametrize("p", [16, 32, 64])
@pytest.mark.parametrize("scale", [1.0, 1e-17, 1e17])
def test_polar_on_both_sides_of_the_lines_of_the_spread(p, scale):
    """The first guess of the smallest singular value hangs on the spread of the squared ones (0.01, 0.18, 0.75, 1.4: kSpread in
    polar_ns.hip).  An eighth of the values lies above the others, so that the spread is 1 % below and above each line.
    Bound: a rounding of 2^-24 in every step, where singular values of 1 / cond weigh it cond times as much."""
    rng = np.random.default_rng(47 + p)
    h, mats, conds = p // 8, [], []
    for line in (0.01, 0.18, 0.6, 0.75, 1.4):
        for want in (0.99 * line, 1.01 * line):
            lo, hi = 1.0, 1e3
            for _ in range(80):
                x = (lo + hi) / 2
                s2 = np.r_[np.full(h, x), np.ones(p - h)]
                lo, hi = (x, hi) if (s2 ** 2).mean() / s2.mean() ** 2 - 1 < want else (lo, x)
            mats.append((synth.random_onb(rng, p) * np.sqrt(s2)) @ synth.random_onb(rng, p) * scale)
            conds.append(np.sqrt(x))
    M32 = np.stack(mats).astype(np.float32)
    with Sbo(p, len(mats), 4, 256) as g:
        D = g.polar(M32, np.zeros_like(M32), None)
        steps = -np.array(sbo.sbo_svd_sweeps(g.ctx, len(mats)))
    Q = np.stack([orc.o_polar(m.astype(np.float64)) for m in M32])
    err = np.sqrt(((D - Q) ** 2).sum((1, 2)) / p)
    print(f"  p={p} scale={scale}: |Q - Q64| {err}, steps {steps}", flush=True)
    assert (steps > 0).all() and (steps <= 7).all()
    assert (err <= steps * np.array(conds) * 2.0 ** -24).all()


@pytest.mark.parametrize("p", [16, 32, 64])
def test_polar_does_not_depend_on_a_power_of_two(p):
    """U V^T has no scale: the steps and the bits are those of the same matrix times 2^k, as long as its squares and its entries are
    fp32 numbers (the spread, by which the steps are chosen, is made of fourth powers)."""
    rng = np.random.default_rng(103 + p)
    mats = [(synth.random_onb(rng, p) * np.geomspace(1, 1 / c, p)) @ synth.random_onb(rng, p) for c in (1.05, 1.5, 3, 10, 100)]
    M = np.stack(mats).astype(np.float32)
    M[np.abs(M) < 2.0 ** -40] = 0
    with Sbo(p, len(M), 4, 256) as g:
        D = g.polar(M, np.zeros_like(M), None)
        steps = sbo.sbo_svd_sweeps(g.ctx, len(M))
        assert all(x < 0 for x in steps)
        for k in (-58, -40, -30, 25, 58):
            np.testing.assert_array_equal(g.polar(M * np.float32(2.0 ** k), np.zeros_like(M), None), D)
            assert sbo.sbo_svd_sweeps(g.ctx, len(M)) == steps, k


@pytest.mark.parametrize("K", [1, 9, 33])               # one team; two groups of eight; teams with three blocks in turn
@pytest.mark.parametrize("jacobi_only", [False, True], ids=["auto", "jacobi"])
def test_polar_p256_teams_of_workgroups(K, jacobi_only):
    """p = 256: blocks of every kind in one launch (a team passes from Newton-Schulz on one block to
    the Jacobi SVD on the next, to an empty one), twice in a row on one context."""
    p = 256
    rng = np.random.default_rng(29 + K)
    M = np.stack([(synth.random_onb(rng, p) * np.geomspace(1, 10.0 ** -(j % 3), p)) @ synth.random_onb(rng, p)
                  for j in range(K)])
    for j in range(4, K, 9):
        M[j][:, 200:] = M[j][:, :56]                     # rank 200: left to the Jacobi SVD
    counts = np.ones(K, np.int32)
    counts[5::7] = 0
    M32 = M.astype(np.float32)
    D_old = synth.random_dictionary(rng, K, p).astype(np.float32)
    Dn = np.stack([orc.o_polar(M32[j].astype(np.float64)) if counts[j] else D_old[j] for j in range(K)])
    with Sbo(p, K, 4, 256, jacobi_only=jacobi_only) as g:
        a, b = g.polar(M32, D_old, counts), g.polar(M32, D_old, counts)
    np.testing.assert_array_equal(a, b)
    w = compare_Q(a, Dn, M32.astype(np.float64), counts > 0)
    print(f"  K={K} jacobi={jacobi_only}: worst |Q - Q_oracle| {w:.2e}", flush=True)


@pytest.mark.parametrize("jacobi_only", [False, True], ids=["auto", "jacobi"])
def test_polar_p256_blocks_in_turn_are_those_of_a_team_of_their_own(jacobi_only):
    """p = 256, 40 orthobases: a team has up to three in turn, in the same memory.  By the Jacobi SVD (full and deficient ranks in
    every order, Newton-Schulz between them) each comes out with the bits that it has where every team has one."""
    p, K = 256, 40
    rng = np.random.default_rng(83)
    M = np.stack([synth.random_onb(rng, p) * np.geomspace(1, 1e-3, p) @ synth.random_onb(rng, p) for _ in range(K)])
    for j in range(K):
        if (j % 16 + j // 16) % 3 == 0:                  # rank 216: one workgroup completes it
            M[j][:, 216:] = M[j][:, :40]
        elif not jacobi_only and (j % 16 + j // 16) % 3 == 1:
            M[j] += synth.random_onb(rng, p)             # well conditioned: Newton-Schulz
    M = M.astype(np.float32)
    old = np.zeros_like(M)
    with Sbo(p, K, 4, 256) as g:
        g.svd_jacobi(jacobi_only)
        print(f"case jacobi={jacobi_only}", flush=True)
        D = g.polar(M, old, None)
        parts = []
        for at in range(0, K, 16):
            n = min(16, K - at)
            sbo.sbo_set_blocks(g.ctx, n)
            parts.append(g.polar(M[at:at + n], old[at:at + n], None))
    # the same teams (16 workgroups) in all of them but the last eight, whose teams may be of pairs: the same bits too
    np.testing.assert_array_equal(D, np.concatenate(parts))
    for j in range(K):
        assert np.abs(D[j] @ D[j].T - np.eye(p)).max() <= 1e-5, j


@pytest.mark.parametrize("K", [1, 8])
@pytest.mark.parametrize("polls", [1 << 22, 40, 3, 0])
def test_polar_p256_teams_of_pairs(K, polls):
    """p = 256, up to eight orthobases: two workgroups to a strip of columns.  The same bits as without the second
    ones, and as by the teams that more orthobases have, for every kind of block; with waits that end early every
    block is finished all the same, and the next call finds the counters set back."""
    p = 256
    rng = np.random.default_rng(61 + K)
    M = np.stack([(synth.random_onb(rng, p) * np.geomspace(1, 10.0 ** -(j % 4), p)) @ synth.random_onb(rng, p)
                  for j in range(9)])
    M[2] = np.diag(rng.uniform(0.98, 1, p))[rng.permutation(p)]                    # a narrow spectrum
    if K > 1:
        M[5][:, 200:] = M[5][:, :56]                     # rank 200: left to the Jacobi SVD
        M[6] = 0
        M[7][3, 5] = np.nan
    M32 = M.astype(np.float32)
    counts = np.ones(9, np.int32)
    counts[4] = 0
    D_old = synth.random_dictionary(rng, 9, p).astype(np.float32)
    good = [j for j in range(K) if K == 1 or j not in (4, 5, 6, 7)]
    with Sbo(p, 9, 4, 256) as g:                         # nine orthobases: teams of 16
        teams = g.polar(M32, D_old, counts)[:K]
        few = lambda: g.polar(M32[:K], D_old[:K], counts[:K])
        sbo.sbo_set_blocks(g.ctx, K)
        pairs = few()
        steps = np.array(sbo.sbo_svd_sweeps(g.ctx, K))
        g.wide_helpers(False)
        alone = few()
        g.wide_helpers(True)
        sbo.sbo_set_option(g.ctx, sbo.SBO_OPT_SVD_WAIT, polls)
        print(f"case K={K} polls={polls} steps {steps}", flush=True)
        ended = few()
        sbo.sbo_set_option(g.ctx, sbo.SBO_OPT_SVD_WAIT, 1 << 22)
        again = few()
    assert (steps[good] < 0).all()
    np.testing.assert_array_equal(pairs, teams)
    np.testing.assert_array_equal(pairs, alone)
    np.testing.assert_array_equal(pairs, again)
    for j in good:
        Q = orc.o_polar(M32[j].astype(np.float64))
        assert np.abs(pairs[j] - Q).max() <= 2e-6
        compare_Q(ended[j:j + 1], Q[None], M32[j:j + 1].astype(np.float64), np.ones(1, bool))
    if K > 1:
        np.testing.assert_array_equal(ended[4], D_old[4])


def test_polar_p256_on_three_streams():
    """Contexts on more than two streams: the teams take the other workgroup order; their launches overlap."""
    import torch
    p, K = 256, 9
    rng = np.random.default_rng(31)
    M32 = np.stack([(synth.random_onb(rng, p) * np.geomspace(1, 0.1, p)) @ synth.random_onb(rng, p)
                    for _ in range(K)]).astype(np.float32)
    M32[4][:, 200:] = M32[4][:, :56]                     # left to the Jacobi SVD
    Dn = np.stack([orc.o_polar(M32[j].astype(np.float64)) for j in range(K)])
    M = torch.from_numpy(M32).cuda()
    D = [torch.zeros_like(M) for _ in range(3)]
    torch.cuda.synchronize()
    ctxs = []
    for _ in range(3):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            ctxs.append((s, sbo.sbo_create(p, K, 4, 256)))
    for _ in range(3):
        for (s, c), d in zip(ctxs, D):
            with torch.cuda.stream(s):
                sbo.sbo_polar(c, M, None, d)
    torch.cuda.synchronize()
    for s, c in ctxs:
        sbo.sbo_destroy(c)
    for d in D:
        compare_Q(d.cpu().numpy(), Dn, M32.astype(np.float64), np.ones(K, bool))
        assert torch.equal(d, D[0])


def test_polar_p256_pairs_have_the_gpu_to_themselves():
    """Teams of pairs take a whole XCD each, so they are for contexts on one stream; on two streams teams of 16, whose launches
    overlap, and the same bits."""
    import torch
    p, K = 256, 8
    rng = np.random.default_rng(97)
    M = torch.from_numpy(np.stack([(synth.random_onb(rng, p) * np.geomspace(1, 0.1, p)) @ synth.random_onb(rng, p)
                                   for _ in range(K)]).astype(np.float32)).cuda()
    pairs = sbo.lib().sbo_test_wide_pairs
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    a = sbo.sbo_create(p, K, 4, 256, streams[0].cuda_stream)
    same = sbo.sbo_create(p, 9, 4, 256, streams[0].cuda_stream)
    assert pairs(a) == 1 and pairs(same) == 0            # nine orthobases: teams of 16
    with torch.cuda.stream(streams[0]):
        alone = torch.zeros_like(M)
        sbo.sbo_polar(a, M, None, alone)
    b = sbo.sbo_create(p, K, 4, 256, streams[1].cuda_stream)
    assert pairs(a) == 0 and pairs(b) == 0
    D = [torch.zeros_like(M) for _ in range(2)]
    torch.cuda.synchronize()
    for _ in range(4):
        for c, d in zip((a, b), D):
            sbo.sbo_polar(c, M, None, d)
    torch.cuda.synchronize()
    assert torch.equal(D[0], alone) and torch.equal(D[1], alone)
    sbo.sbo_destroy(b)
    assert pairs(a) == 1
    sbo.sbo_destroy(a)
    sbo.sbo_destroy(same)


@pytest.mark.parametrize("polls", [0, 1, 8, 60, 400])
@pytest.mark.parametrize("K", [1, 9, 33])
def test_polar_p256_teams_that_give_up(K, polls):
    """Waits between the workgroups of a p = 256 team that end early (none at all, or somewhere on the way): every
    block is finished all the same, empty ones keep their basis, and the next call finds the counters set back."""
    p = 256
    rng = np.random.default_rng(37 + K)
    M = np.stack([(synth.random_onb(rng, p) * np.geomspace(1, 10.0 ** -(j % 3), p)) @ synth.random_onb(rng, p)
                  for j in range(K)])
    for j in range(4, K, 9):
        M[j][:, 200:] = M[j][:, :56]                     # rank 200
    counts = np.ones(K, np.int32)
    counts[5::7] = 0
    M32 = M.astype(np.float32)
    D_old = synth.random_dictionary(rng, K, p).astype(np.float32)
    Dn = np.stack([orc.o_polar(M32[j].astype(np.float64)) if counts[j] else D_old[j] for j in range(K)])
    with Sbo(p, K, 4, 256) as g:
        for jacobi_only in (False, True):
            print(f"case K={K} polls={polls} jacobi={jacobi_only}", flush=True)
            g.svd_jacobi(jacobi_only)
            before = g.polar(M32, D_old, counts)
            sbo.sbo_set_option(g.ctx, sbo.SBO_OPT_SVD_WAIT, polls)
            D = g.polar(M32, D_old, counts)
            work = np.array(sbo.sbo_svd_sweeps(g.ctx, K))
            sbo.sbo_set_option(g.ctx, sbo.SBO_OPT_SVD_WAIT, 1 << 22)
            np.testing.assert_array_equal(g.polar(M32, D_old, counts), before)
            compare_Q(D, Dn, M32.astype(np.float64), counts > 0)
            np.testing.assert_array_equal(D[counts == 0], D_old[counts == 0])
            assert (work[counts == 0] == 0).all() and (work[counts > 0] != 0).all()
            if polls == 0:
                assert (work[counts > 0] > 0).all(), "no team can have met"


@pytest.mark.parametrize("polls", [0, 100])
def test_polar_p256_teams_that_give_up_on_three_streams(polls):
    """The same with the workgroup order of more than two streams, whose launches overlap."""
    import torch
    p, K = 256, 9
    rng = np.random.default_rng(53)
    M32 = np.stack([(synth.random_onb(rng, p) * np.geomspace(1, 0.1, p)) @ synth.random_onb(rng, p)
                    for _ in range(K)]).astype(np.float32)
    M32[4][:, 200:] = M32[4][:, :56]                     # left to the Jacobi SVD
    Dn = np.stack([orc.o_polar(M32[j].astype(np.float64)) for j in range(K)])
    M = torch.from_numpy(M32).cuda()
    D = [torch.zeros_like(M) for _ in range(3)]
    torch.cuda.synchronize()
    ctxs = []
    for _ in range(3):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            ctxs.append((s, sbo.sbo_create(p, K, 4, 256)))
        sbo.sbo_set_option(ctxs[-1][1], sbo.SBO_OPT_SVD_WAIT, polls)
    for _ in range(2):
        for (s, c), d in zip(ctxs, D):
            with torch.cuda.stream(s):
                sbo.sbo_polar(c, M, None, d)
    torch.cuda.synchronize()
    for s, c in ctxs:
        sbo.sbo_destroy(c)
    for d in D:
        compare_Q(d.cpu().numpy(), Dn, M32.astype(np.float64), np.ones(K, bool))


def test_iterate_and_base_at_p256_with_teams_that_give_up():
    """The same inside sbo_iterate: the next coding pass reads the operand orders of what was finished; and the
    eigenvectors of a Gram matrix."""
    pr = _problem("giveup", p=256, K=2, m=1500, s0=12, snr_db=25.0)
    m = pr.Y.shape[0]
    ids = np.arange(0, m, 2).astype(np.int32)
    with Sbo(256, 2, 12, m) as g:
        sbo.sbo_set_option(g.ctx, sbo.SBO_OPT_SVD_WAIT, 0)
        D1, blk, supp, coef, err, sq = g.iterate(pr.Y, pr.D_init, 1)
        Dn, M = orc.o_update(pr.Y, blk, supp, coef, pr.D_init)
        compare_Q(D1, Dn, M, np.bincount(blk, minlength=2) > 0)
        D2, b2, s2, c2, e2, sq2 = g.iterate(pr.Y, pr.D_init, 2)
        compare_code(pr.Y, D1, 12, orc.o_code(pr.Y, D1, 12), (b2, s2, c2, e2))
        assert sq2[0] == sq[0] and sq2[1] <= sq2[0] * (1 + 1e-6)
        Q, sv = g.init_base(pr.Y, ids)
    G = pr.Y[ids].astype(np.float64).T @ pr.Y[ids].astype(np.float64)
    lam = np.linalg.eigvalsh(G)[::-1]
    Q64 = Q.astype(np.float64)
    assert np.abs(Q64 @ Q64.T - np.eye(256)).max() <= 1e-5
    H = Q64 @ G @ Q64.T                                   # (2e-5: the bound of the tests of sbo_init_base)
    assert np.abs(H - np.diag(np.diag(H))).max() <= 2e-5 * lam[0]
    assert np.abs(sv.astype(np.float64) ** 2 - lam).max() <= 2e-5 * lam[0]


JACOBI_CASES = [("tiny", dict(), 12), ("patch8", dict(m=4096 + 77), 10),
                ("p256", dict(p=256, K=2, m=1300, s0=12, snr_db=25.0), 2)]


@pytest.mark.parametrize("name,kw,iters", JACOBI_CASES, ids=[c[0] for c in JACOBI_CASES])
def test_jacobi_only_inside_iterate_and_rounds(name, kw, iters):
    """SBO_SVD_JACOBI (the one-sided Jacobi SVD for every orthobase) inside sbo_iterate and
    sbo_train_rounds: every iteration teacher-forced against the oracle's update, then a
    free-running sbo_iterate over all iterations against the oracle's error curve."""
    pr = _problem(name, **kw)
    cfg = pr.cfg
    m = pr.Y.shape[0]
    print(f"case {name}: p={cfg.p} K={cfg.K} m={m} s0={cfg.s0} iters={iters}", flush=True)
    D = pr.D_init.astype(np.float64)
    with Sbo(cfg.p, cfg.K, cfg.s0, m, jacobi_only=True) as g:
        for it in range(min(iters, 4)):
            D32 = D.astype(np.float32)
            o = orc.o_code(pr.Y, D32, cfg.s0)
            Dg, blk, supp, coef, err, sq = g.iterate(pr.Y, D32, 1)
            assert all(x >= 0 for x in sbo.sbo_svd_sweeps(g.ctx, cfg.K)), "Newton-Schulz ran"
            frac = compare_code(pr.Y, D32, cfg.s0, o, (blk, supp, coef, err))
            counts = np.bincount(blk, minlength=cfg.K)
            Dn, M = orc.o_update(pr.Y, blk, supp, coef, D32)   # the oracle's update from the GPU's code
            w = compare_Q(Dg, Dn, M, counts > 0)
            # the same update through the frozen-assignment rounds
            Dr, sr, cr, er = g.train_rounds(pr.Y, blk, D32, 1)
            assert np.array_equal(sr, supp)
            w2 = compare_Q(Dr, Dn, M, counts > 0)
            print(f"  iter {it}: exempt {frac:.5f}, worst dQ iterate {w:.2e} rounds {w2:.2e}", flush=True)
            D = orc.o_update(pr.Y, o[0], o[1], o[2], D32)[0]
        Dg, blk, supp, coef, err, sq = g.iterate(pr.Y, pr.D_init, iters)
        Dg2, *_r, sq2 = g.iterate(pr.Y, pr.D_init, iters)
        assert np.array_equal(Dg, Dg2) and np.array_equal(sq, sq2), "not bitwise repeatable"
        # R rounds in one call against the chain of single rounds (frozen assignment)
        b0 = orc.o_code(pr.Y, pr.D_init, cfg.s0)[0]
        DR, *_x = g.train_rounds(pr.Y, b0, pr.D_init, 3)
        chain = pr.D_init
        for _ in range(3):
            chain, *_x = g.train_rounds(pr.Y, b0, chain, 1)
        assert np.array_equal(DR, chain)
    sq_o = orc.o_iterate(pr.Y, pr.D_init, cfg.s0, iters)[2]
    print("  oracle sqerr", sq_o, "\n  gpu    sqerr", sq, flush=True)
    assert (np.diff(sq) <= 1e-6 * sq[0]).all(), "error increased"
    np.testing.assert_allclose(sq, sq_o, rtol=1e-3)
    for j in range(cfg.K):
        Q = Dg[j].astype(np.float64)
        assert np.abs(Q @ Q.T - np.eye(cfg.p)).max() <= 1e-5


@pytest.mark.parametrize("arith", ARITH)
@pytest.mark.parametrize("jacobi_only", [False, True], ids=["auto", "jacobi"])
def test_iterate_with_rank_deficient_blocks(jacobi_only, arith):
    """Skewed assignment with more orthobases than the data supports: the rare orthobases get
    fewer than p signals, so their P_j are rank-deficient.  Inside sbo_iterate these go to the
    Jacobi SVD (flagged by Newton-Schulz in the default mode), which completes the basis and
    also writes the dictionary copy the next coding pass reads.  Checked: the updated
    dictionary (polar-factor properties on every orthobase, values where P_j is well
    conditioned) and the NEXT coding pass, element by element against the oracle."""
    pr = synth.generate(synth.custom("rankdef", p=64, K=24, m=3000, s0=4, snr_db=20.0, zipf_s=1.3))
    cfg = pr.cfg
    D0 = pr.D_planted                  # signals go to their planted orthobase: skewed counts
    o = orc.o_code(pr.Y, D0, cfg.s0)
    with Sbo(cfg.p, cfg.K, cfg.s0, pr.Y.shape[0], jacobi_only=jacobi_only, arith=arith) as g:
        D1, blk, supp, coef, err, sq = g.iterate(pr.Y, D0, 1)
        sweeps = sbo.sbo_svd_sweeps(g.ctx, cfg.K)
        compare_code(pr.Y, D0, cfg.s0, o, (blk, supp, coef, err))
        counts = np.bincount(blk, minlength=cfg.K)
        small = (counts > 0) & (counts < cfg.p)
        print(f"  counts {counts.tolist()}\n  svd work {sweeps}", flush=True)
        assert small.sum() >= 3 and (counts >= 2 * cfg.p).sum() >= 3, "the case needs small and large blocks"
        for j in np.nonzero(small)[0]:
            assert sweeps[j] > 0, f"rank-deficient block {j} did not go to the Jacobi SVD"
        if not jacobi_only:
            assert any(x < 0 for x in sweeps), "Newton-Schulz handled no block"
        Dn, M = orc.o_update(pr.Y, blk, supp, coef, D0)
        w = compare_Q(D1, Dn, M, counts > 0)
        assert np.array_equal(D1[counts == 0], D0[counts == 0])
        # two iterations in one call: the codes it leaves are those of pass 2, i.e. with D1
        D2, b2, s2, c2, e2, sq2 = g.iterate(pr.Y, D0, 2)
        assert sq2[0] == sq[0] and sq2[1] <= sq2[0] * (1 + 1e-6)
        frac = compare_code(pr.Y, D1, cfg.s0, orc.o_code(pr.Y, D1, cfg.s0), (b2, s2, c2, e2))
        print(f"  worst dQ {w:.2e}; next coding pass: exempt {frac:.5f}", flush=True)
        c2n = np.bincount(b2, minlength=cfg.K)
        Dn2, M2 = orc.o_update(pr.Y, b2, s2, c2, D1)
        compare_Q(D2, Dn2, M2, c2n > 0)
