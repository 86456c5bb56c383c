"""CPU-side checks of the C-ABI library: it loads, exports what include/isr.h
declares, and its host-only pieces (noise table, statistics, blob validation)
agree with the oracle and the golden values.  No compute call needs a GPU."""
import os
import re
import struct

import numpy as np
import pytest

import oracle
import paper_2108_09413_amd as isr
import synth
from oracle import stats as ostats

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ALPHA = 0.001


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "isr.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(isr_[a-z0-9_]+)\s*\(", header))
    assert declared == set(isr.EXPORTS)
    L = isr.lib()
    for name in declared:
        assert hasattr(L, name), name


@pytest.mark.parametrize("sigma", [1, 2, 15, 32, 64, 128, 256, 1024])
def test_noise_table_identical_to_oracle(sigma):
    T, R = isr.isr_noise_table(sigma)
    To, Ro = oracle.noise_table(sigma)
    assert R == Ro and np.array_equal(T, To)


def test_noise_table_argument_domain():
    for bad in (0, 1025):
        with pytest.raises(isr.IsrError) as e:
            isr.isr_noise_table(bad)
        assert e.value.status == isr.ISR_ERR_ARG


def test_cp_and_radius_against_golden_values(golden_dir):
    for l in open(os.path.join(golden_dir, "cp_radius_values.txt")):
        if l.startswith("#") or not l.strip():
            continue
        n, k, p_txt, r_txt = l.split()
        n, k = int(n), int(k)
        p = isr.isr_cp_lower(k, n, ALPHA)
        assert p == pytest.approx(float(p_txt), rel=2e-15, abs=1e-16)
        c1 = [n - k, k, 0]
        res = isr.isr_decide_certify([0, 5, 1], c1, 64.0, n, ALPHA)
        assert res.n_top == k and res.p_lower == p
        if r_txt == "abstain":
            assert res.cls == isr.ABSTAIN and res.radius == 0.0
        else:
            tol = max(1e-12, 4e-16 / abs(float(p_txt) - 0.5))
            assert res.cls == 1 and res.radius / 64.0 == pytest.approx(float(r_txt), rel=tol)


@pytest.mark.parametrize("n,misses,alpha", [(4_200_000_000, 160, 1e-12), (2 ** 32 - 1, 3, 1e-3), (10 ** 9, 160, 1e-12), (100_000, 50, 1e-3)])
def test_cp_bound_with_few_misses_in_many_trials(n, misses, alpha):
    """The law is narrow there (3e-9 of p), so Newton's last step has to be that much smaller.  By the tail of the misses,
    P[Bin(n, q) <= misses] = alpha at p = 1 - q, summed in 60 digits; within the last place of p (half a place for its
    rounding, the rest for the long double evaluation)."""
    import mpmath as mp
    with mp.workdps(60):
        p = mp.mpf(isr.isr_cp_lower(n - misses, n, alpha))

        def tail(q):
            term = total = mp.exp(n * mp.log1p(-q))
            for j in range(1, misses + 1):
                term *= q / (1 - q) * (n - j + 1) / j
                total += term
            return total

        ulp = mp.mpf(2) ** -53
        assert tail(1 - p - ulp) > alpha > tail(1 - p + ulp)


def test_statistics_agree_with_oracle_on_random_counts():
    rng = np.random.default_rng(3)
    for _ in range(300):
        n = int(rng.choice([100, 1000, 10000, 100000]))
        k = int(rng.integers(0, n + 1))
        alpha = float(rng.choice([0.001, 0.01, 0.05, 0.3]))
        a, b = isr.isr_cp_lower(k, n, alpha), ostats.cp_lower(k, n, alpha)
        assert a == pytest.approx(b, rel=1e-12, abs=1e-15)
        C = int(rng.integers(2, 12))
        c0 = rng.multinomial(100, rng.dirichlet(np.ones(C))).astype(np.uint32)
        c1 = rng.multinomial(n, rng.dirichlet(np.ones(C) * 0.3)).astype(np.uint32)
        sigma = float(rng.choice([32, 64, 128, 256]))
        res = isr.isr_decide_certify(c0, c1, sigma, n, alpha)
        cls, rad, pl, ntop = ostats.certify_decision(c0, c1, sigma, n, alpha)
        assert res.cls == cls and res.n_top == ntop
        assert res.p_lower == pytest.approx(pl, rel=1e-12, abs=1e-15)
        if cls != ostats.ABSTAIN:
            assert res.radius == pytest.approx(rad, rel=max(1e-9, 1e-15 / abs(pl - 0.5)))
        # integer-only tail on the same tallies (Thm 3.2): computed from the library's own bound,
        # which may differ from the oracle's in the last bits -- compare on the library's bound
        icls, t, t2 = ostats.certify_decision_integer(c0, c1, int(sigma), n, alpha)
        assert icls == res.cls
        if cls != ostats.ABSTAIN:
            assert res.radius_int == ostats.discrete_quantile(int(sigma), res.p_lower)
            assert res.radius_sq_int == ostats.radius_squared_int(int(sigma), res.p_lower)
            assert abs(res.radius_int - t) <= (1 if abs(res.p_lower - pl) > 0 else 0)
            assert res.radius - 1.5 - 1e-6 <= res.radius_int <= res.radius - 0.5 + 1e-6 + 1e-3 * sigma
        else:
            assert (res.radius_int, res.radius_sq_int) == (0, 0) and (t, t2) == (0, 0)
        cp = rng.multinomial(int(rng.choice([10, 100, 1000, 100000])), rng.dirichlet(np.ones(C) * 0.5)).astype(np.uint32)
        rp = isr.isr_decide_predict(cp, alpha)
        pc, pv, na, nb = ostats.predict_decision(cp, alpha)
        assert (rp.cls, rp.n_top, rp.n_second) == (pc, na, nb)
        assert rp.p_lower == pytest.approx(pv, rel=1e-10, abs=1e-300)


def test_normal_quantile_and_pvalue_special_values():
    import mpmath as mp
    mp.mp.dps = 80
    for p in (1e-30, 1e-12, 0.001, 0.3, 0.5, 0.5000000001, 0.9, 0.99993092483300939, 1 - 1e-15):
        want = float(mp.sqrt(2) * mp.erfinv(2 * mp.mpf(p) - 1))
        assert isr.isr_normal_quantile(p) == pytest.approx(want, rel=1e-13, abs=1e-16)
    for bad in (0.0, 1.0, -0.1, float("nan")):
        with pytest.raises(isr.IsrError):
            isr.isr_normal_quantile(bad)
    assert isr.isr_binom_pvalue(0, 0) == 1.0
    assert isr.isr_binom_pvalue(5, 5) == 1.0
    assert isr.isr_binom_pvalue(11, 0) == pytest.approx(2.0 ** -10, rel=1e-14)
    assert isr.isr_binom_pvalue(60, 40) == pytest.approx(0.056887933640980784, rel=1e-12)
    with pytest.raises(isr.IsrError):
        isr.isr_cp_lower(5, 4, ALPHA)
    with pytest.raises(isr.IsrError):
        isr.isr_cp_lower(1, 4, 1.5)


def test_validate_model_accepts_workloads_and_rejects_damage():
    for cfg, size in ((0, None), (1, None), (3, 32)):
        assert isr.isr_validate_model(synth.build_model(cfg, size=size)) == isr.ISR_OK
    blob = bytearray(synth.build_model(0))
    assert isr.isr_validate_model(bytes(blob[:-4])) == isr.ISR_ERR_FORMAT          # truncated
    assert isr.isr_validate_model(bytes(blob) + b"\0\0\0\0") == isr.ISR_ERR_FORMAT  # trailing bytes
    bad = bytearray(blob); bad[0] ^= 1
    assert isr.isr_validate_model(bytes(bad)) == isr.ISR_ERR_FORMAT                # magic
    bad = bytearray(blob); struct.pack_into("<I", bad, 4, 2)
    assert isr.isr_validate_model(bytes(bad)) == isr.ISR_ERR_FORMAT                # version
    assert isr.isr_validate_model(b"") == isr.ISR_ERR_FORMAT
    # a weight of -128 is outside the symmetric range
    off = 32 + 5 * 16 + 8 + 24
    bad = bytearray(blob); bad[off] = 0x80
    assert isr.isr_validate_model(bytes(bad)) == isr.ISR_ERR_FORMAT
    # multiplier below 2^30
    from synth.models import NetBuilder
    b = NetBuilder(rng=np.random.default_rng(0), in_shape=(3, 8, 8), num_classes=3)
    t = b.tensor(3, 8, 8, 0, 50.0)
    u = b.conv(t, 4, 3, 1, 1, True, m0=(1 << 30) - 1)
    b.fc(b.gap(u), 3)
    assert isr.isr_validate_model(b.blob()) == isr.ISR_ERR_FORMAT
    # unsupported but well-formed: input width not a multiple of 4
    b = NetBuilder(rng=np.random.default_rng(0), in_shape=(3, 6, 6), num_classes=3)
    t = b.tensor(3, 6, 6, 0, 50.0)
    u = b.conv(t, 4, 3, 1, 1, True)
    b.fc(b.gap(u), 3)
    assert isr.isr_validate_model(b.blob()) == isr.ISR_ERR_UNSUPPORTED


def test_discrete_quantile_matches_the_oracle():
    """Integer-only certification tail (Thm 3.2): the library's table lookup against
    the oracle's on random levels, levels next to table entries, and the edges."""
    from oracle import stats
    rng = np.random.default_rng(77)
    for sigma in (1, 2, 32, 64, 128, 256, 1024):
        T, R = oracle.noise_table(sigma)
        ps = list(rng.uniform(0.0, 1.0, 30)) + [0.0, 0.5, 1.0, 1 - 2.0 ** -53, 2.0 ** -60]
        # levels at and just around a few table entries (floor(2^64 p) == T[i] exactly where representable)
        for i in rng.integers(0, len(T), 6):
            ps.append(float(int(T[i]) >> 11 << 11) / 2.0 ** 64)
        for p in ps:
            t, r2 = isr.isr_discrete_quantile(sigma, float(p))
            want = stats.discrete_quantile(sigma, float(p))
            assert t == want, (sigma, p, t, want)
            assert r2 == stats.radius_squared_int(sigma, float(p))
    with pytest.raises(isr.IsrError):
        isr.isr_discrete_quantile(0, 0.9)
    with pytest.raises(isr.IsrError):
        isr.isr_discrete_quantile(32, 1.5)


def test_certified_metrics_match_the_oracle():
    """CP and CA of the paper's evaluation section: library against the oracle on random
    result lists, plus the empty-denominator and argument cases."""
    rng = np.random.default_rng(17)
    for trial in range(20):
        L = int(rng.integers(1, 60))
        labels = rng.integers(0, 5, size=L)
        classes = np.where(rng.random(L) < 0.6, labels, rng.integers(0, 5, size=L))
        classes = np.where(rng.random(L) < (0.3 if trial else 1.0), ostats.ABSTAIN, classes)
        radii = np.where(classes == ostats.ABSTAIN, 0.0, np.round(rng.random(L) * 50, 1))
        results = [isr.Result(int(c), float(r), 0.9, 10, 0) for c, r in zip(classes, radii)]
        grid = [0.0, 0.1, 5.0, 25.0, 49.9, 50.0, 60.0]
        cp, ca = isr.isr_certified_metrics(results, labels, grid)
        assert cp == ostats.certified_percentage(classes)
        for r, a in zip(grid, ca):
            assert a == ostats.certified_accuracy(classes, radii, labels, r)
    cp, ca = isr.isr_certified_metrics([isr.Result(1, 2.0, 0.9, 5, 0)], [1], [])
    assert cp == 1.0 and ca.size == 0
    res = (isr.Result * 1)(isr.Result(1, 2.0, 0.9, 5, 0))
    assert isr.lib().isr_certified_metrics(res, None, 0, None, 0, None, None) == isr.ISR_ERR_ARG
    assert isr.lib().isr_certified_metrics(res, None, 1, None, 2, None, None) == isr.ISR_ERR_ARG
