"""GPU parity of the OF-MLMC estimator kernels against the oracle, given
identical sample QoIs: relative difference <= 1e-12."""
import numpy as np
import pytest

import oracle.mlmc as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1705_04374_amd import capi
    c = capi.Context(0)
    yield c
    c.close()


def toy_terms(L, Ms, seed):
    rng = np.random.default_rng(seed)
    terms = []
    for l in range(L + 1):
        Y, Z = rng.normal(size=(2, Ms[l]))
        qf = 3.0 + Y + 0.7 * 2.0 ** -l * Z
        qc = 3.0 + Y + 0.7 * 2.0 ** -(l - 1) * Z if l else None
        ok = (rng.uniform(size=Ms[l]) > 0.05).astype(np.int32)
        terms.append((qf, qc, ok))
    return terms


@pytest.mark.parametrize("L,Ms", [(1, [4000, 300]), (3, [65536, 2000, 100, 7])])
def test_estimator_matches_oracle(ctx, L, Ms):
    import torch
    from paper_1705_04374_amd import capi
    terms = toy_terms(L, Ms, L)
    W = np.array([8.0 ** l * (1.0 if l == 0 else 1.125) for l in range(L + 1)])
    mom = torch.zeros((L + 1, 6), dtype=torch.float64, device="cuda")
    refs = []
    for l, (qf, qc, ok) in enumerate(terms):
        tf = torch.tensor(qf, device="cuda")
        tc = torch.tensor(qc, device="cuda") if qc is not None else None
        tok = torch.tensor(ok, device="cuda")
        capi.ofm_mlmc_moments(ctx, tf, tc, tok, mom[l])
        refs.append(O.term_moments(qf, qc, ok.astype(bool)))
    m = mom.cpu().numpy()
    for l, r in enumerate(refs):
        got = dict(M=m[l, 0], mean_f=m[l, 1], mean_c=m[l, 2], Vf=m[l, 3], Vc=m[l, 4], C=m[l, 5])
        for k in ("mean_f", "mean_c", "Vf", "Vc", "C"):
            assert abs(got[k] - r[k]) <= 1e-12 * max(abs(r[k]), 1e-300), (l, k)
        assert got["M"] == r["M"]
    Vf = [r["Vf"] for r in refs]
    Vc = [r["Vc"] for r in refs]
    Cv = [r["C"] for r in refs]
    a_ref = O.coefficients(Vf, Vc, Cv, W)
    Wd = torch.tensor(W, device="cuda")
    alpha = torch.zeros(L + 1, dtype=torch.float64, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    capi.ofm_ofmlmc_coefficients(ctx, L, mom, Wd, alpha, flag)
    a = alpha.cpu().numpy()
    assert flag.item() == 0
    np.testing.assert_allclose(a, a_ref, rtol=1e-12)
    sig = torch.zeros(L + 1, dtype=torch.float64, device="cuda")
    eps2 = torch.zeros(1, dtype=torch.float64, device="cuda")
    capi.ofm_ofmlmc_errors(ctx, L, mom, alpha, sig, eps2)
    s_ref = O.term_variances(Vf, Vc, Cv, a_ref)
    np.testing.assert_allclose(sig.cpu().numpy(), s_ref, rtol=1e-12)
    e_ref = O.error2(s_ref, [r["M"] for r in refs])
    assert abs(eps2.item() - e_ref) <= 1e-12 * e_ref
    E = torch.zeros(1, dtype=torch.float64, device="cuda")
    capi.ofm_ofmlmc_estimate(ctx, L, mom, alpha, E)
    E_ref = O.estimate([r["mean_f"] for r in refs], [r["mean_c"] for r in refs], a_ref)
    assert abs(E.item() - E_ref) <= 1e-12 * abs(E_ref)
    # allocation, both modes
    have = torch.tensor([r["M"] for r in refs], dtype=torch.int64, device="cuda")
    out = torch.zeros(L + 1, dtype=torch.int64, device="cuda")
    for mode, target in ((capi.OFM_MODE_TOLERANCE, 0.003), (capi.OFM_MODE_BUDGET, 1.0e6)):
        capi.ofm_ofmlmc_optimal_M(ctx, L, sig, Wd, have, mode, target, out, flag)
        ref = O.optimal_samples(list(s_ref), list(W), [r["M"] for r in refs],
                                "tol" if mode == capi.OFM_MODE_TOLERANCE else "budget", target)
        assert out.cpu().tolist() == ref and flag.item() == 0


@pytest.mark.parametrize("M", [1, 2, 63, 256, 1023, 1024, 2048, 8192, 8193, 20001])
@pytest.mark.parametrize("paired", [True, False])
def test_moments_at_the_edges_of_their_launches(ctx, M, paired):
    """Fewer samples than threads, exactly one and one more group of loads,
    both workgroup sizes; samples left out are NaN (<= 1e-12 relative)."""
    import torch
    from paper_1705_04374_amd import capi
    rng = np.random.default_rng(M)
    y = rng.normal(size=M)
    qf, qc = 3.0 + y, (5.0 + y + 0.5 * rng.normal(size=M)) if paired else None
    ok = (np.arange(M) % 7 != 3).astype(np.int32)
    for use in (ok, None):
        r = O.term_moments(qf, qc, None if use is None else use.astype(bool))
        bad = np.zeros(M, bool) if use is None else use == 0
        t = [None if q is None else torch.tensor(np.where(bad, np.nan, q), device="cuda") for q in (qf, qc)]
        out = torch.full((6,), -1.0, dtype=torch.float64, device="cuda")
        capi.ofm_mlmc_moments(ctx, t[0], t[1], None if use is None else torch.tensor(use, device="cuda"), out)
        got = out.cpu().tolist()
        assert got[0] == r["M"]
        for g, k in zip(got[1:], ("mean_f", "mean_c", "Vf", "Vc", "C")):
            assert abs(g - r[k]) <= 1e-12 * max(abs(r[k]), 1e-300), (k, g, r[k])


@pytest.mark.parametrize("M", [2047, 2049, 6144, 8191, 8192])
def test_moments_around_the_line_between_their_launches(ctx, M):
    """One to four groups of loads a thread, and the first launch of sixteen
    wavefronts, with the last sample left out (<= 1e-12 relative)."""
    import torch
    from paper_1705_04374_amd import capi
    rng = np.random.default_rng(M)
    y = rng.normal(size=M)
    qf, qc = 3.0 + y, 5.0 + y + 0.5 * rng.normal(size=M)
    ok = np.ones(M, np.int32)
    ok[-1] = 0
    r = O.term_moments(qf, qc, ok.astype(bool))
    out = torch.full((6,), -1.0, dtype=torch.float64, device="cuda")
    capi.ofm_mlmc_moments(ctx, *(torch.tensor(v, device="cuda") for v in (qf, qc, ok)), out)
    got = out.cpu().tolist()
    assert got[0] == r["M"] == M - 1
    for g, k in zip(got[1:], ("mean_f", "mean_c", "Vf", "Vc", "C")):
        assert abs(g - r[k]) <= 1e-12 * max(abs(r[k]), 1e-300), (k, g, r[k])


@pytest.mark.parametrize("L", [0, 1, 5, 31])
def test_sample_counts_with_terms_fixed_in_turn(ctx, L):
    """Terms that hold more samples than their optimum are fixed one after
    another, up to the largest number of terms; and a tolerance that the kept
    terms exhaust: what is held, flagged."""
    import torch
    from paper_1705_04374_amd import capi
    rng = np.random.default_rng(L)
    sig = 4.0 ** -np.arange(L + 1) * rng.uniform(0.5, 1.5, L + 1)
    W = 1.7 ** np.arange(L + 1) * rng.uniform(0.5, 1.5, L + 1)
    have = rng.integers(1, 400, L + 1)
    dev = [torch.tensor(v, device="cuda") for v in (sig, W, have)]
    out = torch.zeros(L + 1, dtype=torch.int64, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    spent = float(np.sum(have * W))
    for mode, name, target in [(capi.OFM_MODE_TOLERANCE, "tol", t) for t in (0.02, 0.1, 0.4)] + \
                              [(capi.OFM_MODE_BUDGET, "budget", b * spent) for b in (0.5, 1.1, 3.0)]:
        capi.ofm_ofmlmc_optimal_M(ctx, L, *dev, mode, target, out, flag)
        try:
            ref, infeasible = O.optimal_samples(list(sig), list(W), have.tolist(), name, target), False
        except O.InfeasibleTolerance:
            ref, infeasible = have.tolist(), True
        assert (flag.item() == capi.OFM_EINFEASIBLE) == infeasible
        assert out.cpu().tolist() == ref, (name, target)


def test_singular_system_falls_back_to_ones(ctx):
    import torch
    from paper_1705_04374_amd import capi
    mom = torch.zeros((3, 6), dtype=torch.float64, device="cuda")
    mom[:, 0] = 10
    alpha = torch.zeros(3, dtype=torch.float64, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    capi.ofm_ofmlmc_coefficients(ctx, 2, mom, torch.ones(3, dtype=torch.float64, device="cuda"), alpha, flag)
    assert flag.item() == capi.OFM_ESINGULAR
    assert alpha.cpu().tolist() == [1.0, 1.0, 1.0]


@pytest.mark.parametrize("Ms,first", [([65536, 2000, 300, 40, 1], 1), ([4000, 900, 120, 9, 1, 1], 0),
                                      ([5000, 700, 60, 12], 1)])
def test_indicator_fit_matches_oracle(ctx, Ms, first):
    """Inferred level-difference variances (App. A.1) and the completed
    moments of the terms with fewer than two samples: <= 1e-12 relative."""
    import torch
    from paper_1705_04374_amd import capi
    L = len(Ms) - 1
    terms = toy_terms(L, Ms, 7 + L)
    mom = torch.zeros((L + 1, 6), dtype=torch.float64, device="cuda")
    refs = []
    for l, (qf, qc, ok) in enumerate(terms):
        ok = np.ones_like(ok)
        capi.ofm_mlmc_moments(ctx, torch.tensor(qf, device="cuda"),
                              torch.tensor(qc, device="cuda") if qc is not None else None,
                              torch.tensor(ok, device="cuda"), mom[l])
        refs.append(O.term_moments(qf, qc, ok.astype(bool)))
    v_ref, ok_ref = O.fit_indicators([r["M"] for r in refs],
                                     [r["Vf"] + r["Vc"] - 2 * r["C"] for r in refs], first)
    assert ok_ref
    O.infer_missing_terms(refs, v_ref, first)
    v_hat = torch.full((L + 1,), -1.0, dtype=torch.float64, device="cuda")
    flag = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    capi.ofm_ofmlmc_fit_indicators(ctx, L, first, 2, mom, v_hat, flag)
    assert flag.item() == 0
    np.testing.assert_allclose(v_hat.cpu().numpy(), v_ref, rtol=1e-12, atol=0)
    m = mom.cpu().numpy()
    for l, r in enumerate(refs):
        for j, k in ((3, "Vf"), (4, "Vc"), (5, "C")):
            assert abs(m[l, j] - r[k]) <= 1e-12 * max(abs(r[k]), 1e-300), (l, k)
    # the completed finest terms are valid covariances whose difference
    # variance is the inferred one, or the smallest the correlation allows
    for l in range(max(first, 1), L + 1):
        if Ms[l] < 2:
            assert m[l, 5] ** 2 <= m[l, 3] * m[l, 4] * (1 + 1e-12)
            assert m[l, 3] + m[l, 4] - 2 * m[l, 5] >= v_ref[l] * (1 - 1e-10)


def test_indicator_fit_needs_two_terms(ctx):
    import torch
    from paper_1705_04374_amd import capi
    mom = torch.zeros((3, 6), dtype=torch.float64, device="cuda")
    mom[:, 0] = torch.tensor([100.0, 50.0, 1.0], dtype=torch.float64)
    mom[:, 3] = 2.0
    mom[1, 4] = 1.5
    mom[1, 5] = 1.0
    before = mom.clone()
    v_hat = torch.full((3,), -1.0, dtype=torch.float64, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    capi.ofm_ofmlmc_fit_indicators(ctx, 2, 1, 2, mom, v_hat, flag)
    assert flag.item() == capi.OFM_ESINGULAR
    assert v_hat.cpu().tolist() == [0.0, 0.0, 0.0]
    assert torch.equal(mom, before)
    _, ok = O.fit_indicators([100, 50, 1], [2.0, 1.5, 0.0], 1)
    assert not ok


@pytest.mark.parametrize("C1", [-0.6, 0.6])
def test_indicator_fit_completion_with_signed_correlation_below(ctx, C1):
    """The completion of a single-sample finest term when the term below has
    a negative (or positive) correlation: the device fit and completion
    equal the oracle's on the same moments (<= 1e-12), for an inferred
    difference variance above and below the smallest one the correlation
    allows."""
    import torch
    from paper_1705_04374_amd import capi
    for V2 in (0.05, 30.0):
        rows = [[100.0, 1.0, 0.0, 4.0, 0.0, 0.0], [50.0, 2.0, 1.0, 1.0, 1.0, C1],
                [20.0, 3.0, 2.0, 0.5 * V2, 0.5 * V2, 0.25 * V2 * (1 if C1 > 0 else -1)],
                [1.0, 4.0, 3.0, 0.0, 0.0, 0.0]]
        mom = torch.tensor(rows, dtype=torch.float64, device="cuda")
        refs = [dict(M=r[0], mean_f=r[1], mean_c=r[2], Vf=r[3], Vc=r[4], C=r[5]) for r in rows]
        v_ref, ok = O.fit_indicators([r["M"] for r in refs], [r["Vf"] + r["Vc"] - 2 * r["C"] for r in refs], 1)
        assert ok
        O.infer_missing_terms(refs, v_ref, 1)
        v_hat = torch.full((4,), -1.0, dtype=torch.float64, device="cuda")
        flag = torch.full((1,), -7, dtype=torch.int32, device="cuda")
        capi.ofm_ofmlmc_fit_indicators(ctx, 3, 1, 2, mom, v_hat, flag)
        assert flag.item() == 0
        np.testing.assert_allclose(v_hat.cpu().numpy(), v_ref, rtol=1e-12, atol=0)
        m = mom.cpu().numpy()
        for j, k in ((3, "Vf"), (4, "Vc"), (5, "C")):
            assert abs(m[3, j] - refs[3][k]) <= 1e-12 * max(abs(refs[3][k]), 1e-300), (V2, k, m[3, j], refs[3][k])


@pytest.mark.parametrize("m_floor", [2, 3, 6])
def test_indicator_fit_keeps_the_inferred_variance_as_a_floor(ctx, m_floor):
    """Terms with at least two but fewer than m_floor samples keep the
    inferred difference variance as a floor of their measured one (App.
    A.1): the device result equals the oracle's fit, completion and
    refinement of the same moments (<= 1e-12), for a measured variance below
    the inferred one, one whose inferred value needs a covariance beyond
    -sqrt(Vf Vc), and one above it (unchanged)."""
    import torch
    from paper_1705_04374_amd import capi
    for V3 in (1e-4, 1e-9, 50.0):
        rows = [[400.0, 1.0, 0.0, 4.0, 0.0, 0.0], [100.0, 2.0, 1.0, 1.0, 1.0, 0.8],
                [30.0, 3.0, 2.0, 0.5, 0.5, 0.45], [4.0, 4.0, 3.0, 0.3 + V3, 0.3, 0.3],
                [1.0, 5.0, 4.0, 0.0, 0.0, 0.0]]
        if V3 == 1e-9:
            rows[3][3:6] = [1e-6, 1e-6, 1e-6]      # tiny members: the bound binds
        mom = torch.tensor(rows, dtype=torch.float64, device="cuda")
        refs = [dict(M=r[0], mean_f=r[1], mean_c=r[2], Vf=r[3], Vc=r[4], C=r[5]) for r in rows]
        v_ref, ok = O.fit_indicators([r["M"] for r in refs], [r["Vf"] + r["Vc"] - 2 * r["C"] for r in refs], 1)
        assert ok
        O.infer_missing_terms(refs, v_ref, 1)
        O.refine_few_sample_terms(refs, v_ref, 1, m_floor)
        v_hat = torch.full((5,), -1.0, dtype=torch.float64, device="cuda")
        flag = torch.full((1,), -7, dtype=torch.int32, device="cuda")
        capi.ofm_ofmlmc_fit_indicators(ctx, 4, 1, m_floor, mom, v_hat, flag)
        assert flag.item() == 0
        np.testing.assert_allclose(v_hat.cpu().numpy(), v_ref, rtol=1e-12, atol=0)
        m = mom.cpu().numpy()
        for l in range(5):
            for j, k in ((3, "Vf"), (4, "Vc"), (5, "C")):
                assert abs(m[l, j] - refs[l][k]) <= 1e-12 * max(abs(refs[l][k]), 1e-300), (V3, l, k)
        v3 = m[3, 3] + m[3, 4] - 2 * m[3, 5]
        if m_floor > 4 and V3 != 50.0:
            # refined: at the inferred value, or as close as a covariance allows
            assert v3 >= min(v_ref[3], (np.sqrt(m[3, 3]) + np.sqrt(m[3, 4])) ** 2) * (1 - 1e-12)
            assert m[3, 5] >= -np.sqrt(m[3, 3] * m[3, 4]) * (1 + 1e-12)
        else:
            assert abs(v3 - (rows[3][3] + rows[3][4] - 2 * rows[3][5])) <= 1e-15 * max(1.0, v3)


def test_merged_shard_moments_match_the_whole(ctx):
    """Per-shard moments merged on the device (the reduction of a per-GPU
    all-reduce) equal the moments of all samples and the oracle's merge."""
    import torch
    from paper_1705_04374_amd import capi
    L = 3
    Ms = [9000, 700, 90, 12]
    terms = toy_terms(L, Ms, 5)
    whole = torch.zeros((L + 1, 6), dtype=torch.float64, device="cuda")
    acc = torch.zeros((L + 1, 6), dtype=torch.float64, device="cuda")    # M = 0: empty
    part = torch.zeros((L + 1, 6), dtype=torch.float64, device="cuda")
    refs = [None] * (L + 1)
    for l, (qf, qc, ok) in enumerate(terms):
        tok = torch.tensor(ok, device="cuda")
        capi.ofm_mlmc_moments(ctx, torch.tensor(qf, device="cuda"),
                              torch.tensor(qc, device="cuda") if qc is not None else None, tok, whole[l])
    # four shards of uneven sizes (one empty for the last term), merged in place
    for s in range(4):
        for l, (qf, qc, ok) in enumerate(terms):
            cut = np.linspace(0, Ms[l], 5).astype(int)
            if l == L:
                cut[2] = cut[3]                         # an empty third shard
            lo, hi = cut[s], cut[s + 1]
            sl = slice(lo, hi)
            if hi > lo:
                capi.ofm_mlmc_moments(ctx, torch.tensor(qf[sl], device="cuda"),
                                      torch.tensor(qc[sl], device="cuda") if qc is not None else None,
                                      torch.tensor(ok[sl], device="cuda"), part[l])
            else:
                part[l].zero_()
            r = O.term_moments(qf[sl], qc[sl] if qc is not None else None, ok[sl].astype(bool))
            refs[l] = r if refs[l] is None else O.merge_moments(refs[l], r)
        capi.ofm_mlmc_merge_moments(ctx, acc, part, acc)
    got, want = acc.cpu().numpy(), whole.cpu().numpy()
    assert np.array_equal(got[:, 0], want[:, 0])
    np.testing.assert_allclose(got[:, 1:], want[:, 1:], rtol=1e-12, atol=0)
    for l, r in enumerate(refs):
        for j, k in ((1, "mean_f"), (2, "mean_c"), (3, "Vf"), (4, "Vc"), (5, "C")):
            assert abs(got[l, j] - r[k]) <= 1e-12 * max(abs(r[k]), 1e-300), (l, k)
