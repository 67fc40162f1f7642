"""The fp32 mode's pair kernel on two fp16 parts per operand, where that form has edges of its own: every kind of last block,
rows whose scale the kernel has to find and to move while it goes over the samples, coordinates beyond the fp16 range."""
import numpy as np
import pytest

import oracle
import sdkde_inputs
from parity import assert_laplace_close, gram_exponent_error, score_resolution
from test_gpu_split_kernel import _score_bound

pytestmark = pytest.mark.gpu


def _gpu(*arrays):
    import torch
    return [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda() for a in arrays]


@pytest.mark.parametrize("d", [8, 9, 15, 17, 24, 25, 40, 41, 48, 56, 65, 72, 73, 85, 104, 105, 112, 120, 127])
@pytest.mark.parametrize("n", [33, 2100])
def test_every_kind_of_last_block(n, d):
    """One to eight columns beyond whole 32-column blocks take one matrix instruction, nine to sixteen two, the rows' constant
    terms in their spare columns; 17 to 24 columns of a 32-column block have spare columns, too; other dimensions have none.  At
    the samples, at points, densities, shifted sums."""
    import paper_2602_10378_amd as P
    P.load()
    m = 45
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=4, seed=n + d)
    h = float(h)
    print(f"last block n={n} m={m} d={d}", flush=True)
    xd, qd = _gpu(x, q)
    s = P.sdkde_score(xd, h).cpu().numpy()
    err = np.linalg.norm(s - oracle.score(x, h), axis=1)
    assert np.all(err <= _score_bound(x, x, h)), (err / _score_bound(x, x, h)).max()
    ref, e = oracle.eval_log_density(x, q, h), gram_exponent_error(x, q, h)
    ref_s, bound = oracle.score(x, h, points=q), _score_bound(x, q, h)
    for flags in (0, P.SDKDE_FLAG_MAX_SHIFT):
        err = np.linalg.norm(P.sdkde_score(xd, h, points=qd, flags=flags).cpu().numpy() - ref_s, axis=1)
        assert np.all(err <= bound), (err / bound).max()
        logd = P.sdkde_eval(xd, qd, h, want="log", flags=flags)[1].cpu().numpy()
        assert np.all(np.abs(logd - ref) <= e + 2.0**-18 + 2.0**-23 * np.abs(ref))
        lap = P.sdkde_eval_laplace(xd, qd, h, flags=flags).cpu().numpy()
        assert_laplace_close(lap, oracle.eval_laplace_density(x, q, h), oracle.eval_laplace_abs_density(x, q, h), "laplace", e, np.exp(ref))


@pytest.mark.parametrize("d", [8, 16, 32, 48, 64, 128])
@pytest.mark.parametrize("splits", [1, 8])
def test_rows_whose_weights_grow_along_the_samples(tuning, d, splits):
    """Samples in the order of their distance from one of them, farthest first: a row's largest weight grows by up to 2^100
    from one chunk to another, its scale has to follow, and what was summed before must count for what it is; then nearest
    first, where most of what follows is negligible.  Exact duplicates of far samples come last: a weight of one for rows that
    had only tiny ones."""
    import paper_2602_10378_amd as P
    P.load()
    n, h = 1500, 1.0
    rng = np.random.default_rng(d)
    step = rng.standard_normal((n, d)) / np.sqrt(d)
    x = (step * np.linspace(0.05, 11.0, n)[:, None]).astype(np.float32)
    tuning(P.SDKDE_TUNE_SCORE_SPLITS, splits)
    for name, order in (("farthest first", np.arange(n)[::-1]), ("nearest first", np.arange(n))):
        y = np.concatenate([x[order], x[[5, n - 1, n - 40]]])
        print(f"growing weights d={d} splits {splits} {name}", flush=True)
        yd, = _gpu(y)
        err = np.linalg.norm(P.sdkde_score(yd, h).cpu().numpy() - oracle.score(y, h), axis=1)
        assert np.all(err <= _score_bound(y, y, h)), (err / _score_bound(y, y, h)).max()
        q = (0.98 * y[::7] + 0.01).astype(np.float32)
        err = np.linalg.norm(P.sdkde_score(yd, h, points=_gpu(q)[0]).cpu().numpy() - oracle.score(y, h, points=q), axis=1)
        assert np.all(err <= _score_bound(y, q, h)), (err / _score_bound(y, q, h)).max()


@pytest.mark.parametrize("d", [9, 32])
def test_many_tiny_weights_beside_a_large_one(d):
    """Every sample has an exact duplicate (weight one, no pull) and thousands of neighbours of weight about 2^-30: the score
    is theirs alone.  Weights are resolved far below the row's largest, so the only error is that of two sums that cancel."""
    import paper_2602_10378_amd as P
    P.load()
    n, h = 6000, 1.0
    rng = np.random.default_rng(d)
    x = rng.standard_normal((n // 2, d))
    x *= np.sqrt(30.0 * np.log(2.0)) / np.linalg.norm(x, axis=1, keepdims=True)      # pairs at sqrt(2) times that on average
    x = np.concatenate([x, x]).astype(np.float32)
    print(f"duplicates among tiny weights d={d}", flush=True)
    err = np.linalg.norm(P.sdkde_score(_gpu(x)[0], h).cpu().numpy() - oracle.score(x, h), axis=1)
    assert np.all(err <= _score_bound(x, x, h)), (err / _score_bound(x, x, h)).max()


@pytest.mark.parametrize("d", [4, 8, 16, 32, 37])
def test_queries_beyond_the_fp16_range(d):
    """Queries up to 10^9 bandwidths away: zero density without the shift, and with it the log density and the score of the
    nearest samples, to what fp32 exponents of that size resolve.  A few of them share a workgroup with ordinary queries."""
    import paper_2602_10378_amd as P
    P.load()
    n, m = 700, 150
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=d)
    h = float(h)
    far = np.arange(3, m, 16)
    q[far] *= np.geomspace(1e4, 1e9, len(far), dtype=np.float32)[:, None] * h / np.linalg.norm(q[far], axis=1, keepdims=True)
    near = np.setdiff1d(np.arange(m), far)
    print(f"far queries n={n} m={m} d={d}", flush=True)
    xd, qd = _gpu(x, q)
    ref, e = oracle.eval_log_density(x, q, h), gram_exponent_error(x, q, h)
    logd = P.sdkde_eval(xd, qd, h, want="log")[1].cpu().numpy()
    assert np.all(np.abs(logd - ref)[near] <= e[near] + 2.0**-18 + 2.0**-23 * np.abs(ref[near]))
    assert np.all(np.isneginf(logd[far]))
    logd = P.sdkde_eval(xd, qd, h, want="log", flags=P.SDKDE_FLAG_MAX_SHIFT)[1].cpu().numpy()
    assert np.all(np.abs(logd - ref) <= e + 2.0**-18 + 2.0**-23 * np.abs(ref)), (np.abs(logd - ref) / (e + 2.0**-18)).max()
    if d > 6:
        ref_s = oracle.score(x, h, points=q)
        s = P.sdkde_score(xd, h, points=qd).cpu().numpy()
        assert np.all(s[far] == 0.0)
        assert np.all(np.linalg.norm(s - ref_s, axis=1)[near] <= _score_bound(x, q, h)[near])
        s = P.sdkde_score(xd, h, points=qd, flags=P.SDKDE_FLAG_MAX_SHIFT).cpu().numpy()
        # a score of about |q| / h^2: the weights of the far queries' nearest samples are not resolved, their distance is
        spread = np.linalg.norm(x - x.mean(axis=0), axis=1).max() * 2.0 / (h * h)
        assert np.all(np.linalg.norm(s - ref_s, axis=1)[far] <= spread + 2.0**-21 * np.linalg.norm(ref_s, axis=1)[far])
        assert np.all(np.linalg.norm(s - ref_s, axis=1)[near] <= _score_bound(x, q, h)[near])


@pytest.mark.parametrize("d", [8, 16, 37])
def test_a_sample_beyond_the_fp16_range_has_no_weight(d):
    """One sample's coordinate at 10^6 and 10^20 bandwidths (not one of the rows the centre is formed of): as without it."""
    import paper_2602_10378_amd as P
    P.load()
    n, m = 4500, 70
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=4, seed=d)
    h = float(h)
    rest = x[:-1]
    logd_ref, e = oracle.eval_log_density(rest, q, h) + np.log((n - 1) / n), gram_exponent_error(rest, q, h)
    for value in (1e6 * h, -1e20):
        y = x.copy()
        y[-1, d // 2] = value
        print(f"sample at {value:.0e} d={d}", flush=True)
        yd, qd = _gpu(y, q)
        for flags in (0, P.SDKDE_FLAG_MAX_SHIFT):
            logd = P.sdkde_eval(yd, qd, h, want="log", flags=flags)[1].cpu().numpy()
            assert np.all(np.abs(logd - logd_ref) <= e + 2.0**-18 + 2.0**-23 * np.abs(logd_ref))
        err = np.linalg.norm(P.sdkde_score(yd, h).cpu().numpy()[:-1] - oracle.score(rest, h), axis=1)
        assert np.all(err <= _score_bound(rest, rest, h))


@pytest.mark.parametrize("d", [8, 16, 32])
def test_points_that_are_not_finite(d):
    """A query with an infinite or NaN coordinate gets NaN, its neighbours in the tile what they get without it."""
    import paper_2602_10378_amd as P
    P.load()
    n, m = 900, 40
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=d)
    h = float(h)
    xd, qd = _gpu(x, q)
    want = P.sdkde_eval(xd, qd, h, want="log")[1].cpu().numpy()
    q[7, d - 1], q[22, 0] = np.inf, np.nan
    print(f"points that are not finite d={d}", flush=True)
    for flags in (0, P.SDKDE_FLAG_MAX_SHIFT):
        got = P.sdkde_eval(xd, _gpu(q)[0], h, want="log", flags=flags)[1].cpu().numpy()
        assert np.isnan(got[[7, 22]]).all()
        rest = np.setdiff1d(np.arange(m), [7, 22])
        assert np.all(np.abs(got[rest] - want[rest]) <= 1e-4)


@pytest.mark.parametrize("d", [17, 32, 44, 48, 90, 128])
def test_shift_from_leading_products(d):
    """The shift of max-shifted sums comes from leading products up to a squared norm of 4096 and from all of them beyond: points
    on both sides of that line, some of them far from every sample, one wave's rows mixed and not."""
    import paper_2602_10378_amd as P
    P.load()
    rng = np.random.default_rng(d)
    n, m, h = 1500, 700, 0.5
    x = rng.standard_normal((n, d)) * 2.0
    x[: n // 3] += 30.0 / np.sqrt(d)                              # clusters: samples with large norms, too
    q = rng.standard_normal((m, d))
    radius = np.repeat([1.0, 15.0, 26.0, 27.0, 40.0, 200.0], m // 6 + 1)[:m]     # 64 in units of h / sqrt(log2 e): 26.6
    radius[m // 2:] = rng.permutation(radius[m // 2:])
    q *= (radius / np.linalg.norm(q, axis=1))[:, None]
    x, q = x.astype(np.float32), q.astype(np.float32)
    print(f"leading products d={d}", flush=True)
    xd, qd = _gpu(x, q)
    flags = P.SDKDE_FLAG_MAX_SHIFT
    ref, e = oracle.eval_log_density(x, q, h), gram_exponent_error(x, q, h)
    logd = P.sdkde_eval(xd, qd, h, want="log", flags=flags)[1].cpu().numpy()
    assert np.all(np.abs(logd - ref) <= e + 2.0**-18 + 2.0**-23 * np.abs(ref))
    bound = _score_bound(x, q, h)
    err = np.linalg.norm(P.sdkde_score(xd, h, points=qd, flags=flags).cpu().numpy() - oracle.score(x, h, points=q), axis=1)
    assert np.all(err <= bound), (err / bound).max()


@pytest.mark.parametrize("n,m,d,splits", [(5000, 100, 16, 1), (5000, 100, 40, 1), (5000, 100, 64, 1), (2000, 4200, 16, 0)])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_a_point_that_is_not_a_number_leaves_the_others_their_scales(tuning, n, m, d, splits, value):
    """Rows r and r + 16 of a wave share a lane, and one test of whether a weight has outgrown its row's scale.  Here row 17's near
    samples come last, so that its scale has to be raised, and row 1's weights are NaN."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    tuning(P.SDKDE_TUNE_SCORE_SPLITS, splits)
    rng = np.random.default_rng(d)
    x, q = rng.standard_normal((n, d)).astype(np.float32), rng.standard_normal((m, d)).astype(np.float32)
    h = 0.5 * d**0.5
    away = np.float32(10.0 * h / d**0.5)                      # e^-50 between the two groups
    x[3 * n // 4:] += away
    q[17::32] += away
    xd, qd = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda()
    print(f"scales beside NaN n={n} m={m} d={d} {value}", flush=True)
    want = P.sdkde_score(xd, h, points=qd)
    qd[1::32, d // 2] = value
    got = P.sdkde_score(xd, h, points=qd)
    keep = np.arange(m) % 32 != 1
    # (a scale that is raised at another chunk is another rounding of the row's term)
    err = (got - want).norm(dim=1).cpu().numpy()[keep]
    assert np.all(err <= score_resolution(x, q[keep], h))
