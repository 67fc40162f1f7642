"""The fp32 mode's two-part operands at the ends of their range: what is far from the centre, what only looks far, what is small."""
import numpy as np
import pytest

import oracle
import sdkde_inputs
from parity import gram_exponent_error

pytestmark = pytest.mark.gpu


def _inside(a):
    """The array as a view into a larger tensor, with other values before and behind it."""
    import torch
    rows, d = a.shape
    whole = torch.full((rows + 4096, d), 3.0e7, device="cuda", dtype=torch.float32)
    whole[1024:1024 + rows] = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    return whole[1024:1024 + rows]


def _prepared_scales(workspace, plan):
    """2^k of the prepared points (2^-k times themselves), behind their rows and the residuals of their norms."""
    import torch
    kb = plan["dp"] // 16
    at = plan["off_ps"] + plan["m_pad"] // 16 * (kb * 1024 + (kb % 2) * 256) + plan["m_pad"] * 4
    return workspace[at:at + plan["m_pad"] * 4].view(torch.float32).cpu().numpy()


@pytest.mark.parametrize("d", [4, 9, 16, 33, 128])
@pytest.mark.parametrize("flag", ["shifted", "plain"])
def test_an_offset_of_all_data_is_not_a_distance(d, flag):
    """All data 10^4 (shifted sums) or 10^5 bandwidths from the origin and close together: no point is far from the centre.
    Padding rows, which stand as zeros, must not be taken for far ones: a row taken for one is read again from the caller's
    array, and a padding row is not in it.  The arrays lie inside larger ones."""
    import paper_2602_10378_amd as P
    P.load()
    n, m = 1000, 75
    flags = P.SDKDE_FLAG_MAX_SHIFT if flag == "shifted" else 0
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=d)
    h = float(h)
    x, q = (a + np.float32(h * (1e4 if flags else 1e5)) for a in (x, q))
    print(f"offset data d={d} {flag}", flush=True)
    xd, qd = _inside(x), _inside(q)
    workspace = P.make_workspace(n, m, d, flags=flags)
    logd = P.sdkde_eval(xd, qd, h, want="log", workspace=workspace, flags=flags)[1].cpu().numpy()
    ref, e = oracle.eval_log_density(x, q, h), gram_exponent_error(x, q, h)
    assert np.all(np.abs(logd - ref) <= e + 2.0**-18 + 2.0**-23 * np.abs(ref))
    assert np.all(_prepared_scales(workspace, P.sdkde_describe_plan(n, m, d, 2, flags)) == 1.0)


def _two_clusters(n, m, d, distance, seed):
    """Samples in two tight clusters, 2 `distance` apart along one column; queries up to 50 from the centre that the library takes
    (the mean of evenly strided samples) and at least 1 from the clusters' middle along it, so that one of them is the nearer one by
    more than what fp32 exponents resolve; and the clusters' size."""
    rng = np.random.default_rng(seed)
    step, c = rng.standard_normal((n, d)), d // 2
    x = step.copy()
    x[:, c] += rng.choice([-distance, distance], n)
    rows = min(max(4096 // d, 32), n)
    q = x[:rows * (n // rows):n // rows].mean(axis=0) + rng.standard_normal((m, d))
    q[:, c] += rng.choice([-1.0, 1.0], m) * rng.uniform(0.0, 50.0, m)
    q[:, c] += np.where(np.abs(q[:, c]) < 1.0, 2.0, 0.0)
    return x.astype(np.float32), q.astype(np.float32), 2.0 * np.linalg.norm(step, axis=1).max()


def _check_shifted_far_points(P, x, q, h, size):
    """Max-shifted log densities and scores where every sample is far; size: how far the samples that may count are apart."""
    import torch
    xd, qd = (torch.from_numpy(a).cuda() for a in (x, q))
    flags = P.SDKDE_FLAG_MAX_SHIFT
    ref = oracle.eval_log_density(x, q, h)
    # roundings at the size of the terms, four more for the lane groups of a matrix instruction; coordinates held to 2^-23 of
    # themselves move an exponent by up to 2^-23 |x| |x - q| / h^2, twice 2^-23 of it here, and the result is rounded once
    allowed = gram_exponent_error(x, q, h, low_precision_inputs=True) + 3.0 * 2.0**-23 * np.abs(ref) + 2.0**-18
    logd = P.sdkde_eval(xd, qd, h, want="log", flags=flags)[1].cpu().numpy()
    worst = (np.abs(logd - ref) / allowed).max()
    print(f"log density {worst:.3f} of the bound", flush=True)
    assert worst <= 1.0
    if x.shape[1] > 6:
        # which of a cluster's samples count is not resolved, only that they do: their distances from each other
        ref_s = oracle.score(x, h, points=q)
        s = P.sdkde_score(xd, h, points=qd, flags=flags).cpu().numpy()
        spread = size / (h * h)
        worst = (np.linalg.norm(s - ref_s, axis=1) / (spread + 2.0**-21 * np.linalg.norm(ref_s, axis=1))).max()
        assert worst <= 1.0


@pytest.mark.parametrize("d", [7, 17, 32, 48, 128])
@pytest.mark.parametrize("distance", [200.0, 2000.0, 6000.0, 12000.0])
def test_shifted_sums_between_far_clusters(d, distance):
    """Every sample far from queries near the centre: the exponents are of the size of the samples' norms, and a shift from
    leading products only would miss the largest by more than fp32 exponents hold."""
    import paper_2602_10378_amd as P
    P.load()
    n, m, h = 1500, 400, 1.0
    print(f"far clusters d={d} distance {distance}", flush=True)
    x, q, size = _two_clusters(n, m, d, distance, d)
    _check_shifted_far_points(P, x, q, h, size)


@pytest.mark.parametrize("d", [4, 7, 16, 17, 24, 32, 37, 56, 128])
@pytest.mark.parametrize("spread", [12000.0, 25000.0, 45000.0])
def test_a_bandwidth_far_below_every_distance(d, spread):
    """Coordinates of up to some 10^4 bandwidths: inside the fp16 range one by one or just beyond, but their norms are beyond
    what a row's constant term takes in its spare columns.  Every pair is too far apart to count, so densities and scores are 0."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    n, m, h = 1100, 200, 1.0
    rng = np.random.default_rng(d)
    x, q = (rng.standard_normal((k, d)).astype(np.float32) * np.float32(spread) for k in (n, m))
    q[::2] *= np.float32(0.01)                                                 # rows on both sides of the line in one tile
    print(f"narrow bandwidth d={d} spread {spread}", flush=True)
    xd, qd = (torch.from_numpy(a).cuda() for a in (x, q))
    dens, logd = (a.cpu().numpy() for a in P.sdkde_eval(xd, qd, h, want="both"))
    assert np.all(dens == 0.0) and np.all(np.isneginf(logd))
    assert np.all(P.sdkde_eval_laplace(xd, qd, h).cpu().numpy() == 0.0)
    if d > 6:
        assert np.all(P.sdkde_score(xd, h).cpu().numpy() == 0.0)
        assert np.all(P.sdkde_score(xd, h, points=qd).cpu().numpy() == 0.0)


@pytest.mark.parametrize("d", [7, 37, 64, 128])
def test_shifted_sums_of_points_far_in_every_coordinate(d):
    """Points with coordinates of up to 2000 units each: far by their norm, 23000 at d = 128, though by no single coordinate.  Their
    exponents are rounded at the size of the norm, for the maximum and for the sums alike."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    n, m = 1500, 300
    rng = np.random.default_rng(d)
    h = float(np.sqrt(np.log2(np.e)))                                        # one unit is 1
    x = rng.standard_normal((n, d)).astype(np.float32)
    q = (rng.choice([-1.0, 1.0], (m, d)) * rng.uniform(1500.0, 2000.0, (m, d))).astype(np.float32)
    q[::3] *= np.float32(0.5)
    print(f"far in every coordinate d={d}", flush=True)
    _check_shifted_far_points(P, x, q, h, 2.0 * np.linalg.norm(x - x.mean(axis=0), axis=1).max())


@pytest.mark.parametrize("d", [4, 7, 17, 32, 48, 128])
@pytest.mark.parametrize("distance", [30000.0, 1e5, 1e7, 1e9])
def test_shifted_densities_where_every_sample_is_beyond_the_range(d, distance):
    """Two clusters beyond what the unshifted sums reach, queries between them, and some at the clusters' distance on other
    sides: their log densities are those of the nearest samples, to what fp32 exponents of that size resolve."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    n, m, h = 1500, 300, 1.0
    print(f"every sample beyond d={d} distance {distance}", flush=True)
    x, q, _ = _two_clusters(n, m, d, distance, d)
    q[1::5, 0] += np.float32(distance)
    xd, qd = (torch.from_numpy(a).cuda() for a in (x, q))
    flags = P.SDKDE_FLAG_MAX_SHIFT
    ref = oracle.eval_log_density(x, q, h)
    # as in _check_shifted_far_points; the samples a distance r away are as far from the centre, the queries up to that
    allowed = gram_exponent_error(x, q, h, low_precision_inputs=True) + 4.0 * 2.0**-23 * np.abs(ref)
    logd = P.sdkde_eval(xd, qd, h, want="log", flags=flags)[1].cpu().numpy()
    worst = (np.abs(logd - ref) / allowed).max()
    print(f"log density {worst:.3f} of the bound", flush=True)
    assert worst <= 1.0
    # the others take no notice of one such sample
    x, q, _ = _two_clusters(n, m, d, 5.0, d)
    ref, e = oracle.eval_log_density(x, q, h), gram_exponent_error(x, q, h)
    y = np.concatenate([x, np.zeros((1, d), np.float32)])
    y[-1, d - 1] = distance
    for f in (0, flags):
        logd = P.sdkde_eval(torch.from_numpy(y).cuda(), torch.from_numpy(q).cuda(), h, want="log", flags=f)[1].cpu().numpy()
        seen = np.isfinite(logd)
        assert seen.all() or f == 0
        assert np.all(np.abs(logd - ref - np.log(n / (n + 1)))[seen] <= (e + 2.0**-18 + 2.0**-23 * np.abs(ref))[seen])


def _column_bound(x, p, h):
    """Per point and column: an error e in every exponent moves a weight by e of itself (twice: numerator and denominator), the
    parts of a weight hold it to 2^-22 and sums round some more, 2^-20 of each term's pull in the column; and coordinates are held to
    2^-23 of themselves and of the column's spread, so the two sums that cancel to 2^-21 of the mean coordinate."""
    x, p = x.astype(np.float64), p.astype(np.float64)
    c = x.mean(axis=0)
    x, p = x - c, p - c
    r2 = np.maximum((p * p).sum(1)[:, None] + (x * x).sum(1)[None] - 2.0 * p @ x.T, 0.0)
    u = r2 / (2.0 * h * h)
    w = np.exp(-(u - u.min(axis=1, keepdims=True)))
    w /= w.sum(axis=1, keepdims=True)
    pull = np.stack([(w * np.abs(x[:, k] - p[:, k, None])).sum(1) for k in range(x.shape[1])], axis=1)
    e = 2.0 * gram_exponent_error(x, p, h)[:, None] + 2.0**-20
    return (e * pull + 2.0**-21 * (np.abs(p) + w @ np.abs(x) + x.std(axis=0))) / (h * h)


def _check_columns(P, x, q, h):
    import torch
    xd, qd = (torch.from_numpy(a).cuda() for a in (x, q))
    score, sd = torch.empty_like(xd), torch.empty_like(xd)
    P.sdkde_fit_eval(xd, qd, h, score_out=score, samples_sd_out=sd, log_density_out=torch.empty(len(q), device="cuda"))
    worst = []
    for got, at in ((P.sdkde_score(xd, h), x), (score, x), (P.sdkde_score(xd, h, points=qd), q),
                    (P.sdkde_score(xd, h, points=qd, flags=P.SDKDE_FLAG_MAX_SHIFT), q)):
        ref = oracle.score(x, h) if at is x else oracle.score(x, h, points=q)
        worst.append((np.abs(got.cpu().numpy() - ref) / _column_bound(x, at, h)).max())
    print("scores by column:", " ".join(f"{v:.3f}" for v in worst), "of the bound", flush=True)
    assert max(worst) <= 1.0


@pytest.mark.parametrize("d,n", [(7, 700), (7, 2100), (16, 700), (16, 2100), (17, 1100), (32, 700), (37, 2100), (64, 1100), (128, 500)])
def test_scores_of_columns_far_narrower_than_the_bandwidth(d, n):
    """Columns from as wide as the others to 10^-9 of that, and all of them 1000 times narrower than the bandwidth: two fp16
    parts resolve 2^-25 of a bandwidth, of which such a column's score is far more than the rounding."""
    import paper_2602_10378_amd as P
    P.load()
    m = 90
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=d)
    narrow = np.float32(10.0) ** -(np.arange(d) % 10).astype(np.float32)
    print(f"narrow columns n={n} d={d}", flush=True)
    _check_columns(P, x * narrow, q * narrow, float(h))
    _check_columns(P, x, q, 1000.0 * float(h))


@pytest.mark.parametrize("d", [7, 16, 17, 37, 64])
def test_a_value_far_outside_its_narrow_column(d):
    """A column 10^6 times narrower than the others, but for a few rows (none of those the centre is formed of) with values of
    the others' size: beyond the fp16 range in the column's unit."""
    import paper_2602_10378_amd as P
    P.load()
    n, m = 1300, 90
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=d)
    c = d // 2
    x[:, c] *= np.float32(1e-6)
    q[:, c] *= np.float32(1e-6)
    x[[1003, 1009, 1201], c] += np.array([1.0, -0.5, 2.0], dtype=np.float32) * np.float32(h)
    print(f"values outside a narrow column d={d}", flush=True)
    _check_columns(P, x, q, float(h))


@pytest.mark.parametrize("d", [7, 17, 32, 128])
@pytest.mark.parametrize("distance", [1e5, 1e7, 1e9])
def test_shifted_scores_where_every_sample_is_beyond_the_range(d, distance):
    """The score between two clusters beyond the fp16 range: the nearer one's samples, less the query."""
    import paper_2602_10378_amd as P
    P.load()
    n, m, h = 1500, 300, 1.0
    print(f"scores, every sample beyond d={d} distance {distance}", flush=True)
    x, q, size = _two_clusters(n, m, d, distance, d)
    q[1::2, d // 2] += np.float32(0.5 * distance)           # not only around the middle, where the nearer one is not resolved
    q[::2, d // 2] -= np.float32(0.5 * distance)
    _check_shifted_far_points(P, x, q, h, size + 2.0**-22 * distance)


@pytest.mark.parametrize("d", [4, 16, 37])
def test_prepared_samples_with_far_ones_serve_shifted_and_plain_calls(d):
    """Samples stand prepared by one call and serve others with and without the max shift, some of them beyond the fp16 range."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    n, m = 1500, 90
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=d)
    h = float(h)
    x[[1003, 1203]] += np.float32(1e5 * h)
    q[::4] += np.float32(0.999e5 * h)
    xd, qd = (torch.from_numpy(a).cuda() for a in (x, q))
    ws = P.make_workspace(n, m, d)
    print(f"prepared samples with far ones d={d}", flush=True)
    want = {f: P.sdkde_eval(xd, qd, h, want="log", flags=f)[1] for f in (0, P.SDKDE_FLAG_MAX_SHIFT)}
    ref = oracle.eval_log_density(x, q, h)
    allowed = gram_exponent_error(x, q, h, low_precision_inputs=True) + 4.0 * 2.0**-23 * np.abs(ref) + 2.0**-18
    assert np.all(np.abs(want[P.SDKDE_FLAG_MAX_SHIFT].cpu().numpy() - ref)[::4] <= allowed[::4])
    for first in want:
        P.sdkde_eval(xd, qd, h, want="log", flags=first, workspace=ws)
        for f in want:
            got = P.sdkde_eval(xd, qd, h, want="log", flags=f | P.SDKDE_FLAG_SAMPLES_PREPARED, workspace=ws)[1]
            assert torch.equal(got, want[f])


def test_points_in_batches_over_narrow_columns(tuning):
    """Batches after the first find the columns' units where the first one's samples left them: the same bits as in one pass."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    n, m, d = 700, 40000, 16
    tuning(P.SDKDE_TUNE_SCORE_SPLITS, 1)
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=3)
    narrow = np.float32(10.0) ** -(np.arange(d) % 6).astype(np.float32)
    xd, qd = (torch.from_numpy(a * narrow).cuda() for a in (x, q))
    plan = P.sdkde_describe_plan(n, m, d, 1)
    assert plan["splits"] == 1
    tight = torch.empty(plan["workspace_bytes"] - 2 * plan["dp"] * (2 * plan["n_pad"] + plan["m_pad"]), dtype=torch.uint8, device="cuda")
    print("batches over narrow columns", flush=True)
    for flags in (0, P.SDKDE_FLAG_MAX_SHIFT):
        want = P.sdkde_score(xd, float(h), points=qd, flags=flags)
        assert torch.equal(P.sdkde_score(xd, float(h), points=qd, flags=flags, workspace=tight), want)
