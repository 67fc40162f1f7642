"""The fp32 mode's pair kernel (two fp16 parts per operand) in every workgroup shape it is built in, at its edges: one
and several 16-column blocks, even and odd block counts, a nearly empty and a full last block, a ragged last chunk of
samples, fewer chunks than splits, own chunks split over workgroups, splits long enough to fold their running sums, and
weights at the bottom of the range.  Held to what fp32 arithmetic costs, not only to the general tolerance."""
import numpy as np
import pytest

import oracle
import sdkde_inputs
from parity import assert_laplace_close, gram_exponent_error, score_resolution

pytestmark = pytest.mark.gpu


def _score_bound(x, p, h):
    """Per point: an error e in every exponent moves a weight by e of itself, so the numerator by at most
    e sum_j phi_j |x_j - p| and, through the denominator, the score by e |s| <= the same over h^2 D; on top of it what the
    two cancelling sums resolve (score_resolution)."""
    x, p = x.astype(np.float64), p.astype(np.float64)
    c = x.mean(axis=0)
    x, p = x - c, p - c
    r2 = np.maximum((p * p).sum(1)[:, None] + (x * x).sum(1)[None] - 2.0 * p @ x.T, 0.0)
    u = r2 / (2.0 * h * h)
    w = np.exp(-(u - u.min(axis=1, keepdims=True)))
    pull = (w * np.sqrt(r2)).sum(1) / w.sum(1) / (h * h)
    return 2.0 * gram_exponent_error(x, p, h) * pull + score_resolution(x, p, h)


@pytest.mark.parametrize("d", [7, 16, 17, 32, 37, 64, 80, 96, 97, 128])
@pytest.mark.parametrize("row_tiles", [2, 4, 8])
@pytest.mark.parametrize("n", [40, 1111, 4500])
def test_every_workgroup_shape(tuning, n, d, row_tiles):
    import torch
    import paper_2602_10378_amd as P
    P.load()
    m = 70
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=4, seed=n + d)
    h = float(h)
    tuning(P.SDKDE_TUNE_SCORE_ROW_TILES, row_tiles)
    tuning(P.SDKDE_TUNE_EVAL_ROW_TILES, row_tiles)
    ran = 0
    xd, qd = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda()
    print(f"split kernel n={n} m={m} d={d} row tiles {row_tiles}", flush=True)
    if P.sdkde_describe_plan(n, n, d, 0)["row_tiles"] == row_tiles:
        ran += 1
        s = P.sdkde_score(xd, h).cpu().numpy()
        err = np.linalg.norm(s - oracle.score(x, h), axis=1)
        assert np.all(err <= _score_bound(x, x, h)), (err / _score_bound(x, x, h)).max()
        s = P.sdkde_score(xd, h, points=qd).cpu().numpy()
        err = np.linalg.norm(s - oracle.score(x, h, points=q), axis=1)
        assert np.all(err <= _score_bound(x, q, h)), (err / _score_bound(x, q, h)).max()
    if P.sdkde_describe_plan(n, m, d, 2)["row_tiles"] == row_tiles:
        ran += 1
        ref = oracle.eval_log_density(x, q, h)
        e = gram_exponent_error(x, q, h)
        for flags in (0, P.SDKDE_FLAG_MAX_SHIFT):
            logd = P.sdkde_eval(xd, qd, h, want="log", flags=flags)[1].cpu().numpy()
            # + the sum's own rounding (chains of 64 tiles and the splits) and the output's
            assert np.all(np.abs(logd - ref) <= e + 2.0**-18 + 2.0**-23 * np.abs(ref))
        lap = P.sdkde_eval_laplace(xd, qd, h).cpu().numpy()
        assert_laplace_close(lap, oracle.eval_laplace_density(x, q, h), oracle.eval_laplace_abs_density(x, q, h), "laplace", e,
                             np.exp(ref))
    if ran == 0:
        pytest.skip("not built")


@pytest.mark.parametrize("d", [4, 5])
@pytest.mark.parametrize("row_tiles", [2, 4, 8])
@pytest.mark.parametrize("n", [40, 1111, 4500])
def test_row_maxima_of_four_columns(tuning, n, d, row_tiles):
    """The shifted sums' first pass holds all part products of up to four columns in one matrix instruction (d = 5: the
    general form), in every workgroup shape, for queries among the samples and up to 300 bandwidths away."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    m = 70
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=4, seed=n + d)
    h = float(h)
    q[m // 2:] *= np.geomspace(1.0, 100.0, m - m // 2, dtype=np.float32)[:, None]
    tuning(P.SDKDE_TUNE_EVAL_ROW_TILES, row_tiles)
    assert P.sdkde_describe_plan(n, m, d, 2)["row_tiles"] == row_tiles
    print(f"row maxima n={n} m={m} d={d} row tiles {row_tiles}", flush=True)
    xd, qd = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda()
    ref = oracle.eval_log_density(x, q, h)
    e = gram_exponent_error(x, q, h)
    logd = P.sdkde_eval(xd, qd, h, want="log", flags=P.SDKDE_FLAG_MAX_SHIFT)[1].cpu().numpy()
    assert np.all(np.abs(logd - ref) <= e + 2.0**-18 + 2.0**-23 * np.abs(ref)), np.abs(logd - ref).max()
    lap = P.sdkde_eval_laplace(xd, qd, h, flags=P.SDKDE_FLAG_MAX_SHIFT).cpu().numpy()
    assert_laplace_close(lap, oracle.eval_laplace_density(x, q, h), oracle.eval_laplace_abs_density(x, q, h), "laplace", e,
                         np.exp(ref))


@pytest.mark.parametrize("d,row_tiles", [(16, 8), (32, 4), (64, 4), (64, 2), (80, 4), (80, 2), (90, 4), (96, 4), (96, 2), (112, 2),
                                         (128, 2)])
@pytest.mark.parametrize("splits", [1, 2])
def test_splits_that_fold_their_running_sums(tuning, d, row_tiles, splits):
    """A split of more than 64 sample tiles folds its running sums, at dp <= 64 into LDS, above into its own rows of the
    partial slot (stored first, then read and added to, and read once more at the end): several folds and a ragged
    remainder, at the samples and at separate points, one and two slots."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    n, m = 4517, 130
    x, q, _ = sdkde_inputs.gaussian_mixture(n, m, d, components=4, seed=d)
    h = 0.5 * d**0.5        # every sample of a component weighs about exp(-4): no fold is small beside the others
    tuning(P.SDKDE_TUNE_SCORE_ROW_TILES, row_tiles)
    tuning(P.SDKDE_TUNE_SCORE_SPLITS, splits)
    print(f"folds n={n} m={m} d={d} row tiles {row_tiles} splits {splits}", flush=True)
    for call in (0, 1):
        p = P.sdkde_describe_plan(n, m, d, call)
        assert p["row_tiles"] == row_tiles and p["splits"] == splits and p["tiles_per_split"] >= 128
        assert p["tiles_per_split"] % 64 != 0
    xd, qd = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda()
    s = P.sdkde_score(xd, h).cpu().numpy()
    err = np.linalg.norm(s - oracle.score(x, h), axis=1)
    assert np.all(err <= _score_bound(x, x, h)), (err / _score_bound(x, x, h)).max()
    s = P.sdkde_score(xd, h, points=qd, flags=P.SDKDE_FLAG_MAX_SHIFT).cpu().numpy()
    err = np.linalg.norm(s - oracle.score(x, h, points=q), axis=1)
    assert np.all(err <= _score_bound(x, q, h)), (err / _score_bound(x, q, h)).max()


@pytest.mark.parametrize("d", [7, 16, 40])
@pytest.mark.parametrize("binades", [109, 112, 115])
def test_weights_whose_lower_parts_leave_the_bf16_range(d, binades):
    """Points about sqrt(2 binades ln 2) bandwidths from a tight cloud: weights about 2^-binades, whose second and third
    parts lie near or below 2^-126, in T but not in D.  A part cut there is less than 2^-126 of each sample's weight, so
    beside the bound that the exponents give, T / D may be off by n 2^-126 (max_j |x_j - c| + |p - c|) / D per part."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    n, m, h = 1000, 64, 1.0
    rng = np.random.default_rng(binades + d)
    x = (0.05 * rng.standard_normal((n, d))).astype(np.float32)
    q = rng.standard_normal((m, d))
    q = (q / np.linalg.norm(q, axis=1, keepdims=True) * np.sqrt(2.0 * binades * np.log(2.0)) * h).astype(np.float32)
    print(f"weights about 2^-{binades}, d={d}", flush=True)
    s = P.sdkde_score(torch.from_numpy(x).cuda(), h, points=torch.from_numpy(q).cuda()).cpu().numpy().astype(np.float64)
    x64, q64 = x.astype(np.float64), q.astype(np.float64)
    weight_sum = np.exp(-((q64[:, None, :] - x64[None]) ** 2).sum(-1) / (2.0 * h * h)).sum(1)
    live = weight_sum > 1.01 * 1000.0 * n * 2.0**-126          # below: reported as underflow
    assert live.all() and weight_sum.max() < n * 2.0 ** (-binades + 12)
    cut = 2.0 * n * 2.0**-126 * (np.linalg.norm(x64, axis=1).max() + np.linalg.norm(q64, axis=1)) / weight_sum / (h * h)
    err = np.linalg.norm(s - oracle.score(x, h, points=q), axis=1)
    assert np.all(err <= _score_bound(x, q, h) + cut), (err / (_score_bound(x, q, h) + cut)).max()


@pytest.mark.parametrize("d", [7, 16, 24, 37])
def test_a_sample_at_infinity_has_no_weight(d):
    """One infinite coordinate of one sample (not one of the rows the centre is formed of: every 17th at d = 16, every
    40th at d = 37): its weight is zero wherever it is looked at from, whatever the signs of the other coordinates, so
    every other output is that of the samples without it."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    n, m = 4500, 70
    print(f"sample at infinity n={n} m={m} d={d}", flush=True)
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=4, seed=d)
    h = float(h)
    rest = x[:-1]
    logd_ref = oracle.eval_log_density(rest, q, h) + np.log((n - 1) / n)
    e = gram_exponent_error(rest, q, h)
    for value in (np.inf, -np.inf):
        y = x.copy()
        y[-1, d // 2] = value
        yd, qd = torch.from_numpy(y).cuda(), torch.from_numpy(q).cuda()
        for flags in (0, P.SDKDE_FLAG_MAX_SHIFT):
            logd = P.sdkde_eval(yd, qd, h, want="log", flags=flags)[1].cpu().numpy()
            assert np.all(np.abs(logd - logd_ref) <= e + 2.0**-18 + 2.0**-23 * np.abs(logd_ref))
            s = P.sdkde_score(yd, h, points=qd, flags=flags).cpu().numpy()
            err = np.linalg.norm(s - oracle.score(rest, h, points=q), axis=1)
            assert np.all(err <= _score_bound(rest, q, h))
        s = P.sdkde_score(yd, h).cpu().numpy()[:-1]
        err = np.linalg.norm(s - oracle.score(rest, h), axis=1)
        assert np.all(err <= _score_bound(rest, rest, h))
