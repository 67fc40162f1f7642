"""Max-shifted sums of the fp32 mode's matrix path, which find a row's shift while they go over the samples: shifts that have to be
raised, on both levels of the sums and between splits, first chunks that say nothing, and neighbours in a wave that differ."""
import numpy as np
import pytest

import oracle
from parity import assert_laplace_close, gram_exponent_error
from test_gpu_split_kernel import _score_bound

pytestmark = pytest.mark.gpu


def _gpu(*arrays):
    import torch
    return [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda() for a in arrays]


def _check(P, x, q, h, keep=slice(None), rows=slice(None)):
    """All three shifted calls at q, the results for q[rows] against the oracle on the samples x[keep], to what fp32 exponents resolve."""
    flags = P.SDKDE_FLAG_MAX_SHIFT
    xd, qd = _gpu(x, q)
    y, q = x[keep], q[rows]
    ref, e = oracle.eval_log_density(y, q, h) + np.log(len(y) / len(x)), gram_exponent_error(y, q, h)
    logd = P.sdkde_eval(xd, qd, h, want="log", flags=flags)[1].cpu().numpy()[rows]
    assert np.all(np.abs(logd - ref) <= e + 2.0**-18 + 2.0**-23 * np.abs(ref)), np.max(np.abs(logd - ref) - e)
    if x.shape[1] >= 7:
        err = np.linalg.norm(P.sdkde_score(xd, h, points=qd, flags=flags).cpu().numpy()[rows] - oracle.score(y, h, points=q), axis=1)
        assert np.all(err <= _score_bound(y, q, h)), (err / _score_bound(y, q, h)).max()
    if np.isinf(x).any():               # (an infinite sample makes every Laplace estimate NaN)
        return
    lap = P.sdkde_eval_laplace(xd, qd, h, flags=flags).cpu().numpy()[rows]
    scale = len(y) / len(x)
    assert_laplace_close(lap, scale * oracle.eval_laplace_density(y, q, h), scale * oracle.eval_laplace_abs_density(y, q, h), "laplace", e, np.exp(ref))


@pytest.mark.parametrize("d", [4, 8, 16, 24, 48, 64, 85, 128])
@pytest.mark.parametrize("splits", [1, 8])
def test_shifts_that_grow_along_the_samples(tuning, d, splits):
    """Samples in the order of their distance, farthest first: exponents grow by 800 from the first chunk to the last, so that shifts
    are raised after sums have been folded into the second level; then nearest first."""
    import paper_2602_10378_amd as P
    P.load()
    n, h = 1200, 1.0
    rng = np.random.default_rng(d)
    step = rng.standard_normal((n, d)) / np.sqrt(d)
    x = (step * np.linspace(0.05, 33.0, n)[:, None]).astype(np.float32)
    q = np.concatenate([0.3 * rng.standard_normal((35, d)) / np.sqrt(d), 0.98 * x[::50] + 0.01]).astype(np.float32)
    tuning(P.SDKDE_TUNE_SCORE_SPLITS, splits)
    tuning(P.SDKDE_TUNE_EVAL_SPLITS, splits)
    for name, order in (("farthest first", np.arange(n)[::-1]), ("nearest first", np.arange(n))):
        print(f"growing shifts d={d} splits {splits} {name}", flush=True)
        _check(P, x[order], q, h)


@pytest.mark.parametrize("d", [9, 16, 24, 64, 128])
@pytest.mark.parametrize("what", ["infinite", "beyond the range", "distant"])
def test_first_chunks_without_a_sample_that_counts(tuning, d, what):
    """A split's first chunk holds only samples without a weight: with infinite coordinates, beyond the fp16 range, or far enough for the
    exponents of far rows.  The ones that count come after it."""
    import paper_2602_10378_amd as P
    P.load()
    n, h = 400, 1.0
    rng = np.random.default_rng(d)
    x = rng.standard_normal((n, d)).astype(np.float32)
    # the centre is the mean of up to 4096 / d (at least 32) evenly strided rows, over which offsets have to cancel
    rows = min(max(4096 // d, 32), n)
    used = np.intersect1d(np.arange(32), np.arange(0, rows * (n // rows), n // rows))
    if what == "infinite" and n // rows == 1:
        pytest.skip("every sample is among the rows of the centre")
    offset = {"infinite": 1e4, "beyond the range": 1e6, "distant": 1e4}[what]
    x[:32, 1] = np.inf if what == "infinite" else offset
    signs = (-1.0) ** np.arange(len(used))
    if len(used) % 2:
        signs[:3] = (1.0, 1.0, -2.0)
    x[used, 1] = offset * signs
    keep = np.abs(x).max(axis=1) < 1e3
    q = rng.standard_normal((40, d)).astype(np.float32)
    tuning(P.SDKDE_TUNE_SCORE_SPLITS, 1)
    tuning(P.SDKDE_TUNE_EVAL_SPLITS, 1)
    print(f"first chunk without weight d={d} {what}", flush=True)
    _check(P, x, q, h, keep)


@pytest.mark.parametrize("d", [8, 16, 64])
def test_a_query_without_a_value_leaves_its_neighbours_alone(d):
    import paper_2602_10378_amd as P
    P.load()
    rng = np.random.default_rng(d)
    x, q = rng.standard_normal((900, d)).astype(np.float32), (3.0 * rng.standard_normal((130, d))).astype(np.float32)
    bad = q.copy()
    bad[[5, 77], 2] = np.nan
    good = np.ones(130, bool)
    good[[5, 77]] = False
    print(f"queries without a value d={d}", flush=True)
    _check(P, x, bad, 1.0, rows=good)
    flags = P.SDKDE_FLAG_MAX_SHIFT
    assert bool(P.sdkde_eval(*_gpu(x, bad), 1.0, want="log", flags=flags)[1][[5, 77]].isnan().all())


@pytest.mark.parametrize("d", [8, 16, 24, 32, 64, 128])
def test_queries_beside_padding_rows_are_as_they_are_beside_others(tuning, d):
    """One distant sample, and queries near the others, whose weights do not differ enough for a shift to be raised (which all rows of
    a wave would be): those that share a wave with padding rows have the bits they have beside other queries."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    rng = np.random.default_rng(d)
    x, q = rng.standard_normal((1000, d)).astype(np.float32), rng.standard_normal((256, d)).astype(np.float32)
    h = float(np.sqrt(d))
    x[601, 0] = 5000.0 * h
    (xd, qd), flags = _gpu(x, q), P.SDKDE_FLAG_MAX_SHIFT
    for knob in (P.SDKDE_TUNE_SCORE_ROW_TILES, P.SDKDE_TUNE_EVAL_ROW_TILES):
        tuning(knob, 2)
    for knob in (P.SDKDE_TUNE_SCORE_SPLITS, P.SDKDE_TUNE_EVAL_SPLITS):
        tuning(knob, 1)
    print(f"beside padding rows d={d}", flush=True)
    calls = (lambda p: P.sdkde_eval(xd, p, h, want="log", flags=flags)[1], lambda p: P.sdkde_eval_laplace(xd, p, h, flags=flags),
             lambda p: P.sdkde_score(xd, h, points=p, flags=flags))
    for call in calls:
        assert torch.equal(call(qd[:200].contiguous()), call(qd)[:200])
