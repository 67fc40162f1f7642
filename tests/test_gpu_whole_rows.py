"""Small sample sets in the fp32 mode: a workgroup sums its rows over all samples (pair_whole_kernel).  Against the oracle and against
the kernels with split slots, which a forced number of splits selects, at the edges of tiles, chunks, waves and row counts."""
import numpy as np
import pytest

import oracle
import sdkde_inputs
from parity import assert_shifted_close, gram_exponent_error, score_resolution
from test_gpu_split_kernel import _score_bound

pytestmark = pytest.mark.gpu


def _gpu(*arrays):
    import torch
    return [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda() for a in arrays]


def _all_calls(P, xd, qd, h, workspace=None):
    import torch
    s = torch.full_like(xd, float("nan"))
    x_sd, _, logd = P.sdkde_fit_eval(xd, qd, h, score_out=s, want="log", workspace=workspace)
    alone = P.sdkde_score(xd, h, workspace=workspace)
    assert torch.equal(alone, s) or not bool(torch.isfinite(s).all())
    return {"score": s, "x_sd": x_sd, "log of shifted": logd, "at points": P.sdkde_score(xd, h, points=qd, workspace=workspace),
            "log": P.sdkde_eval(xd, qd, h, want="log", workspace=workspace)[1],
            "laplace": P.sdkde_eval_laplace(xd, qd, h, workspace=workspace)}


def _both(P, tuning, xd, qd, h):
    """The calls on whole rows, and with split slots."""
    whole = _all_calls(P, xd, qd, h)
    tuning(P.SDKDE_TUNE_SCORE_SPLITS, 1)
    tuning(P.SDKDE_TUNE_EVAL_SPLITS, 1)
    split = _all_calls(P, xd, qd, h)
    tuning(P.SDKDE_TUNE_SCORE_SPLITS, 0)
    tuning(P.SDKDE_TUNE_EVAL_SPLITS, 0)
    return whole, split


@pytest.mark.parametrize("d", [4, 7, 8, 9, 16, 17, 24, 25, 32, 37, 48, 56, 64, 72, 80, 90, 112, 119, 128])
@pytest.mark.parametrize("n,m", [(1, 1), (31, 16), (33, 17), (513, 250), (767, 4097)])
def test_whole_rows_match_the_oracle_and_the_split_slots(tuning, n, m, d):
    import torch
    import paper_2602_10378_amd as P
    P.load()
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=4, seed=n + d)
    # (one sample has no rule-of-thumb bandwidth: the mixture's size, so that no weight is below the fp32 range)
    h = float(h) if n > 1 else 3.0 * d**0.5
    q = q[:m]
    print(f"whole rows n={n} m={m} d={d}", flush=True)
    whole, split = _both(P, tuning, *_gpu(x, q), h)
    ref_s = oracle.score(x, h)
    # the same exponents up to the rounding of a row's scale, other orders of the same sums: each within its own resolution
    for key, at in (("score", x), ("at points", q)):
        err = np.linalg.norm((whole[key] - split[key]).cpu().numpy().astype(np.float64), axis=1)
        assert np.all(err <= 2.0 * score_resolution(x, at, h)), key
    at = slice(0, m, max(1, m // 300))
    if d >= 7:
        err = np.linalg.norm(whole["score"].cpu().numpy() - ref_s, axis=1)
        assert np.all(err <= _score_bound(x, x, h)), (err / _score_bound(x, x, h)).max()
        err = np.linalg.norm(whole["at points"].cpu().numpy()[at] - oracle.score(x, h, points=q[at]), axis=1)
        assert np.all(err <= _score_bound(x, q[at], h))
    assert_shifted_close(whole["x_sd"].cpu().numpy(), x + 0.5 * h * h * ref_s, ref_s, h) if n > 1 else None
    ref, e = oracle.eval_log_density(x, q[at], h), gram_exponent_error(x, q[at], h)
    assert np.all(np.abs(whole["log"].cpu().numpy()[at] - ref) <= e + 2.0**-18 + 2.0**-23 * np.abs(ref))
    for key in ("log", "log of shifted"):           # at most 2 x 80 roundings of a positive sum, and the logarithm's own
        a, b = (v[key].cpu().numpy().astype(np.float64) for v in (whole, split))
        # (x_sd of the two paths differs by their scores' resolution, which moves an exponent by that times the distance)
        more = 0.0 if key == "log" else 2.0 * 0.5 * h * np.max(score_resolution(x, x, h)) * h * 14.0
        assert np.all(np.abs(a - b) <= 160 * 2.0**-24 + 2.0**-23 * np.abs(b) + more), key
    lap, other = whole["laplace"].double(), split["laplace"].double()
    dens = torch.exp(split["log"].double())
    # terms of size up to phi (1 + d/2 + 88), each sum rounded 80 times
    assert bool((abs(lap - other) <= 160 * 2.0**-24 * (90.0 + d) * dens + 1e-37).all())


@pytest.mark.parametrize("d", [9, 16, 24, 40, 128])
@pytest.mark.parametrize("what", ["far", "infinite", "nan", "narrow", "duplicates"])
def test_whole_rows_on_unusual_samples(tuning, d, what):
    """Samples beyond the fp16 range, without a finite norm, NaN in one; columns in units of their own, with chunks that need other
    ones; exact duplicates: as the split slots have them, the same outputs finite."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    n, m = 700, 65
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=d)
    h = float(h)
    if what == "far":
        x[[601, 650, 683]] += np.float32(1e6 * h)       # none of the rows that the centre is the mean of
    elif what == "infinite":
        x[5, d - 1] = np.inf
    elif what == "nan":
        x[690, 0] = np.nan
    elif what == "narrow":
        narrow = np.float32(10.0) ** -(np.arange(d) % 6).astype(np.float32)
        x, q = x * narrow, q * narrow
        x[100:104, d - 1] = 3.0 * h
    else:
        x[350:] = x[:350]
    print(f"whole rows, unusual samples d={d} {what}", flush=True)
    whole, split = _both(P, tuning, *_gpu(x, q), h)
    usual = np.isfinite(x).all(axis=1)
    for key in whole:
        a, b = whole[key], split[key]
        assert torch.equal(torch.isfinite(a), torch.isfinite(b)), key
        assert torch.equal(torch.isnan(a), torch.isnan(b)), key
    near = usual if what != "far" else np.abs(x).max(axis=1) < 1e5 * h
    for key, at, rows in (("score", x, near), ("at points", q, np.ones(m, bool))):
        a, b = (v[key].cpu().numpy().astype(np.float64)[rows] for v in (whole, split))
        fine = np.isfinite(a).all(axis=1)
        bound = 2.0**-19 * (1.0 + np.linalg.norm(at[rows] - x[near].mean(axis=0), axis=1) / h) / h
        assert np.all(np.linalg.norm(a - b, axis=1)[fine] <= bound[fine]), key


@pytest.mark.parametrize("n,m,d", [(600, 50, 8), (1000, 333, 16), (2000, 100, 37), (700, 3000, 64)])
def test_whole_rows_leave_prepared_samples_and_fit_smaller_buffers(n, m, d):
    """The one-call pass leaves the shifted samples prepared for later calls; misaligned outputs and a samples array that is also the
    output of the shift are served; with a buffer too small for both passes' operands together the passes run one by one: the same
    scores, shifted samples prepared with the centre of the samples in either case, so the same densities."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=n)
    xd, qd = _gpu(x, q)
    h = float(h)
    print(f"whole rows, buffers n={n} m={m} d={d}", flush=True)
    ws = P.make_workspace(n, m, d)
    s = torch.empty_like(xd)
    x_sd, _, logd = P.sdkde_fit_eval(xd, qd, h, score_out=s, want="log", workspace=ws)
    for flags in (0, P.SDKDE_FLAG_MAX_SHIFT):
        again = P.sdkde_eval(x_sd, qd, h, want="log", workspace=ws, flags=flags | P.SDKDE_FLAG_SAMPLES_PREPARED)[1]
        assert torch.equal(again, logd) if flags == 0 else torch.allclose(again, logd, atol=1e-4)
    assert bool(torch.isnan(P.sdkde_eval(xd, qd, h, want="log", workspace=ws, flags=P.SDKDE_FLAG_SAMPLES_PREPARED)[1]).all())
    flat = torch.full((2 * n * d + 2,), float("nan"), device="cuda")
    odd_s, odd_x = flat[1:1 + n * d].view(n, d), flat[1 + n * d:1 + 2 * n * d].view(n, d)
    P.sdkde_fit_eval(xd, qd, h, score_out=odd_s, samples_sd_out=odd_x, want="log", workspace=ws)
    assert torch.equal(odd_s, s) and torch.equal(odd_x, x_sd) and bool(torch.isnan(flat[[0, -1]]).all())
    inplace = xd.clone()
    P.sdkde_fit_eval(inplace, qd, h, samples_sd_out=inplace, want="log", workspace=ws)
    assert torch.equal(inplace, x_sd)
    need = P.sdkde_workspace_bytes(n, m, d)
    tight = torch.empty(need, dtype=torch.uint8, device="cuda")
    s2 = torch.empty_like(xd)
    x_sd2, _, logd2 = P.sdkde_fit_eval(xd, qd, h, score_out=s2, want="log", workspace=tight)
    assert torch.equal(s2, s) and torch.equal(x_sd2, x_sd) and torch.equal(logd2, logd)
    static = [torch.empty_like(t) for t in (xd, xd, logd)]
    P.sdkde_fit_eval_static(xd, qd, h, static[0], score_out=static[1], log_density_out=static[2])
    assert torch.equal(static[0], x_sd) and torch.equal(static[1], s) and torch.equal(static[2], logd)


@pytest.mark.parametrize("n,d", [(600, 8), (700, 64), (1000, 24), (5000, 16), (4000, 24)])
@pytest.mark.parametrize("which", ["shifted", "in place", "score"])
def test_queries_that_the_same_call_writes_are_read_after_it_has(n, d, which):
    """Queries in the array that the shifted samples or the scores go to: as in the three separate calls, the density is that at what
    has been written there, also where the pass would prepare the queries before (small sets) or while (d <= 16) the score is formed."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    x, _, h = sdkde_inputs.gaussian_mixture(n, 1, d, components=3, seed=n)
    (xd,), h = _gpu(x), float(h)
    print(f"queries the call writes n={n} d={d} {which}", flush=True)
    s, x_sd = torch.empty_like(xd), torch.empty_like(xd)
    P.sdkde_fit_eval(xd, xd, h, score_out=s, samples_sd_out=x_sd, want="log")
    want = P.sdkde_fit_eval(xd, (s if which == "score" else x_sd).clone(), h, want="log")[2]
    out = xd.clone() if which == "in place" else torch.zeros_like(xd)
    score = torch.zeros_like(xd)
    got = P.sdkde_fit_eval(out if which == "in place" else xd, score if which == "score" else out, h, score_out=score, samples_sd_out=out, want="log")[2]
    assert torch.equal(score, s) and torch.equal(out, x_sd)
    assert torch.equal(got, want)


@pytest.mark.parametrize("n,m,d,whole", [(1536, 1023, 24, True), (1537, 1023, 24, False), (2560, 1024, 32, True), (2561, 1024, 32, False), (3072, 2047, 24, False),
                                         (3072, 2048, 24, True), (768, 64, 64, True), (769, 64, 64, False), (1024, 100, 80, True), (1025, 100, 80, False),
                                         (1025, 1024, 80, True)])
def test_scores_at_few_points_keep_the_split_slots(tuning, n, m, d, whole):
    """Both sides of the lines between whole rows and split slots for scores at separate points: close to what the split slots give, which
    are what runs beyond the line, bit for bit."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=n + d)
    xd, qd = _gpu(x, q)
    print(f"whole rows or split slots n={n} m={m} d={d}", flush=True)
    got = P.sdkde_score(xd, float(h), points=qd)
    tuning(P.SDKDE_TUNE_SCORE_SPLITS, P.sdkde_describe_plan(n, m, d, 1)["splits"])
    split = P.sdkde_score(xd, float(h), points=qd)
    assert torch.equal(got, split) != whole
    err = (got - split).norm(dim=1).cpu().numpy()
    assert np.all(err <= 2.0 * score_resolution(x, q, h))
