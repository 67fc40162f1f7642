"""Scores of the thin path on few samples, which one launch takes: against the oracle and the split slots (a forced number of splits
selects them) at the edges of threads' shares and row blocks, over inputs as outputs, and what the call leaves of prepared samples."""
import numpy as np
import pytest

import oracle
import sdkde_inputs
from parity import assert_score_close, assert_shifted_close, score_resolution

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("n,m", [(1, 1), (15, 17), (16, 16), (127, 33), (129, 8192), (1000, 50), (4096, 100)])
def test_thin_whole_matches_the_oracle_and_the_split_slots(tuning, n, m, d):
    import torch
    import paper_2602_10378_amd as P
    P.load()
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=n + d)
    h = float(h) if n > 1 else 8.0
    x, q = x + np.float32(40.0), q + np.float32(40.0)
    xd, qd = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda()
    print(f"thin whole n={n} m={m} d={d}", flush=True)

    def calls():
        s = torch.empty_like(xd)
        x_sd, _, logd = P.sdkde_fit_eval(xd, qd, h, score_out=s, want="log")
        assert torch.equal(P.sdkde_score(xd, h), s) and torch.equal(P.sdkde_debias(xd, s, h), x_sd)
        return s, x_sd, logd, P.sdkde_score(xd, h, points=qd)

    whole = [t.cpu().numpy().astype(np.float64) for t in calls()]
    tuning(P.SDKDE_TUNE_SCORE_SPLITS, 1)
    split = [t.cpu().numpy().astype(np.float64) for t in calls()]
    at = slice(0, m, max(1, m // 200))
    ref = oracle.score(x, h)
    assert_score_close(whole[0], ref, "samples", score_resolution(x, x, h))
    trusted = np.any(whole[3][at] != 0.0, axis=1) | (n == 1)        # (0 where the weights are below the fp32 range)
    assert_score_close(whole[3][at][trusted], oracle.score(x, h, points=q[at][trusted]), "points", score_resolution(x, q[at][trusted], h))
    if n > 1:
        assert_shifted_close(whole[1], x + 0.5 * h * h * ref, ref, h)
    # coordinates rounded to 2^-24 of their distance from the centre on one side, differences on the other, and sums of two orders
    for k, p in ((0, x), (3, q)):
        assert np.all(np.linalg.norm(whole[k] - split[k], axis=1) <= 2.0 * score_resolution(x, p, h))
    finite = np.isfinite(split[2])
    assert np.array_equal(finite, np.isfinite(whole[2])) and np.allclose(whole[2][finite], split[2][finite], rtol=0, atol=2e-4)


@pytest.mark.parametrize("d", [1, 3, 6])
def test_thin_whole_over_its_inputs_and_prepared_samples(tuning, d):
    """Outputs over the samples take the other way, since workgroups still read them; a score call ends what an eval call prepared."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    n, m = 3000, 70
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=d)
    xd, qd, h = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), float(h)
    print(f"thin whole over its inputs d={d}", flush=True)
    tuning(P.SDKDE_TUNE_SCORE_SPLITS, 0)
    want = P.sdkde_fit_eval(xd, qd, h, want="log")
    inplace = xd.clone()
    got = P.sdkde_fit_eval(inplace, qd, h, samples_sd_out=inplace, want="log")
    assert torch.allclose(got[0], want[0], rtol=1e-5, atol=1e-5) and torch.allclose(got[2], want[2], atol=2e-4)
    over = xd.clone()
    s = P.sdkde_score(over, h, out=over)
    assert torch.allclose(s, P.sdkde_score(xd, h), rtol=1e-4, atol=1e-5)
    ws = P.make_workspace(n, m, d)
    first = P.sdkde_eval(xd, qd, h, want="log", workspace=ws)[1]
    prepared = P.SDKDE_FLAG_SAMPLES_PREPARED
    assert torch.equal(P.sdkde_eval(xd, qd, h, want="log", workspace=ws, flags=prepared)[1], first)
    P.sdkde_score(xd, h, workspace=ws)
    assert bool(torch.isnan(P.sdkde_eval(xd, qd, h, want="log", workspace=ws, flags=prepared)[1]).all())
    x_sd, _, logd = P.sdkde_fit_eval(xd, qd, h, want="log", workspace=ws)
    assert torch.equal(P.sdkde_eval(x_sd, qd, h, want="log", workspace=ws, flags=prepared)[1], logd)


@pytest.mark.parametrize("d", [1, 2, 3, 6])
@pytest.mark.parametrize("n,m", [(17, 5), (600, 50), (4096, 100)])
def test_an_infinite_sample_weighs_nothing_on_the_thin_path(n, m, d):
    """Score at the other samples and at points: that of the set without the sample (all its weights are zero)."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=n + d)
    h = 2.0 * float(h)
    rest = np.arange(n) != n // 2
    for value, k in ((np.inf, d - 1), (-np.inf, 0)):
        x[n // 2, k] = value
        xd, qd, restd = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), torch.from_numpy(x[rest]).cuda()
        print(f"thin whole, infinite sample n={n} m={m} d={d} {value}", flush=True)
        s, x_sd = torch.empty_like(xd), torch.empty_like(xd)
        P.sdkde_fit_eval(xd, qd, h, score_out=s, samples_sd_out=x_sd, want="log")
        keep = torch.from_numpy(rest).cuda()
        for got, want, at in ((s[keep], P.sdkde_score(restd, h), x[rest]), (P.sdkde_score(xd, h, points=qd), P.sdkde_score(restd, h, points=qd), q)):
            err = (got - want).norm(dim=1).cpu().numpy()        # (the terms come in another order)
            assert np.all(err <= 2.0 * score_resolution(x[rest], at, h))
        assert bool(torch.isfinite(x_sd[keep]).all())
