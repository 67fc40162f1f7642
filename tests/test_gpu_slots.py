"""Sums over split slots: every number of slots that leaves a thread groups of four, a pair or a single one, with 4 and with 32 threads an
output, plain and with a shift a slot."""
import numpy as np
import pytest

import oracle
import sdkde_inputs
from parity import assert_laplace_close, assert_log_density_close, assert_score_close, score_resolution

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("splits", [1, 2, 3, 4, 5, 8, 9, 12, 13, 16, 17, 20, 31, 33, 63, 64, 65, 96, 97, 130])
@pytest.mark.parametrize("d", [3, 9, 16])
def test_any_number_of_slots(tuning, d, splits):
    import torch
    import paper_2602_10378_amd as P
    P.load()
    n, m = 4200, 70
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=d)
    xd, qd, h = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), float(h)
    tuning(P.SDKDE_TUNE_SCORE_SPLITS, splits)
    tuning(P.SDKDE_TUNE_EVAL_SPLITS, splits)
    print(f"slots d={d} splits={splits}", flush=True)
    s = torch.empty_like(xd)
    x_sd, _, logd = P.sdkde_fit_eval(xd, qd, h, score_out=s, want="log")
    assert torch.equal(P.sdkde_score(xd, h), s) and torch.equal(P.sdkde_debias(xd, s, h), x_sd)
    at = np.arange(0, n, 29)
    assert_score_close(s.cpu().numpy()[at], oracle.score(x, h)[at], f"slots {splits}", score_resolution(x, x[at], h))
    assert_log_density_close(logd.cpu().numpy(), oracle.eval_log_density(x_sd.cpu().numpy(), q, h), f"slots {splits}")
    for flags in (0, P.SDKDE_FLAG_MAX_SHIFT):
        sp = P.sdkde_score(xd, h, points=qd, flags=flags).cpu().numpy()
        assert_score_close(sp, oracle.score(x, h, points=q), f"slots {splits} points {flags}", score_resolution(x, q, h))
        _, logd = P.sdkde_eval(xd, qd, h, want="log", flags=flags)
        assert_log_density_close(logd.cpu().numpy(), oracle.eval_log_density(x, q, h), f"slots {splits} log {flags}")
        lap = P.sdkde_eval_laplace(xd, qd, h, flags=flags).cpu().numpy()
        assert_laplace_close(lap, oracle.eval_laplace_density(x, q, h), oracle.eval_laplace_abs_density(x, q, h), f"slots {splits} laplace {flags}")
