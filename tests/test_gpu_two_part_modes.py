"""The fp16x2 mode and the calls that run as it are served by the fp32 mode's kernels where the buffer holds their operands, whatever the
number of points, and by their own where it does not."""
import numpy as np
import pytest

import sdkde_inputs

pytestmark = pytest.mark.gpu


def _calls(P, xd, qd, h, flags, ws):
    import torch
    s = torch.empty_like(xd)
    x_sd, _, logd = P.sdkde_fit_eval(xd, qd, h, score_out=s, want="log", workspace=ws, flags=flags)
    return [s, x_sd, logd, P.sdkde_score(xd, h, workspace=ws, flags=flags), P.sdkde_score(xd, h, points=qd, workspace=ws, flags=flags),
            P.sdkde_eval(xd, qd, h, want="log", workspace=ws, flags=flags)[1], P.sdkde_eval_laplace(xd, qd, h, workspace=ws, flags=flags)]


@pytest.mark.parametrize("n,m,d,flags", [(5000, 700, 16, 1), (3072, 100, 16, 2), (1500, 4100, 9, 3), (4000, 900, 33, 2), (3500, 65, 128, 3),
                                         (5000, 700, 24, 17), (600, 50, 7, 18), (200, 30, 16, 33), (9000, 300, 24, 1), (100, 900, 128, 1),
                                         (600, 20, 48, 3), (14000, 100, 16, 1), (3100, 64, 96, 2)])
def test_calls_on_the_fp32_kernels_have_their_bits(n, m, d, flags):
    import torch
    import paper_2602_10378_amd as P
    P.load()
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=d)
    xd, qd, h = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), float(h) * (1.5 if d > 64 else 1.0)
    print(f"calls on the fp32 kernels n={n} m={m} d={d} flags={flags}", flush=True)
    own = torch.empty(P.sdkde_workspace_bytes(n, m, d, flags), dtype=torch.uint8, device="cuda")
    for ws in (P.make_workspace(n, m, d), own):
        for got, want in zip(_calls(P, xd, qd, h, flags, ws), _calls(P, xd, qd, h, flags & 16, ws)):
            assert torch.equal(got, want)
    # prepared samples are those of the mode that was asked for
    ws = P.make_workspace(n, m, d)
    want = P.sdkde_eval(xd, qd, h, want="log", workspace=ws, flags=flags)[1]
    few = qd[:5].contiguous()
    prepared = P.SDKDE_FLAG_SAMPLES_PREPARED
    assert torch.equal(P.sdkde_eval(xd, qd, h, want="log", workspace=ws, flags=flags | prepared)[1], want)
    assert not bool(torch.isnan(P.sdkde_eval(xd, few, h, want="log", workspace=ws, flags=flags | prepared)[1]).any())
    assert bool(torch.isnan(P.sdkde_eval(xd, qd, h, want="log", workspace=ws, flags=(flags & 16) | prepared)[1]).all())


@pytest.mark.parametrize("n,m,d", [(4000, 200, 24), (700, 900, 16), (5000, 64, 100)])
def test_buffers_without_room_for_the_fp32_operands(tuning, n, m, d):
    """What the mode's own kernels need with one split, and no more: served by them, score and density close to the fp32 mode's."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=n)
    xd, qd, h = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), float(h) * (1.5 if d > 64 else 1.0)
    print(f"buffers without room n={n} m={m} d={d}", flush=True)
    want_s, want_e = P.sdkde_score(xd, h), P.sdkde_eval(xd, qd, h, want="log")[1]
    tuning(P.SDKDE_TUNE_SCORE_SPLITS, 1)
    tuning(P.SDKDE_TUNE_EVAL_SPLITS, 1)
    for call, run, want in ((0, lambda ws: P.sdkde_score(xd, h, workspace=ws, flags=1), want_s),
                            (2, lambda ws: P.sdkde_eval(xd, qd, h, want="log", workspace=ws, flags=1)[1], want_e)):
        plan = P.sdkde_describe_plan(n, n if call == 0 else m, d, call, 1)
        assert plan["splits"] == 1
        got = run(torch.empty(plan["workspace_bytes"], dtype=torch.uint8, device="cuda"))
        # two roundings of 2^-22 a product against two of 2^-23 a coordinate: some 1e-6 of a score, of an exponent 2^-22 of the norms
        assert float((got - want).norm() / want.norm()) < 1e-5
        with pytest.raises(P.SdkdeError):
            run(torch.empty(plan["workspace_bytes"] - 256, dtype=torch.uint8, device="cuda"))
    ws = torch.empty(P.sdkde_describe_plan(n, m, d, 2, 1)["workspace_bytes"], dtype=torch.uint8, device="cuda")
    first = P.sdkde_eval(xd, qd, h, want="log", workspace=ws, flags=1)[1]
    few = P.sdkde_eval(xd, qd[:3].contiguous(), h, want="log", workspace=ws, flags=1 | P.SDKDE_FLAG_SAMPLES_PREPARED)[1]
    assert float((few - first[:3]).abs().max()) < 1e-4


@pytest.mark.parametrize("n,m,d,flags", [(4000, 500, 16, 1), (9000, 700, 24, 1), (20000, 100, 16, 1), (6000, 800, 64, 2), (300, 40, 33, 3)])
def test_static_scratch_has_the_bits_of_a_buffer_of_the_size_that_is_asked_for(n, m, d, flags):
    import torch
    import paper_2602_10378_amd as P
    P.load()
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=d)
    xd, qd, h = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), float(h)
    print(f"static scratch in fp16 modes n={n} m={m} d={d} flags={flags}", flush=True)
    need = P.sdkde_workspace_bytes(n, m, d, flags)
    assert need <= P.SDKDE_STATIC_SCRATCH_BYTES
    s, x_sd, logd = torch.empty_like(xd), torch.empty_like(xd), torch.empty(m, device="cuda")
    P.sdkde_fit_eval_static(xd, qd, h, x_sd, score_out=s, log_density_out=logd, flags=flags)
    own_s = torch.empty_like(xd)
    own_x, _, own_logd = P.sdkde_fit_eval(xd, qd, h, score_out=own_s, want="log", workspace=torch.empty(need, dtype=torch.uint8, device="cuda"), flags=flags)
    assert torch.equal(s, own_s) and torch.equal(x_sd, own_x) and torch.equal(logd, own_logd)


@pytest.mark.parametrize("first,then,d", [(1, 2, 24), (3, 1, 64), (2, 3, 128), (2, 2, 16)])
def test_samples_prepared_in_a_mode_serve_those_that_run_as_it(first, then, d):
    """From 17 columns on all three fp16 modes are the first: samples that one has prepared are those of the others."""
    import torch
    import paper_2602_10378_amd as P
    P.load()
    n, m = 4000, 90
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=d)
    xd, qd, h = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), float(h) * (1.5 if d > 64 else 1.0)
    print(f"prepared in mode {first}, used in {then}, d={d}", flush=True)
    ws = P.make_workspace(n, m, d)
    want = P.sdkde_eval(xd, qd, h, want="log", workspace=ws, flags=first)[1]
    assert torch.equal(P.sdkde_eval(xd, qd, h, want="log", workspace=ws, flags=then | P.SDKDE_FLAG_SAMPLES_PREPARED)[1], want)


@pytest.mark.parametrize("flags", [0, 1, 17])
@pytest.mark.parametrize("n,d", [(9000, 9), (9000, 16), (9000, 33), (30000, 16)])
def test_scores_from_many_slots_are_as_exact_as_from_few(tuning, n, d, flags):
    """A call with few points has more slots, each a shorter sum, and 32 threads an output for them: the error is to be no larger than
    with the 32 slots that the fp16x2 mode's own kernels had there (0.92 to 0.94 of it; 1.60 to 1.74 with the 32 parts added one after the other)."""
    import torch
    import oracle
    import paper_2602_10378_amd as P
    P.load()
    m = 300
    error = {}
    print(f"many slots n={n} d={d} flags={flags}", flush=True)
    for seed in range(3):
        x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=4, seed=seed)
        xd, qd, h = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), float(h)
        ref = oracle.score(x, h, points=q)
        for splits in (0, 32):
            tuning(P.SDKDE_TUNE_SCORE_SPLITS, splits)
            assert splits or P.sdkde_describe_plan(n, m, d, 1, flags & 16)["splits"] >= 64
            got = P.sdkde_score(xd, h, points=qd, flags=flags).cpu().numpy()
            error[splits] = error.get(splits, 0.0) + np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print(f"many slots / 32: {error[0] / error[32]:.3f} of {error[32] / 3:.3g}", flush=True)
    assert error[0] <= 1.1 * error[32]


@pytest.mark.parametrize("shift", [0, 16])
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("d", [4, 9, 16, 24, 32, 64, 128])
def test_the_modes_own_kernels_match_the_oracle(tuning, d, splits, shift):
    """Every call of the fp16x2 mode on a buffer that holds its own operands and not the fp32 mode's; at d <= 16 also the two other modes, which
    keep their own kernels above 3072 samples."""
    import torch
    import oracle
    import paper_2602_10378_amd as P
    from parity import assert_laplace_close, assert_log_density_close, assert_score_close, score_resolution
    P.load()
    n, m = 4000, 200
    x, q, h = sdkde_inputs.gaussian_mixture(n, m, d, components=3, seed=d)
    h = np.float64(h) * (1.8 if d > 64 else 1.2)
    if shift:
        q[: m // 2] += np.float32(9.0 * h / np.sqrt(d))       # beyond what plain sums hold
    x, q, h = x * np.float32(0.4 / h), q * np.float32(0.4 / h), np.float64(0.4)         # (h^-d (2 pi)^-d/2 about one: densities in the fp32 range)
    xd, qd, h = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), float(h)
    tuning(P.SDKDE_TUNE_SCORE_SPLITS, splits)
    tuning(P.SDKDE_TUNE_EVAL_SPLITS, splits)
    at = np.arange(0, n, 17)
    ref = {"score": oracle.score(x, h)[at], "points": oracle.score(x, h, points=q), "log": oracle.eval_log_density(x, q, h),
           "laplace": oracle.eval_laplace_density(x, q, h)}
    size = oracle.eval_laplace_abs_density(x, q, h)
    for mode in (1, 2, 3) if d <= 16 else (1,):
        flags = mode | shift
        print(f"own kernels d={d} splits={splits} flags={flags}", flush=True)
        calls = {"points": (1, lambda ws, f: P.sdkde_score(xd, h, points=qd, workspace=ws, flags=f)),
                 "log": (2, lambda ws, f: P.sdkde_eval(xd, qd, h, want="log", workspace=ws, flags=f)[1]),
                 "laplace": (2, lambda ws, f: P.sdkde_eval_laplace(xd, qd, h, workspace=ws, flags=f))}
        if not shift:
            calls["score"] = (0, lambda ws, f: P.sdkde_score(xd, h, workspace=ws, flags=f))
        for what, (call, run) in calls.items():
            if d <= (6 if what in ("score", "points") else 3):
                continue                                        # (no matrix units there)
            plan = P.sdkde_describe_plan(n, m, d, call, flags)
            assert plan["splits"] == splits and not plan["thin"]
            got = run(torch.empty(plan["workspace_bytes"], dtype=torch.uint8, device="cuda"), flags)
            assert not torch.equal(got, run(P.make_workspace(n, m, d), shift)), what      # (the fp32 mode's kernels have other bits)
            got = got.cpu().numpy()
            if what == "laplace":
                assert_laplace_close(got, ref[what], size, f"{what} d={d}")
            elif what == "log":
                assert_log_density_close(got, ref[what], f"{what} d={d}")
            elif mode == 3:         # weights of one fp16 value: 2^-11 of sum phi |x - p| / (h^2 D) at most, see the header
                pull = np.array([np.sum(w * np.linalg.norm(x - p, axis=1)) / np.sum(w) for p in (x[at] if what == "score" else q).astype(np.float64)
                                 for w in [np.exp(-(np.sum((x - p) ** 2, axis=1) - np.min(np.sum((x - p) ** 2, axis=1))) / (2 * h * h))]])
                err = np.linalg.norm((got[at] if what == "score" else got) - ref[what], axis=1)
                assert np.all(err <= 2.0**-11 * pull / h**2 + score_resolution(x, x[at] if what == "score" else q, h)), (err * h**2 / pull).max()
            else:
                assert_score_close(got[at] if what == "score" else got, ref[what], f"{what} d={d}", score_resolution(x, x[at] if what == "score" else q, h))
