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
    """Samples in two tight clusters `distance` on either side of the middle along a diagonal, queries up to 50 around the
    middle, at least 1 off it along the axis so that a cluster is the nearer one by more than what fp32 exponents resolve."""
    rng = np.random.default_rng(seed)
    axis = rng.choice([-1.0, 1.0], d) / np.sqrt(d)
    side = np.where(np.arange(n) % 2, 1.0, -1.0)
    x = side[:, None] * distance * axis + rng.standard_normal((n, d))
    q = rng.standard_normal((m, d))
    q *= rng.uniform(0.0, 50.0, m)[:, None] / np.linalg.norm(q, axis=1, keepdims=True)
    along = q @ axis
    q += (np.where(along < 0.0, -1.0, 1.0) * np.maximum(1.0 - np.abs(along), 0.0))[:, None] * axis
    return x.astype(np.float32), q.astype(np.float32)


def _check_shifted_far_clusters(P, x, q, h):
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
        spread = 2.0 * np.linalg.norm(x[::2] - x[::2].mean(axis=0), axis=1).max() / (h * h)
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
    x, q = _two_clusters(n, m, d, distance, d)
    _check_shifted_far_clusters(P, x, q, h)


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
