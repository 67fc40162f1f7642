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
