"""What is timed: the work a program that uses this package has it do, through the public calls.

A case is one call pattern (`call`) at one shape: n samples of dimension d, m queries (or separate points), a data
distribution and the flags of the call.  The shapes are those of the paper's runs as bench.py states them (16-D mixture
at 4096 x 1024, 32768 x 4096, 32768 x 32768 and 1048576 x 131072, the 1-D mixture at 32768 x 65536, the 64-D diagonal
mixture at 262144 x 65536), a tiny pass as a serving loop makes it, and odd sizes and dimensions between them.

Call patterns
  fit_eval      sdkde_fit_eval, score, shifted samples and both densities wanted
  fit_static    sdkde_fit_eval_static, the same on the library's own scratch buffer
  three_calls   sdkde_score at the samples, sdkde_debias, sdkde_eval of the shifted samples
  score         sdkde_score at the samples
  score_points  sdkde_score at m separate points
  eval          sdkde_eval at m queries
  serve         sdkde_eval at m new queries against samples an earlier call on the same workspace has prepared
  laplace       sdkde_eval_laplace at m queries
"""
from __future__ import annotations

import math

import torch

import paper_2602_10378_amd as P

FP32, X2, X2_ALL, X2_PHI16 = (P.SDKDE_PREC_FP32, P.SDKDE_PREC_FP16X2, P.SDKDE_PREC_FP16X2_ALL, P.SDKDE_PREC_FP16X2_PHI16)
SHIFT, SYM, PREPARED = P.SDKDE_FLAG_MAX_SHIFT, P.SDKDE_FLAG_SYMMETRIC, P.SDKDE_FLAG_SAMPLES_PREPARED


def _case(name, call, n, m, d, data="iso", flags=FP32, spread=1.0):
    return {"name": name, "call": call, "n": n, "m": m, "d": d, "data": data, "flags": flags, "spread": spread}


def listed():
    return [
        # a serving loop's smallest pass: a few hundred samples, nothing but launches
        _case("tiny_static_n600_m50_d8", "fit_static", 600, 50, 8),
        # the smallest benchmark config, one call
        _case("fit_n4096_m1024_d16", "fit_eval", 4096, 1024, 16),
        # the paper's table shape (n_test = n_train / 8)
        _case("fit_n32768_m4096_d16", "fit_eval", 32768, 4096, 16),
        # as many queries as samples, as the three separate calls
        _case("calls_n32768_m32768_d16", "three_calls", 32768, 32768, 16),
        # the 1-D benchmark: VALU kernel, queries on a grid
        _case("fit_n32768_m65536_d1", "fit_eval", 32768, 65536, 1, data="mix_1d"),
        # ragged sizes and a dimension between the padded ones
        _case("fit_n30011_m3001_d37", "fit_eval", 30011, 3001, 37),
        # a score field at separate points in space, thin path
        _case("points_n100003_m20011_d3", "score_points", 100003, 20011, 3),
        # queries far from the samples, as a density map or an outlier test has them: two-pass shifted sums
        _case("shifted_eval_n50021_m10007_d24", "eval", 50021, 10007, 24, flags=SHIFT, spread=3.0),
        # the Laplace-corrected estimate, which needs no score pass
        _case("laplace_n65536_m8192_d16", "laplace", 65536, 8192, 16),
        # small batches of queries against a large fitted estimate
        _case("serve_n1048576_m1024_d16", "serve", 1048576, 1024, 16),
        # the 64-D benchmark
        _case("calls_n262144_m65536_d64", "three_calls", 262144, 65536, 64, data="diag"),
        # the headline benchmark
        _case("fit_n1048576_m131072_d16", "fit_eval", 1048576, 131072, 16),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["fit_eval", "fit_eval", "fit_eval", "three_calls", "score", "score_points", "eval", "serve",
                       "laplace", "fit_static"])
    d = _log_uniform(rng, 1, 128) if rng.random() < 0.7 else rng.choice([1, 2, 3, 8, 16, 16, 16, 32, 64, 128])
    data = "mix_1d" if d == 1 else rng.choice(["iso", "iso", "diag"])
    flags, spread = FP32, 1.0
    if rng.random() < 0.25:
        flags = rng.choice([X2, X2_ALL, X2_PHI16])
    if call in ("score_points", "eval", "laplace") and rng.random() < 0.3:
        flags |= SHIFT
        spread = rng.choice([1.0, 2.0])
    if call in ("score", "fit_eval") and rng.random() < 0.15:
        flags |= SYM
    if call == "fit_static":                    # what its 64 MiB scratch buffer serves
        n = _log_uniform(rng, 100, 8000)
        m = _log_uniform(rng, 10, 2000)
    else:
        n = _log_uniform(rng, 200, 262144)
        m = _log_uniform(rng, 50, 65536)
    return {"call": call, "n": n, "m": m, "d": d, "data": data, "flags": flags, "spread": spread}


def _inputs(case, seed):
    """Samples [n, d], queries [m, d] (fp32, on the GPU) and the rule-of-thumb bandwidth of the samples."""
    n, m, d = case["n"], case["m"], case["d"]
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)

    if case["data"] == "mix_1d":                # 0.7 N(0, 1) + 0.3 N(3, 1/4), queries on a grid
        second = torch.rand(n, 1, generator=g, device="cuda") < 0.3
        z = normal(n, 1)
        x = torch.where(second, 3.0 + 0.5 * z, z)
        q = torch.linspace(-5.0, 6.0, m, device="cuda", dtype=torch.float32).reshape(m, 1)
        q += 1e-3 * float(torch.rand(1, generator=g, device="cuda"))
    else:                                       # equal-weight mixture, means ~ N(0, 9), unit or diagonal covariance
        k = 8 if case["data"] == "diag" else 4
        means = 3.0 * normal(k, d)
        scale = torch.ones(k, d, device="cuda")
        if case["data"] == "diag":
            scale = (0.5 + 1.5 * torch.rand(k, d, generator=g, device="cuda")).sqrt()
        lx = torch.randint(0, k, (n,), generator=g, device="cuda")
        x = means[lx] + scale[lx] * normal(n, d)
        lq = torch.randint(0, k, (m,), generator=g, device="cuda")
        q = means[lq] + case["spread"] * scale[lq] * normal(m, d)
    sigma = float(x.double().var(dim=0, unbiased=True).mean().sqrt())
    h = sigma * (4.0 / ((d + 2.0) * n)) ** (1.0 / (d + 4.0))
    return x.contiguous(), q.contiguous(), h


def prepare(case, seed):
    x, q, h = _inputs(case, seed)
    n, m, d, flags, call = case["n"], case["m"], case["d"], case["flags"], case["call"]
    state = {"case": case, "x": x, "q": q, "h": h}
    state["score"] = torch.empty(m if call == "score_points" else n, d, device="cuda", dtype=torch.float32)
    state["x_sd"] = torch.empty_like(x)
    state["density"] = torch.empty(m, device="cuda", dtype=torch.float32)
    state["log_density"] = torch.empty_like(state["density"])
    if call != "fit_static":
        state["workspace"] = P.make_workspace(n, m, d, flags=flags)
    if call == "serve":                         # the program has evaluated its estimate before
        P.sdkde_eval(x, q, h, log_density_out=state["log_density"], workspace=state["workspace"], flags=flags)
    return state


def run(state):
    case, x, q, h = state["case"], state["x"], state["q"], state["h"]
    call, flags, ws = case["call"], case["flags"], state.get("workspace")
    score, x_sd, dens, logd = state["score"], state["x_sd"], state["density"], state["log_density"]
    if call == "fit_eval":
        P.sdkde_fit_eval(x, q, h, score_out=score, samples_sd_out=x_sd, density_out=dens, log_density_out=logd,
                         workspace=ws, flags=flags)
        return {"score": score, "x_sd": x_sd, "density": dens, "log_density": logd}
    if call == "fit_static":
        P.sdkde_fit_eval_static(x, q, h, x_sd, score_out=score, density_out=dens, log_density_out=logd, flags=flags)
        return {"score": score, "x_sd": x_sd, "density": dens, "log_density": logd}
    if call == "three_calls":
        P.sdkde_score(x, h, out=score, workspace=ws, flags=flags)
        P.sdkde_debias(x, score, h, out=x_sd)
        P.sdkde_eval(x_sd, q, h, density_out=dens, log_density_out=logd, workspace=ws, flags=flags)
        return {"score": score, "x_sd": x_sd, "density": dens, "log_density": logd}
    if call == "score":
        return {"score": P.sdkde_score(x, h, out=score, workspace=ws, flags=flags)}
    if call == "score_points":
        return {"score": P.sdkde_score(x, h, points=q, out=score, workspace=ws, flags=flags)}
    if call == "eval":
        P.sdkde_eval(x, q, h, log_density_out=logd, workspace=ws, flags=flags)
        return {"log_density": logd}
    if call == "serve":
        P.sdkde_eval(x, q, h, log_density_out=logd, workspace=ws, flags=flags | PREPARED)
        return {"log_density": logd}
    if call == "laplace":
        return {"density": P.sdkde_eval_laplace(x, q, h, density_out=dens, workspace=ws, flags=flags)}
    raise ValueError(call)


_WITH_SCORE = ("fit_eval", "fit_static", "three_calls", "score", "score_points")
_WITH_EVAL = ("fit_eval", "fit_static", "three_calls", "eval", "serve", "laplace")


def work(case):
    """Each pair once: squared distance 2d, exponential and sum 2, and for the score the weighted sum 2d.  Bytes:
    samples, queries and outputs once."""
    n, m, d, call = case["n"], case["m"], case["d"], case["call"]
    flops, floats = 0, n * d
    if call in _WITH_SCORE:
        rows = m if call == "score_points" else n
        flops += rows * n * (4 * d + 2)
        floats += rows * d + (m * d if call == "score_points" else 0)
    if call in _WITH_EVAL:
        flops += n * m * (2 * d + 2)
        floats += m * d + m
    if call in ("fit_eval", "fit_static", "three_calls"):
        floats += n * d + m
    return {"bytes": 4 * floats, "flops": flops}


def tolerance(case):
    prec = case["flags"] & 15
    if prec == X2_PHI16 and case["d"] <= 16 and case["call"] in _WITH_SCORE:
        return {"rel": 1e-3}                    # single-fp16 weights: 2^-11 a term
    if case["call"] == "laplace":
        return {"rel": 1e-4}                    # signed sum whose terms cancel
    # measured against 64 bits at fp32: up to 5e-6 for the score (d = 128, where T - p D cancels most), 7e-7 elsewhere
    return {"rel": 2e-5}


def _weights(x, p, h, c):
    """-|p - x|^2 / 2h^2 in double, [rows of p, n]; x and p relative to the same centre c."""
    xc, pc = x - c, p - c
    e = torch.addmm((xc * xc).sum(1)[None, :], pc, xc.t(), beta=1.0, alpha=-2.0)
    e += (pc * pc).sum(1)[:, None]
    return e.mul_(-0.5 / (h * h)).clamp_(max=0.0)


def _blocks(n, rows):
    step = max(1, (1 << 27) // n)
    return [(lo, min(rows, lo + step)) for lo in range(0, rows, step)]


def _exact_score(x, p, h, c):
    out = torch.empty(p.shape[0], x.shape[1], device=x.device, dtype=torch.float64)
    for lo, hi in _blocks(x.shape[0], p.shape[0]):
        e = _weights(x, p[lo:hi], h, c)
        w = (e - e.amax(dim=1, keepdim=True)).exp_()
        out[lo:hi] = ((w @ (x - c)) / w.sum(1, keepdim=True) - (p[lo:hi] - c)) / (h * h)
    return out


def _exact_log_density(x, q, h, c):
    n, d = x.shape
    out = torch.empty(q.shape[0], device=x.device, dtype=torch.float64)
    for lo, hi in _blocks(n, q.shape[0]):
        out[lo:hi] = torch.logsumexp(_weights(x, q[lo:hi], h, c), dim=1)
    return out - math.log(n) - d * math.log(h) - 0.5 * d * math.log(2.0 * math.pi)


def _exact_laplace(x, q, h, c):
    n, d = x.shape
    out = torch.empty(q.shape[0], device=x.device, dtype=torch.float64)
    for lo, hi in _blocks(n, q.shape[0]):
        e = _weights(x, q[lo:hi], h, c)
        out[lo:hi] = (e.exp() * (1.0 + 0.5 * d + e)).sum(1)
    return out * math.exp(-math.log(n) - d * math.log(h) - 0.5 * d * math.log(2.0 * math.pi))


def exact(case, seed):
    n, m, d, call = case["n"], case["m"], case["d"], case["call"]
    pairs = (n * (m if call == "score_points" else n) if call in _WITH_SCORE else 0) + (n * m if call in _WITH_EVAL else 0)
    if pairs * (1.0 + d / 32.0) > 6e11:
        return None
    x32, q32, h = _inputs(case, seed)
    x, q = x32.double(), q32.double()
    c = x.mean(dim=0)
    if call == "laplace":
        return {"density": _exact_laplace(x, q, h, c)}
    if call in ("eval", "serve"):
        return {"log_density": _exact_log_density(x, q, h, c)}
    if call == "score_points":
        return {"score": _exact_score(x, q, h, c)}
    s = _exact_score(x, x, h, c)
    if call == "score":
        return {"score": s}
    x_sd = x + 0.5 * h * h * s
    logd = _exact_log_density(x_sd, q, h, c)
    dens = logd.exp()
    # densities of large dimension lie below the fp32 range, where only the logarithm has a value
    return {"score": s, "x_sd": x_sd, "density": dens if float(dens.min()) > 1e-35 else None, "log_density": logd}
