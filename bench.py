"""Benchmark of the SD-KDE hot path on one MI355X.

A step is one pass of the whole path (score at all samples -> debias -> KDE of the shifted samples at the
queries) over one synthetic batch that is already resident in HBM.  Prints one JSON line: the headline
numbers for --config (default C5, the shape the metric is quoted on), a `per_config` block with the other
configs timed in the same process, the separately reported modes with their own bounds, and the CPU oracle
timed on a bounded sample of the same workload, which also serves as the reference of the sampled parity check.

  python bench.py [--gpus 1] [--steps K] [--warmup W] [--config C5] [--no-cpu-baseline] [--no-other-modes]
                  [--no-per-config]
"""
import argparse
import glob
import json
import os
import re
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

# The paper's two timed shapes (one RTX A6000, TF32 dots), keyed by (config, n, m): seconds end to end.
PAPER_SECONDS = {("C5", 1048576, 131072): 2.3,        # abstract / conclusion
                 ("C2", 32768, 4096): 2.11e-3}        # runtime table of the Results section (--config C2 --m 4096)
MODE_FLAGS = {"fp32": 0, "fp16x2": 1, "fp16x2_all": 2, "fp16x2_phi16": 3, "symmetric": 32}
MODE_NOTES = {
    "fp16x2": "inputs split into fp16 hi+lo on the fp16 matrix units, fp32 accumulate: served by the fp32 mode's kernels",
    "fp16x2_all": "both contractions on the fp16 matrix units (inputs and Phi split into fp16 hi+lo), fp32 accumulate, "
                  "exp and row sums fp32",
    "fp16x2_phi16": "cross-term inputs as fp16 hi+lo, Phi X on the fp16 matrix units with every weight rounded to one fp16 value "
                    "(the row sums take the same rounded weights); fp32 accumulate, exp fp32: the least precise mode",
    "symmetric": "fp32 path; the score computes each unordered pair of samples once (phi_ij = phi_ji) and is still "
                 "counted as n^2 pairs, as the paper counts them"}


def traffic_from_profile(config, plan, launch_ms=None):
    """HBM bytes per launch of the score main kernel as the committed rocprofv3 --pmc summary of this config
    recorded them (FETCH_SIZE / WRITE_SIZE, calibrated on a plain streaming kernel), with the kernel's algorithmic
    bytes beside them: the prepared samples read once plus one partial-sum slot written per split."""
    files = sorted(glob.glob(os.path.join(ROOT, "profiles", f"pipeline_{config}_*.txt")))
    if not files:
        return None, None
    text = open(files[0]).read()
    m = re.search(r"^traffic_json (.*)$", text, flags=re.M)
    if not m:
        return None, None
    rec = json.loads(m.group(1))
    n_pad, m_pad, dp, slots = plan["n_pad"], plan["m_pad"], plan["dp"], plan["partial_slots"]
    xt = plan["xt_scale"] * n_pad * dp if plan["off_xt"] >= 0 else 0
    operand_bytes = 4.0 if plan["thin"] else 6.0              # fp32 coordinates, or their parts
    algorithmic = operand_bytes * (n_pad * dp + xt) + 4.0 * n_pad + 4.0 * slots * m_pad * ((dp + 1) if plan["off_part_t"] >= 0 else 1)
    detail = {"source": os.path.relpath(files[0], ROOT), "kernel": rec["kernel"], "read_bytes": rec["read_bytes"],
              "written_bytes": rec["written_bytes"], "algorithmic_bytes_of_the_launch": algorithmic,
              "ratio_to_algorithmic": rec["bytes"] / algorithmic,
              "hbm_gb_per_s": (rec["bytes"] / (launch_ms * 1e-3) / 1e9) if launch_ms else None,
              "hbm_frac_of_8_tb_per_s": (rec["bytes"] / (launch_ms * 1e-3) / 8e12) if launch_ms else None,
              "note": "re-reads of the streamed samples come from L2 misses per XCD (each XCD streams its share of the "
                      "samples once per round of resident workgroups); HBM stays non-binding"}
    return rec["bytes"], detail


class Workload:
    """One config resident on the GPU, with its outputs and a workspace that serves every mode."""

    def __init__(self, P, torch, sdkde_inputs, name, seed, n=None, m=None):
        self.P, self.torch, self.name = P, torch, name
        self.x, self.q, self.h = sdkde_inputs.make(name, seed=seed, n=n, m=m)
        self.n, self.d = self.x.shape
        self.m = self.q.shape[0]
        dev = torch.device("cuda:0")
        self.xd, self.qd = torch.from_numpy(self.x).to(dev), torch.from_numpy(self.q).to(dev)
        self.ws = P.make_workspace(self.n, self.m, self.d, device=dev, flags=P.SDKDE_FLAG_SYMMETRIC)
        self.s = torch.empty_like(self.xd)
        self.x_sd = torch.empty_like(self.xd)
        self.dens = torch.empty(self.m, dtype=torch.float32, device=dev)
        self.logd = torch.empty(self.m, dtype=torch.float32, device=dev)
        self.pairs = float(self.n) * self.n + float(self.m) * self.n

    def step(self, flags=0):
        P = self.P
        P.sdkde_score(self.xd, self.h, out=self.s, workspace=self.ws, flags=flags)
        P.sdkde_debias(self.xd, self.s, self.h, out=self.x_sd)
        P.sdkde_eval(self.x_sd, self.qd, self.h, density_out=self.dens, log_density_out=self.logd, workspace=self.ws,
                     flags=flags)

    def fused_step(self, flags=0):
        self.P.sdkde_fit_eval(self.xd, self.qd, self.h, score_out=self.s, samples_sd_out=self.x_sd, density_out=self.dens,
                              log_density_out=self.logd, workspace=self.ws, flags=flags)

    def graph_replay_ms(self, steps):
        """ms per replay of sdkde_fit_eval captured once into a HIP graph on a side stream (what a caller with a small,
        fixed-shape problem in a loop would do: one graph launch instead of one launch per kernel); the replayed
        outputs are checked against the eager call's bit for bit."""
        torch = self.torch
        self.fused_step()
        torch.cuda.synchronize()
        want = [t.clone() for t in (self.s, self.x_sd, self.dens, self.logd)]
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            self.fused_step()
            side.synchronize()
            with torch.cuda.graph(graph, stream=side):
                self.fused_step()
        torch.cuda.synchronize()
        for t in (self.s, self.x_sd, self.dens, self.logd):
            t.fill_(float("nan"))
        for _ in range(3):
            graph.replay()
        torch.cuda.synchronize()
        same = all(torch.equal(a, b) for a, b in zip((self.s, self.x_sd, self.dens, self.logd), want))
        ms = float("inf")
        for _ in range(3):
            t0 = time.perf_counter()
            for _ in range(steps):
                graph.replay()
            torch.cuda.synchronize()
            ms = min(ms, (time.perf_counter() - t0) / steps * 1e3)
        del graph
        return ms, same

    def timed(self, fn, steps, warmup):
        """(seconds per step by the host clock around synchronisations, sorted per-step ms from events or None,
        main-kernel ms per launch of the score and of the eval call from the library's own events on the launch
        stream).  Where a step lasts milliseconds, the kernel events and one mark per step are recorded inside the
        timed region.  Every event costs ~3 us on this machine (the next kernel waits for it): four kernel events
        and a mark are 40 % of a C1 step, so short steps are timed with no event at all and the kernel events
        are taken over a second pass of the same steps right after."""
        P, torch = self.P, self.torch
        for _ in range(warmup - 1):
            fn()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        if warmup > 0:
            fn()                              # the last warm-up step, timed alone to see how long a step is
        torch.cuda.synchronize()
        long_steps = (time.perf_counter() - t0 if warmup > 0 else self.pairs / 2e12) >= 5e-3
        marks = [torch.cuda.Event(enable_timing=True) for _ in range(steps + 1)] if long_steps else None
        P.sdkde_profile_enable(long_steps)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        if long_steps:
            marks[0].record()
        for k in range(steps):
            fn()
            if long_steps:
                marks[k + 1].record()
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        per_step = sorted(marks[k].elapsed_time(marks[k + 1]) for k in range(steps)) if long_steps else None
        if not long_steps:
            P.sdkde_profile_enable(True)
            for _ in range(min(steps, 200)):
                fn()
            torch.cuda.synchronize()
        (ls, score_ms), (le, eval_ms) = P.sdkde_profile_summary(0), P.sdkde_profile_summary(1)
        P.sdkde_profile_enable(False)
        return dt / steps, per_step, score_ms / max(ls, 1), eval_ms / max(le, 1)

    def rooflines(self, score_ms, eval_ms, mode="fp32"):
        from paper_2602_10378_amd import cost_model as cm
        P, n, m, d = self.P, self.n, self.m, self.d
        flags = MODE_FLAGS[mode]
        plan_s, plan_e = P.sdkde_describe_plan(n, n, d, 0, flags), P.sdkde_describe_plan(n, m, d, 2, flags)
        # the fp32 mode's matrix path multiplies two fp16 parts per operand, its symmetric mode three bf16 parts
        # (which serve the fp16x2 mode, too, and whatever runs as it)
        eff = {"fp32": "half2", "fp16x2": "half2", "symmetric": "symmetric_bf16x3"}.get(mode, mode)
        if mode == "symmetric" and not plan_s["symmetric"]:
            eff = "half2"
        if mode == "fp16x2_all" and plan_s["xt_scale"] != 2:
            eff = "half2"
        if mode == "fp16x2_phi16" and plan_s["dp"] != 16:
            eff = "half2"
        out = {}
        for key, stage, ms, plan, pairs in (("roofline", "score", score_ms, plan_s, float(n) * n),
                                            ("roofline_eval_kernel", "eval", eval_ms, plan_e, float(m) * n)):
            thin = bool(plan["thin"])
            stage_eff = "half2" if (stage == "eval" and eff == "symmetric_bf16x3") else eff
            r = cm.roofline(stage, d, pairs, ms * 1e-3, stage_eff, thin)
            r["launch_ms"] = ms
            r["kernel"] = ("pair_thin_kernel" if thin else "pair_sym_kernel + in-block pass" if stage_eff == "symmetric_bf16x3"
                           else "pair_half_kernel" if stage_eff == "half2" else "pair_mfma_kernel") + f" ({stage})"
            r["ceiling"] = self.mix_ceiling(stage, stage_eff, thin, ms, pairs, max(r["seconds_at_peak"].values()))
            out[key] = r
        return out, plan_s

    def mix_ceiling(self, stage, mode, thin, ms, pairs, at_peak_s):
        """What this kernel's instruction mix can reach on gfx950, where matrix and vector work of a SIMD overlap little
        (fp32 MFMA: not at all): SIMD clocks per 256 pairs (nominal 2.4 GHz, 1024 SIMDs) of the kernel as timed, of its mix as
        sdkde_peaks measures it (profiles/peaks_mfma_valu_coissue.txt), and of the bound resource alone at its
        published peak; frac = the last over the second = the share of the peak the mix allows."""
        d = self.d
        to_clk = lambda seconds: seconds * 1024 * 2.4e9 / (pairs / 256.0)
        out = {"kernel_clk_per_256_pairs": to_clk(ms * 1e-3), "resource_clk_per_256_pairs_at_peak": to_clk(at_peak_s),
               "mix_clk_per_256_pairs": None, "frac": None}
        blocks = -(-d // 16)
        if thin:
            plain = (3 * d + 1) if stage == "score" else (2 * d + 1)
            out["mix_clk_per_256_pairs"] = 4 * (8.1 + 3.05 * plain)
            out["basis"] = ("per pair and lane one v_exp_f32 (8.1 clk per wave instruction, overlaps nothing) and the plain "
                            "instructions at the 3.05 clk measured next to exps (2 at the published rate)")
        elif mode == "half2":
            score = stage == "score"
            mfmas = 3 * (blocks // 2) + (blocks % 2 and (1 if (d - 1) % 16 < 8 else 2)) + (1.5 * blocks if score else 0)
            plain = (4 if blocks % 2 else 8) + (4 + 2 * blocks if score else 0)
            out["mix_clk_per_256_pairs"] = 16.0 * mfmas + 4 * 8.1 + 2.4 * plain + 4.6 * (8 if score else 0)
            out["basis"] = ("per 16x16 tile: the fp16 MFMAs at 16 clk each (about 21 under the power limit), 4 v_exp_f32 (8.1 clk), plain "
                            "instructions at 2.4, conversions and v_fma_mix_f32 at 4.6, added up: they overlap by little")
        elif blocks == 1:
            measured = {("symmetric_bf16x3", "score"): (155.0, "9 bf16 MFMAs at 16 clk, 4 exp, split, row and column sums and fold per tile of "
                                                               "unordered pairs, added up: 310 clk per 512 ordered pairs"),
                        ("fp16x2", "score"): (226.0, "2 fp16 + 4 fp32 MFMAs + 4 exp + 8 add: 226-250 clk"),
                        ("fp16x2", "eval"): (92.0, "2 fp16 MFMAs + 4 exp + 8 add: 92-108 clk"),
                        ("fp16x2_all", "score"): (139.0, "4 fp16 MFMAs + 4 exp + 16 plain instructions: 139-147 clk")}
            key = (mode if stage == "score" else "fp16x2", stage)
            measured[("fp16x2_phi16", "score")] = (107.0, "3 fp16 MFMAs + 4 exp + 10 plain instructions (4 add, 2 cvt, 2 dot2, 2 mov): 107-115 clk")
            if key in measured:
                out["mix_clk_per_256_pairs"], out["basis"] = measured[key]
        if out["mix_clk_per_256_pairs"]:
            out["frac"] = out["resource_clk_per_256_pairs_at_peak"] / out["mix_clk_per_256_pairs"]
        return out

    def run(self, steps, warmup, fn=None, mode="fp32"):
        flags = MODE_FLAGS[mode]
        sec, per_step, score_ms, eval_ms = self.timed(fn or (lambda: self.step(flags)), steps, warmup)
        roofs, plan = self.rooflines(score_ms, eval_ms, mode)
        out = {"ms_per_step": sec * 1e3, "value": self.pairs / sec, "unit": "pairs/s", "steps": steps,
               "ms_per_step_min": per_step[0] if per_step else None,
               "ms_per_step_median": per_step[len(per_step) // 2] if per_step else None,
               "stages_ms": {"score_main_kernel": score_ms, "eval_main_kernel": eval_ms,
                             "everything_else": sec * 1e3 - score_ms - eval_ms}}
        out.update(roofs)
        return out, plan


def oracle_sample(w, budget_s=15.0):
    """The CPU-baseline leg: the double-precision oracle (as is) timed on a bounded sample of the same workload,
    score rows and queries chosen as the parity tests choose them (random rows plus the rows at tile, row-block
    and split boundaries), each against ALL n samples.  The eval leg evaluates the KDE of the unshifted samples
    (the oracle cannot produce all n shifted samples at this size; the cost per pair is the same).  Returns the
    baseline record and the reference values for the sampled parity checks."""
    import oracle
    import sdkde_inputs
    n, m = w.n, w.m
    cal_rows, rate = 16, 0.0
    while True:                      # calibrate on a run long enough to amortise thread start-up
        cal_rows = min(n, cal_rows * 4)
        t0 = time.perf_counter()
        oracle.score(w.x, w.h, points=w.x[:cal_rows])
        cal = time.perf_counter() - t0
        rate = cal_rows * n / max(cal, 1e-9)
        if cal >= 0.5 or cal_rows == n:
            break
    want_rows = int(min(n, max(cal_rows, budget_s * rate / (n * (1.0 + m / n)))))
    rows = sdkde_inputs.sample_rows(n, max(want_rows - 48, 16), seed=0)
    qrows = sdkde_inputs.sample_rows(m, max(int(round(len(rows) * m / n)) - 48, 16), seed=1)
    t0 = time.perf_counter()
    s_ref = oracle.score(w.x, w.h, points=w.x[rows])
    logp_ref = oracle.eval_log_density(w.x, w.q[qrows], w.h)
    dt = time.perf_counter() - t0
    pairs = float(len(rows)) * n + float(len(qrows)) * n
    base = {"value": pairs / dt, "unit": "pairs/s", "cores": oracle.threads(), "kind": "oracle",
            "whole_config_seconds_extrapolated": w.pairs / (pairs / dt),
            "sample": f"{len(rows)} of {n} score rows + {len(qrows)} of {m} queries (random + tile/split-boundary rows), "
                      f"each against all {n} samples ({pairs:.3g} pairs in {dt:.1f} s, fp64)"}
    return base, {"rows": rows, "qrows": qrows, "s_ref": s_ref, "logp_ref": logp_ref}


def oracle_whole(w):
    """A config small enough for the oracle to run whole: the full chain (score at every sample, shift, KDE of the
    shifted samples at every query) timed on the host cores, and the GPU pass compared with it element by element."""
    import numpy as np
    import oracle
    sys.path.insert(0, os.path.join(ROOT, "tests"))
    from parity import score_error
    t0 = time.perf_counter()
    s_ref, _, logp_ref = oracle.sd_kde_log_density(w.x, w.q, w.h)
    dt = time.perf_counter() - t0
    base = {"value": w.pairs / dt, "unit": "pairs/s", "cores": oracle.threads(), "kind": "oracle",
            "sample": f"the whole config: score at all {w.n} samples, shift, KDE of the shifted samples at all {w.m} "
                      f"queries ({w.pairs:.3g} pairs in {dt:.2f} s, fp64)"}
    w.step()
    worst, frob = score_error(w.s.cpu().numpy(), s_ref)
    logd = w.logd.cpu().numpy().astype(np.float64)
    return base, {"score_worst_of_allowance": worst, "score_rel_frobenius_vs_oracle": frob,
                  "max_abs_log_density_err_vs_oracle": float(np.max(np.abs(logd - logp_ref))),
                  "rows": w.n, "queries": w.m, "tolerance": 1e-3,
                  "density": "SD-KDE (of the shifted samples), whole pipeline"}


def parity_on_sample(w, ref, flags):
    """Score of the mode on the sampled rows and KDE of the unshifted samples at the sampled queries, against the
    oracle's values: per-point worst error as a multiple of the 1e-3 allowance, and the global figures."""
    import numpy as np
    sys.path.insert(0, os.path.join(ROOT, "tests"))
    from parity import score_error
    P, torch = w.P, w.torch
    P.sdkde_score(w.xd, w.h, out=w.s, workspace=w.ws, flags=flags)
    got = w.s[torch.from_numpy(ref["rows"]).to(w.s.device)].cpu().numpy()
    worst, frob = score_error(got, ref["s_ref"])
    _, logd = P.sdkde_eval(w.xd, w.qd, w.h, want="log", workspace=w.ws, flags=flags & ~32)
    lp = logd[torch.from_numpy(ref["qrows"]).to(logd.device)].cpu().numpy().astype(np.float64)
    return {"score_worst_of_allowance": worst, "score_rel_frobenius_vs_oracle": frob,
            "max_abs_log_density_err_vs_oracle": float(np.max(np.abs(lp - ref["logp_ref"]))),
            "rows": int(len(ref["rows"])), "queries": int(len(ref["qrows"])), "tolerance": 1e-3}


def _round(node):
    if isinstance(node, dict):
        return {k: _round(v) for k, v in node.items()}
    if isinstance(node, float):
        return float(f"{node:.5g}")
    return node


def _slim_roofline(r, with_clocks=False):
    out = {k: r[k] for k in ("bound", "resource", "achieved", "peak", "unit", "frac") if k in r}
    if "traffic" in r:
        out["traffic"] = r["traffic"]
    if with_clocks:
        out["kernel_clk_per_256_pairs"] = r["ceiling"]["kernel_clk_per_256_pairs"]
        out["mix_clk_per_256_pairs"] = r["ceiling"]["mix_clk_per_256_pairs"]
    return out


def _slim_run(rec, with_clocks=False):
    out = {"ms_per_step": rec["ms_per_step"], "value": rec["value"], "score_ms": rec["stages_ms"]["score_main_kernel"],
           "eval_ms": rec["stages_ms"]["eval_main_kernel"], "roofline": _slim_roofline(rec["roofline"], with_clocks),
           "eval_frac": rec["roofline_eval_kernel"]["frac"]}
    if "fused_call_ms_per_step" in rec:
        out["fused_call_ms_per_step"] = rec["fused_call_ms_per_step"]
    if "fused_call_graph_replay_ms_per_step" in rec:
        out["fused_call_graph_replay_ms_per_step"] = rec["fused_call_graph_replay_ms_per_step"]
    if "config" in rec:
        out.update({k: rec["config"][k] for k in ("n", "m", "d")})
    if "parity_on_sample" in rec:
        ps = rec["parity_on_sample"]
        out["err_vs_oracle"] = {k: ps[k] for k in ("score_rel_frobenius_vs_oracle", "score_worst_of_allowance",
                                                    "max_abs_log_density_err_vs_oracle", "rows", "queries")}
    if "cpu_baseline" in rec:
        out["cpu_baseline"] = {k: rec["cpu_baseline"][k] for k in ("value", "unit", "cores", "kind")}
    return out


def compact(out):
    """The record as printed by default, a few KB: the headline entries in full (without the explanatory strings),
    one short record per separately reported mode and per config, floats rounded to five significant digits.
    --verbose prints everything."""
    slim = {k: v for k, v in out.items() if k not in ("other_modes", "per_config")}
    for key in ("roofline", "roofline_eval_kernel"):
        r = dict(slim[key])
        for drop in ("work_per_pair", "seconds_at_peak"):
            r.pop(drop, None)
        r["ceiling"] = {k: v for k, v in r["ceiling"].items() if k != "basis"}
        if "traffic_detail" in r:
            r["traffic_detail"] = {k: v for k, v in r["traffic_detail"].items() if k not in ("note", "kernel")}
        slim[key] = r
    if "other_modes" in out:
        slim["other_modes"] = {k: (v if "error" in v else _slim_run(v, with_clocks=True)) for k, v in out["other_modes"].items()}
    if "per_config" in out:
        slim["per_config"] = {k: (v if "error" in v else _slim_run(v)) for k, v in out["per_config"].items()}
    return _round(slim)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--config", default="C5")
    ap.add_argument("--seed", type=int, default=0)
    ap.add_argument("--n", type=int, default=None, help="override the config's sample count (same distribution)")
    ap.add_argument("--m", type=int, default=None, help="override the config's query count")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-other-modes", action="store_true", help="skip the separately reported modes")
    ap.add_argument("--no-per-config", action="store_true", help="skip the block that times the other configs")
    ap.add_argument("--verbose", action="store_true", help="keep the explanatory strings and every derived figure in the line")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        sys.exit("bench.py: this build is single-GPU; run with --gpus 1 (no multi-GPU path exists)")

    import torch
    import paper_2602_10378_amd as P
    import sdkde_inputs

    P.load()
    cfg = sdkde_inputs.CONFIGS[args.config]
    w = Workload(P, torch, sdkde_inputs, args.config, args.seed, args.n, args.m)
    n, m, d = w.n, w.m, w.d
    main_run, plan = w.run(args.steps, args.warmup)
    s_fp32, logd_fp32 = w.s.clone(), w.logd.clone()
    default_shape = args.n is None and args.m is None
    if main_run["roofline"]["bound"] == "mfma":
        r = main_run["roofline"]
        r["flops_per_launch"] = r["work_per_pair"][r["resource"]] * float(n) * n
    traffic, traffic_detail = (traffic_from_profile(args.config, plan, main_run["roofline"]["launch_ms"]) if default_shape
                               else (None, None))
    main_run["roofline"]["traffic"] = traffic
    if traffic_detail:
        main_run["roofline"]["traffic_detail"] = traffic_detail

    mode_steps = max(1, min(args.steps, 5))
    other = {}
    if not args.no_other_modes:
        fused, _ = w.run(mode_steps, 1, fn=w.fused_step)
        fused["max_abs_log_density_diff_vs_three_calls"] = float((w.logd - logd_fp32).abs().max())
        fused["note"] = "sdkde_fit_eval: score, shift and eval in one call (fp32 path)"
        other["fused_call"] = fused
        if not plan["thin"]:
            modes = ["fp16x2"]
            if P.sdkde_describe_plan(n, n, d, 0, P.SDKDE_PREC_FP16X2_ALL)["xt_scale"] == 2:      # else it runs as fp16x2 (d > 16)
                modes.append("fp16x2_all")
                modes.append("fp16x2_phi16")
            if P.sdkde_describe_plan(n, n, d, 0, P.SDKDE_FLAG_SYMMETRIC)["symmetric"]:
                modes.append("symmetric")
            for mode in modes:
                try:
                    rec, _ = w.run(mode_steps, 1, mode=mode)
                    rec["score_rel_frobenius_vs_fp32_path"] = float((w.s - s_fp32).norm() / s_fp32.norm())
                    rec["max_abs_log_density_diff_vs_fp32_path"] = float((w.logd - logd_fp32).abs().max())
                    rec["note"] = MODE_NOTES[mode]
                    other[mode] = rec
                except Exception as e:                               # the headline record must survive
                    other[mode] = {"error": f"{type(e).__name__}: {e}"[:300]}

    paper_s = PAPER_SECONDS.get((args.config, n, m))
    sec = main_run["ms_per_step"] * 1e-3
    out = {
        "metric": "pair-interactions/sec (score n^2 + eval m*n)", "value": main_run["value"], "unit": "pairs/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": main_run["ms_per_step"],
        "higher_is_better": True, "scaling": None,
        "vs_baseline": (paper_s / sec) if paper_s else None,
        "baseline_note": (f"paper: {paper_s:g} s end-to-end at this shape on one RTX A6000 with TF32 dots "
                          "(context, other hardware)") if paper_s else None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": f"{cfg.name}: n={n} samples, m={m} queries, d={d}, Gaussian mixture, "
                               f"Silverman h={w.h:.4f}, score+debias+eval", "n": n, "m": m, "d": d, "seed": args.seed},
        "end_to_end_s": sec,
    }
    for key in ("ms_per_step_min", "ms_per_step_median", "stages_ms", "roofline", "roofline_eval_kernel"):
        out[key] = main_run[key]

    if not args.no_cpu_baseline:
        base, ref = oracle_sample(w)
        out["cpu_baseline"] = base
        out["parity_on_sample"] = parity_on_sample(w, ref, 0)
        for mode in other:
            if mode in MODE_FLAGS and "error" not in other[mode]:
                other[mode]["parity_on_sample"] = parity_on_sample(w, ref, MODE_FLAGS[mode])
    if other:
        out["other_modes"] = other

    if not args.no_per_config and default_shape:
        # The other configs, timed in this process with the same protocol (three calls per step; the one-call
        # entry point beside them, which is what a small problem should use): driver-visible numbers per config.
        del w, s_fp32, logd_fp32
        torch.cuda.empty_cache()
        per = {}
        shapes = [(name, None, None) for name in ("C1", "C2", "C3", "C4", "C5") if name != args.config]
        shapes.append(("C2", 32768, 4096))          # the shape of the paper's runtime table
        for name, n_o, m_o in shapes:
            key = name if n_o is None else f"{name}_n{n_o}_m{m_o}"
            try:
                wc = Workload(P, torch, sdkde_inputs, name, args.seed, n_o, m_o)
                est = wc.pairs / 1.5e12                                  # seconds per step, roughly
                k = int(max(3, min(200, 0.6 / max(est, 1e-6))))
                # short steps: enough warm-up for the clocks to settle (a few hundred launches), best of three runs
                warm = int(max(3, min(3000, 0.15 / max(est, 1e-6))))
                tries = 3 if est < 5e-3 else 1
                runs = [wc.run(k, warm if r == 0 else 3) for r in range(tries)]
                rec, plan_c = min(runs, key=lambda rp: rp[0]["ms_per_step"])
                rec["ms_per_step_of_each_run"] = [r[0]["ms_per_step"] for r in runs]
                fused = min((wc.run(k, 3, fn=wc.fused_step)[0] for _ in range(tries)), key=lambda r: r["ms_per_step"])
                rec["fused_call_ms_per_step"] = fused["ms_per_step"]
                rec["fused_call_value"] = fused["value"]
                if est < 5e-3:                                           # launch-bound sizes: the same call replayed from a HIP graph
                    try:
                        rec["fused_call_graph_replay_ms_per_step"], rec["graph_replay_bitwise_equal_to_eager"] = wc.graph_replay_ms(k)
                    except Exception as e:                               # an extra: its failure must not cost the record
                        rec["graph_replay_error"] = f"{type(e).__name__}: {e}"[:200]
                rec["config"] = {"n": wc.n, "m": wc.m, "d": wc.d, "h": wc.h}
                if not args.no_cpu_baseline:
                    if wc.pairs <= 4e9:                                  # a few seconds of oracle time: run it whole
                        rec["cpu_baseline"], rec["parity_on_sample"] = oracle_whole(wc)
                    else:
                        rec["cpu_baseline"], ref_c = oracle_sample(wc, budget_s=3.0)
                        rec["parity_on_sample"] = parity_on_sample(wc, ref_c, 0)
                traffic, detail = (traffic_from_profile(name, plan_c, rec["roofline"]["launch_ms"]) if (n_o is None and m_o is None)
                                   else (None, None))
                rec["roofline"]["traffic"] = traffic
                if detail:
                    rec["roofline"]["traffic_detail"] = detail
                ps = PAPER_SECONDS.get((name, wc.n, wc.m))
                if ps:
                    rec["paper_seconds_other_hardware"] = ps
                per[key] = rec
                del wc
                torch.cuda.empty_cache()
            except Exception as e:                                   # the headline record must survive
                per[key] = {"error": f"{type(e).__name__}: {e}"[:300]}
        out["per_config"] = per
    print(json.dumps(out if args.verbose else compact(out), separators=(",", ":")))


if __name__ == "__main__":
    main()
