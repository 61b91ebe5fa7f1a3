"""Autotuner for the kernel variants of stap_run.

For each shape class it runs stap_run on a seeded cube of that shape under
every candidate variant of the fused covariance->solve kernel (the
column-sweep solve on a 16 x 16 or 32 x 16 thread grid per system, the
blocked matrix-core solve with 4 or 8 waves, or the stage covariance
followed by the one-wave solve), keeps the fastest by HIP-event time, and
stores the choice in a JSON cache keyed by GPU architecture, kernel kind,
DOF class, steering class, precision and refinement.  It then times the
stage covariance kernel under each wave count per system (kind "cov"), which
must reproduce the default bit for bit.  (Kind "inner", range tiles per wave
step of the inner products, has no effect any more and is not timed; caches
that hold it still load.)  The binding applies the cache
(``tune_cache.json`` beside this file, or ``$STAP_TUNE_CACHE``) at import.

    python -m paper_2203_06233_amd.tune [--workload large] [--reps 10]
"""
from __future__ import annotations

import argparse
import json
import os
import sys

CACHE = os.environ.get("STAP_TUNE_CACHE",
                       os.path.join(os.path.dirname(os.path.abspath(__file__)), "tune_cache.json"))
CANDIDATES = (16, 32, 4, 8)


def candidates(dof, refine, kind=0, n_steer=16):
    """Variants worth timing for a shape (the 32-row grid needs D > 32; above
    D = 128 the column sweep picks its own grid and the blocked solve runs
    with 16 waves under variant 8).  Variant 1 (D <= 96, S <= 32) is the
    one-wave register-resident solve: as a stage solve (kind 1), and for
    kind 0 stap_run's route through the stage covariance and that solve."""
    if dof > 128:
        return [0, 8]
    out = [v for v in CANDIDATES if not (v == 32 and dof <= 32)]
    if dof <= 96 and n_steer <= 32:
        out.append(1)
    return out


def arch() -> str:
    import torch
    p = torch.cuda.get_device_properties(0)
    return getattr(p, "gcnArchName", p.name).split(":")[0]


KINDS = {"fused": 0, "stage": 1, "cov": 2, "inner": 3}


def kernel_candidates(kind, dof, precision):
    """Values that kinds "cov" (waves per system) and "inner" (range tiles per
    wave step, without effect) take for a DOF class; 0 is the built-in default."""
    if kind == KINDS["cov"]:
        if dof <= 32 or dof > 128:
            return [0]
        return [0, 4, 8] if dof <= 64 else [0, 4, 16] if dof <= 96 else [0, 16]
    if kind == KINDS["inner"]:
        return [0, 1, 2] if precision != "fp32" and dof <= 128 else [0, 1, 2, 4]
    return [0]


def kind_of(wl, precision):
    """stap_run takes the fused covariance->solve kernel (kind 0) for D <= 128
    in FP32 or BF16, else the stage covariance and solve (kind 1)."""
    return 0 if wl.dof <= 128 and precision != "fp8" else 1


def key(arch_name, dof, n_steer, precision, refine, kind=0):
    name = [k for k, v in KINDS.items() if v == kind][0]
    return f"{arch_name}|{name}|dof<={dof}|s<={n_steer}|{precision}|refine={int(refine > 0)}"


def load_cache(path=CACHE):
    if not os.path.exists(path):
        return {}
    with open(path) as f:
        return json.load(f)


def apply_cache(stap, path=CACHE, arch_name=None):
    """Write every cached choice for this architecture into the library."""
    cache = load_cache(path)
    if not cache:
        return 0
    n = 0
    for k, v in cache.items():
        parts = k.split("|")
        if arch_name is not None and parts[0] != arch_name:
            continue
        kind = KINDS[parts[1]]
        dof = int(parts[2].split("<=")[1])
        s = int(parts[3].split("<=")[1])
        prec = parts[4]
        refine = int(parts[5].split("=")[1])
        stap.tune_set(dof, s, prec, refine, int(v["variant"]), kind=kind)
        n += 1
    return n


def tune_workload(wl, precision, refine, reps=10, warmup=3):
    import torch

    import synth
    from paper_2203_06233_amd import stap

    dev = torch.device("cuda:0")
    cube = torch.from_numpy(synth.make_cube(wl)).to(dev)
    V = torch.from_numpy(synth.steering(wl)).to(dev)
    prob = stap.problem(wl.n_chan, wl.n_pulse, wl.n_range, wl.tdof, wl.n_block, wl.n_steer,
                        load_eps=wl.load_eps, precision=precision, refine_steps=refine, n_sub=wl.n_sub)
    runner = stap.Runner([prob], device=dev)
    power = torch.empty((wl.n_pulse, wl.n_steer, wl.n_range), dtype=torch.float32, device=dev)
    W = torch.empty((wl.n_pulse, wl.n_block, wl.n_steer, wl.dof), dtype=torch.complex64, device=dev)
    times = {}
    ref = None
    kind = kind_of(wl, precision)
    for v in candidates(wl.dof, refine, kind, wl.n_steer):
        stap.tune_set(wl.dof, wl.n_steer, precision, refine, v, kind=kind)
        for _ in range(warmup):
            runner.run([cube], [V], powers=[power], weights=[W])
        st = torch.cuda.current_stream()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(st)
        for _ in range(reps):
            runner.run([cube], [V], powers=[power], weights=[W])
        e1.record(st)
        torch.cuda.synchronize()
        times[v] = e0.elapsed_time(e1) / reps
        # every variant computes the same weights up to rounding order (the
        # systems are ill-conditioned, so only a gross disagreement is an error)
        w = W.cpu()
        if ref is None:
            ref = w
        else:
            rel = float(torch.linalg.vector_norm(w - ref) / torch.linalg.vector_norm(ref))
            if not rel <= 1e-2:
                raise RuntimeError(f"variant {v} disagrees with the first variant timed: {rel}")
    best = min(times, key=times.get)
    stap.tune_set(wl.dof, wl.n_steer, precision, refine, best, kind=kind)
    return best, times


def tune_covariance(wl, precision, refine, reps=10, warmup=3):
    """Time stap_covariance on the workload's snapshots under each candidate
    wave count; the outputs must agree bit for bit (the variants only regroup
    the same arithmetic)."""
    import torch

    import synth
    from paper_2203_06233_amd import stap

    dev = torch.device("cuda:0")
    kind = KINDS["cov"]
    cube = torch.from_numpy(synth.make_cube(wl)).to(dev)
    prob = stap.problem(wl.n_chan, wl.n_pulse, wl.n_range, wl.tdof, wl.n_block, wl.n_steer,
                        load_eps=wl.load_eps, precision=precision, refine_steps=refine, n_sub=wl.n_sub)
    snap = stap.doppler(prob, cube)
    cov, delta = stap.covariance(prob, snap)
    times, ref = {}, None
    for v in kernel_candidates(kind, wl.dof, precision):
        stap.tune_set(wl.dof, wl.n_steer, precision, refine, v, kind=kind)
        for _ in range(warmup):
            stap.covariance(prob, snap, cov, delta)
        st = torch.cuda.current_stream()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(st)
        for _ in range(reps):
            stap.covariance(prob, snap, cov, delta)
        e1.record(st)
        torch.cuda.synchronize()
        times[v] = e0.elapsed_time(e1) / reps
        o = cov.cpu()
        if ref is None:
            ref = o
        elif not torch.equal(o, ref):
            raise RuntimeError(f"covariance variant {v} does not reproduce the default bit for bit")
    best = min(times, key=times.get)
    stap.tune_set(wl.dof, wl.n_steer, precision, refine, best, kind=kind)
    return best, times


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--workload", default="all",
                    choices=["all", "small", "medium", "large", "xlarge", "uneven", "paper"])
    ap.add_argument("--reps", type=int, default=10)
    ap.add_argument("--out", default=CACHE)
    args = ap.parse_args()
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    sys.path.insert(0, root)
    import synth

    # the paper's cube shape class (D = 60, S = 32) on a 3000-cell slice of it
    sel = {"small": [synth.SMALL], "medium": [synth.MEDIUM], "large": [synth.LARGE], "xlarge": [synth.XLARGE],
           "uneven": synth.uneven_batch(8), "paper": [synth.with_(synth.PAPER, n_range=3000, n_block=25)]}
    wls = sum(sel.values(), []) if args.workload == "all" else sel[args.workload]
    a = arch()
    cache = load_cache(args.out)
    dof_cls = (16, 32, 48, 64, 96, 128, 160, 192)
    s_cls = (16, 32, 64)
    seen = set()
    for wl in wls:
        dc = next(c for c in dof_cls if wl.dof <= c)
        sc = next(c for c in s_cls if wl.n_steer <= c)
        combos = (("fp32", 0), ("fp8", 1)) if wl.dof > 128 else (("fp32", 0), ("bf16", 1), ("bf16", 0))
        for precision, refine in combos:
            k = key(a, dc, sc, precision, refine, kind_of(wl, precision))
            if k in seen:
                continue
            seen.add(k)
            best, times = tune_workload(wl, precision, refine, reps=args.reps)
            cache[k] = {"variant": best, "ms": {str(v): t for v, t in times.items()}, "workload": wl.name}
            print(json.dumps({"key": k, **cache[k]}), flush=True)
            kk = key(a, dc, sc, precision, refine, KINDS["cov"])
            if kk in seen:
                continue
            seen.add(kk)
            if len(kernel_candidates(KINDS["cov"], wl.dof, precision)) < 2:
                continue
            best, times = tune_covariance(wl, precision, refine, reps=args.reps)
            cache[kk] = {"variant": best, "ms": {str(v): t for v, t in times.items()}, "workload": wl.name}
            print(json.dumps({"key": kk, **cache[kk]}), flush=True)
    with open(args.out, "w") as f:
        json.dump(cache, f, indent=1, sort_keys=True)
    print(f"wrote {args.out}")


if __name__ == "__main__":
    main()
