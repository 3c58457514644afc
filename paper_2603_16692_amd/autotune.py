"""Per-parameter choice of the KeySwitch dataflow (DSOB / DPOB / DSOC / DPOC).

The paper's finding (Quantitative Analysis section, Fig. 4) is that the best
dataflow depends on (dnum, N, L) and on the GPU: as the on-chip footprint of a
dataflow (Qualitative Analysis section, Table III and Fig. 3) outgrows the
cache, the best choice moves to the dataflow with the next smaller footprint
(roughly when the cache holds less than about twice the footprint). This
module turns that finding into a per-parameter choice by measurement: it
enumerates the valid plans (dataflow x chunks x NTT split), orders them by the
footprint prior, times each on the device, keeps only plans whose output is
bit-identical to the reference plan's, and caches the fastest per
(GPU architecture, ROCm version, dnum, N, L, batch).

On MI355X the paper's "L2" maps to two levels: a private 4 MB L2 per XCD (32 MB
in all, not shared across XCDs) and the 256 MB MALL (Infinity Cache) shared by
every XCD, through which data written by one kernel and read by the next
passes. The prior therefore compares footprints with the MALL.
"""
import json
import os
import statistics

import torch

from . import (DPOB, DPOC, DSOB, DSOC, STAGED, DATAFLOW_NAMES, HipEvents,
               KsError, PLAN_HOIST_FWD, PLAN_MFMA_BCONV, Plan, make_plan)

WORD = 8
MALL_BYTES = 256 << 20
L2_PER_XCD_BYTES = 4 << 20
CHUNK_RANGE = range(2, 11)  # the paper searches chunks in 2..10 (Quantitative Analysis section)


def footprint_bytes(dnum: int, n: int, ell: int, dataflow: int, chunks: int = 1, batch: int = 1) -> int:
    """The paper's on-chip footprint model: N*L words for DigitSerial, times
    dnum for DigitParallel, divided by `chunks` for OutputChunked (Table III),
    times the batch. (2, 2^15, 10) under DPOB gives 2 * 2^15 * 10 * 8 B."""
    f = n * ell * WORD * batch
    if dataflow in (DPOB, DPOC):
        f *= dnum
    if dataflow in (DSOC, DPOC):
        f //= max(1, chunks)
    return f


def candidate_plans(params, batch: int, chunk_range=CHUNK_RANGE, mfma=(False, True), split=None, tiles=None):
    """Every plan libks accepts for these parameters and batch, without and with the
    flag that asks for the int8-MFMA BConv, and (batch >= 2) with
    the batch on one stream or split over two; for batch >= 4 also the
    digit-parallel plans (DPOB, STAGED) run in passes of batch/2 and batch/4
    items, whose footprint is that of the smaller pass (the batch tile)."""
    if split is None:
        split = (False, True) if batch >= 2 else (False,)
    if tiles is None:
        tiles = sorted({batch // 2, batch // 4} - {0, 1}, reverse=True) if batch >= 4 else []
    plans = []
    for sp in split:
        for mx in mfma:
            for log_r in range(0, 6):
                log_m = params.log_n - log_r
                if log_m < 3 or log_m > 14:
                    continue
                for df in (DSOB, DPOB, STAGED):
                    plans.append(make_plan(df, 1, log_r, mx, sp))
                    if df == DPOB:  # the forward pass of the raised digits as a launch of its own
                        plans.append(make_plan(df, 1, log_r, mx, sp, hoist=True))
                    if df != DSOB and not sp:
                        plans += [make_plan(df, 1, log_r, mx, sp, t) for t in tiles]
                for df in (DSOC, DPOC):
                    for c in chunk_range:
                        if c <= params.ell:
                            plans.append(make_plan(df, c, log_r, mx, sp))
    valid = []
    for p in plans:
        try:
            params.workspace_bytes(batch, p)
            valid.append(p)
        except KsError:
            pass
    return valid


def distinct_plans(params, plans):
    """`plans` without those that launch the same kernels as another one: where a
    digit has 4 primes or more, every BConv runs on the matrix cores with or
    without PLAN_MFMA_BCONV, and the plan without the flag stands for both."""
    if min(params.alpha, params.ell) < 4:
        return list(plans)
    keys = {p.key() for p in plans}
    twin = lambda k: (k[0], k[1], k[2], k[3] & ~PLAN_MFMA_BCONV, k[4])
    return [p for p in plans if not p.flags & PLAN_MFMA_BCONV or twin(p.key()) not in keys]


def prior_order(params, batch: int, plans, cache_bytes: int = MALL_BYTES):
    """Order plans by the footprint prior: the largest-parallelism plan whose
    footprint stays within half of the cache comes first (the paper's 2x
    rule), then the others by how far their footprint is from that target."""
    def key(p):
        per_pass = min(batch, p.batch_tile) if p.batch_tile else batch
        f = footprint_bytes(params.dnum, params.n, params.ell, p.dataflow if p.dataflow != STAGED else DPOB,
                            p.chunks, per_pass)
        fits = f * 2 <= cache_bytes
        launches = params.launch_count(batch, p)
        return (0 if fits else 1, launches if fits else f, p.log_r)
    return sorted(plans, key=key)


def _cache_key(params, batch: int) -> str:
    """Device, ROCm version and the shape of the computation: dnum, N, the
    Q limbs of the ciphertext (L, the level for a level handle) and the P
    limbs k (= alpha, the digit size). A level handle keeps its top level's k,
    so level 16 of (4, 2^16, 32) (k = 8, two digits) and a top-level
    (4, 2^16, 16) set (k = 4, four digits) are different entries."""
    arch = torch.cuda.get_device_properties(0).gcnArchName if torch.cuda.is_available() else "cpu"
    rocm = getattr(torch.version, "hip", None) or "none"
    return f"{arch}|rocm{rocm}|dnum{params.dnum}|logn{params.log_n}|L{params.ell}|k{params.k}|B{batch}"


SHIPPED_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "tuned_plans.json")


def shipped_cache() -> dict:
    """Winners of earlier tuning runs on this hardware, shipped with the
    package (same keys and entries as the tuning cache)."""
    return load_cache(SHIPPED_PATH)


def default_cache_path() -> str:
    return os.environ.get("KS_AUTOTUNE_CACHE", os.path.join(os.path.expanduser("~"), ".cache", "ks_autotune.json"))


def load_cache(path: str = None) -> dict:
    path = path or default_cache_path()
    try:
        with open(path) as f:
            return json.load(f)
    except (OSError, ValueError):
        return {}


def save_cache(cache: dict, path: str = None) -> None:
    path = path or default_cache_path()
    os.makedirs(os.path.dirname(path) or ".", exist_ok=True)
    tmp = path + ".tmp"
    with open(tmp, "w") as f:
        json.dump(cache, f, indent=1, sort_keys=True)
    os.replace(tmp, path)


def time_plan(params, d, evk, out, batch: int, plan, reps: int = 5, trials: int = 3, stream=None) -> float:
    """Median over trials of the mean time (ms) of `reps` back-to-back KeySwitch calls."""
    ws = params.workspace(batch, plan)
    params.keyswitch(d, evk, out, batch, ws, plan, stream=stream)
    ev = HipEvents(2)
    times = []
    for _ in range(trials):
        ev.record(0, stream)
        for _ in range(reps):
            params.keyswitch(d, evk, out, batch, ws, plan, stream=stream)
        ev.record(1, stream)
        torch.cuda.synchronize()
        times.append(ev.elapsed_ms(0, 1) / reps)
    return statistics.median(times)


def tune(params, d, evk, batch: int, plans=None, reps: int = 5, trials: int = 3, max_plans: int = None,
         cache: dict = None, verbose: bool = False, margin: float = 0.01):
    """Time the candidate plans on (d, evk) and return (best_plan, results).

    results is a list of {"plan", "ms", "ks_per_s", "bit_exact"} in the order
    tried. A plan counts only if its output equals the reference plan's (the
    default plan, itself checked against the oracle by the test suite)
    element for element, and replaces the best so far only if it is faster
    by more than `margin` (a fraction), so that timing noise does not pick a
    later plan of the prior order (for instance the two-stream variant of a
    plan) over an equally fast earlier one. With `cache`, the winner is
    stored under this device, ROCm version, parameter set and batch."""
    if plans is None:
        plans = prior_order(params, batch, distinct_plans(params, candidate_plans(params, batch)))
    if max_plans:
        plans = plans[:max_plans]
    out = torch.empty((batch, 2, params.ell, params.n), dtype=torch.int64, device=d.device)
    ref_plan = params.default_plan(batch)
    params.keyswitch(d, evk, out, batch, params.workspace(batch, ref_plan), ref_plan)
    torch.cuda.synchronize()
    ref = out.clone()
    results, best, best_ms = [], None, float("inf")
    for p in plans:
        out.fill_(0)
        ms = time_plan(params, d, evk, out, batch, p, reps, trials)
        exact = bool(torch.equal(out, ref))
        results.append({"plan": list(p.key()), "name": repr(p), "ms": ms,
                        "ks_per_s": batch / ms * 1e3, "bit_exact": exact})
        if verbose:
            print(f"  {p!r}: {ms:.4f} ms, {batch / ms * 1e3:.1f} KS/s, bit-exact={exact}", flush=True)
        if exact and ms < best_ms * (1.0 - margin):
            best, best_ms = p, ms
    if best is None:
        raise RuntimeError("no candidate plan reproduced the reference output")
    if cache is not None:
        cache[_cache_key(params, batch)] = {"plan": list(best.key()), "ms": best_ms,
                                             "name": repr(best)}
    return best, results


def cached_plan(params, batch: int, cache: dict):
    """The cached winner for this device and parameter set, or None."""
    e = cache.get(_cache_key(params, batch))
    if not e:
        return None
    df, chunks, log_r = e["plan"][:3]
    flags = e["plan"][3] if len(e["plan"]) > 3 else 0
    tile = e["plan"][4] if len(e["plan"]) > 4 else 0
    p = Plan(df, chunks, log_r, flags, tile)
    try:
        params.workspace_bytes(batch, p)
    except KsError:
        return None
    return p


def plan_for(params, batch: int, cache: dict):
    """The cached winner for this batch, else the winner cached for the same
    device and parameter set at the nearest other batch size, else None."""
    p = cached_plan(params, batch, cache)
    if p is not None:
        return p
    head = _cache_key(params, batch).rsplit("|B", 1)[0] + "|B"
    near = sorted((abs(int(k[len(head):]) - batch), k) for k in cache if k.startswith(head))
    for _, k in near:
        p = cached_plan(params, int(k[len(head):]), cache)
        if p is not None:
            return p
    return None


def describe(plan) -> str:
    return repr(plan)


# The paper's parameter grid (Evaluation section): N in 2^14..2^17,
# L in {10, 30, 50}, dnum in {2, 4, 6, 8}.
PAPER_GRID = {"log_n": (14, 15, 16, 17), "ell": (10, 30, 50), "dnum": (2, 4, 6, 8)}


def grid_map(batch: int = 1, chunk_range=(2, 4, 8), reps: int = 3, trials: int = 2, table: dict = None,
             grid=PAPER_GRID, log=print):
    """Tune every (dnum, N, L) of the grid on the current device (the
    per-parameter dataflow map of the paper's Fig. 4, measured here). Returns
    one row per set: the winning plan, its time, and the best time of each
    dataflow over the other knobs (NTT split, chunks, BConv variant, split)."""
    import numpy as np

    from . import KsParams
    from synth import ciphertext_batch, uniform_key

    rows = []
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).to("cuda")
    for log_n in grid["log_n"]:
        for ell in grid["ell"]:
            for dnum in grid["dnum"]:
                G = KsParams(dnum, log_n, ell)
                d = dev(ciphertext_batch(G.moduli[:ell], G.n, batch))
                evk = dev(uniform_key(G.moduli, G.n, G.ndig))
                plans = prior_order(G, batch, distinct_plans(G, candidate_plans(G, batch, chunk_range)))
                best, results = tune(G, d, evk, batch, plans=plans, reps=reps, trials=trials, cache=table)
                per_df = {}
                for r in results:
                    names = [DATAFLOW_NAMES[r["plan"][0]]]
                    if r["plan"][3] & PLAN_HOIST_FWD:  # also kept apart: DPOB with the hoisted forward pass
                        names.append(names[0] + "-hoist")
                    for name in names:
                        if r["bit_exact"] and (name not in per_df or r["ms"] < per_df[name]):
                            per_df[name] = r["ms"]
                best_ms = next(r["ms"] for r in results if r["plan"] == list(best.key()))
                row = {"dnum": dnum, "log_n": log_n, "L": ell, "batch": batch, "best": repr(best),
                       "best_ms": best_ms, "per_dataflow_ms": per_df, "plans": len(results),
                       "footprint_dpob_mb": footprint_bytes(dnum, G.n, ell, DPOB, 1, batch) / 1e6}
                rows.append(row)
                log(json.dumps(row))
                del G, d, evk
                torch.cuda.empty_cache()
    return rows


if __name__ == "__main__":
    import argparse
    import sys
    sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    ap = argparse.ArgumentParser(description="per-parameter dataflow map over the paper's grid")
    ap.add_argument("--batch", type=int, default=1)
    ap.add_argument("--save-tuned", default="", help="merge the winners into this JSON table")
    ap.add_argument("--log-n", default="", help="comma-separated subset of the grid's log N values")
    args = ap.parse_args()
    table = load_cache(args.save_tuned) if args.save_tuned else {}
    grid = dict(PAPER_GRID)
    if args.log_n:
        grid["log_n"] = tuple(int(v) for v in args.log_n.split(","))
    grid_map(args.batch, table=table, grid=grid, log=lambda s: print(s, flush=True))
    if args.save_tuned:
        save_cache(table, args.save_tuned)
