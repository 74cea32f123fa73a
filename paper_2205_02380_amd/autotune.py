"""Autotuner: pick patch size, ghost width, kernel schedule, tile shape and field
placement for a grid.

Every candidate (patch M, ghost g, schedule, tile shape -- the launch-shape variant of
the SLAB and PLAIN passes: x3-slabs per slab block and lines per pencil block --, in
place or out of place through a second field) that has compiled kernels is timed on the
workload's own field (HIP events around its calls) and its result after the
tuning steps is compared with the most accurate candidate (the largest ghost width,
then the largest patch): the PMBC truncation error shrinks like |sqrt3 - 2|^g, so a
smaller g is faster to compute but drifts from the untruncated spline.  The winner is
the fastest candidate whose result stays within `tol` (relative to max|f|) of that
reference; candidates within `margin` (relative) of the fastest time count as equally
fast (timing noise on a few steps is about 1 %), and among them the most accurate one
wins (in place is listed before out of place, so the second field is taken only when
it is faster by more than the margin).  Candidates are timed as the run they are tuned for steps: with the
per-step FP64 diagnostics on when it records them (`reduce_each_step`), since the
reduction epilogue changes a pass's register use, and in calls of as many steps as it
makes (`steps_per_call`), since calls of several steps without diagnostics run other kernels.
Of candidates that then launch the same kernels on the same fields one is timed.
Results can be cached in a JSON file keyed by the grid, dt and these two.

Host logic only: every step runs through the C ABI.  Parity of each compiled (M, g)
with the FP64 oracle is the test suite's job, not the tuner's.
"""
from __future__ import annotations

import argparse
import json
import os
from typing import Dict, List, Optional, Sequence

from . import chasm, inputs


def candidates(grid: inputs.Grid, dt: float, patches: Sequence[int], ghosts: Sequence[int],
               schedules: Sequence[str], placements: Sequence[bool] = (False, True),
               tiles: Sequence[int] = chasm.TILES) -> List[dict]:
    """Every (patch, ghost, schedule, tile, placement) the library accepts for the grid
    (its own descriptor validation decides; tile variants exist for some shapes only)."""
    out = []
    for M in patches:
        for g in ghosts:
            for sc in schedules:
                for tile in tiles:
                    d = chasm.make_desc(grid, M, g, dt, schedule=sc, flags=chasm.CHASM_FLAG_TILE(tile))
                    try:
                        chasm.chasm_advect_workspace_bytes(d)
                    except chasm.ChasmError:
                        continue
                    for oop in placements:
                        out.append({"patch": M, "ghost": g, "schedule": sc, "tile": tile, "out_of_place": oop})
    return out


def distinct(cands: List[dict], reduce_each_step: bool, steps_per_call: int) -> List[dict]:
    """The candidates without those that launch what another one does: without per-step
    diagnostics CUBE handles step in place, and SLAB calls of several steps have one launch
    shape (up to 64 steps at a time; a single step left over has the variant's own)."""
    several = steps_per_call > 1 and steps_per_call % 64 != 1

    def launches(c):
        own = reduce_each_step or c["schedule"] == "plain"
        return (c["patch"], c["ghost"], c["schedule"],
                c["tile"] if own or not several else 0,
                c["out_of_place"] if own or c["schedule"] == "slab" else False)
    out: Dict[tuple, dict] = {}
    for c in sorted(cands, key=accuracy_order):
        out.setdefault(launches(c), c)
    return list(out.values())


def accuracy_order(c: dict):
    """Most accurate first: largest ghost width, then largest patch; in place before out
    of place (equal results, less memory)."""
    return (-c["ghost"], -c["patch"], c["schedule"], c["out_of_place"], c.get("tile", 0))


def choose(cands: List[dict], margin: float = 0.01) -> dict:
    """Among the candidates within tolerance (`ok`), those within `margin` of the fastest
    time count as equally fast; of these the one with the smallest deviation wins, ties
    going to the earliest in accuracy order."""
    ok = sorted((c for c in cands if c["ok"]), key=accuracy_order)
    if not ok:
        raise ValueError("no candidate within tolerance")
    fastest = min(c["ms_per_step"] for c in ok)
    return min((c for c in ok if c["ms_per_step"] <= fastest * (1.0 + margin)), key=lambda c: c["deviation"])


def tune(grid: inputs.Grid, dt: float, packets: inputs.Packets, patches=(8, 12, 16), ghosts=(4, 6, 8),
         schedules=("cube", "slab", "plain"), placements=(False, True), tiles=chasm.TILES, steps: int = 5,
         warmup: int = 2, tol: float = 1e-5, margin: float = 0.01, device: str = "cuda:0", log=None,
         reduce_each_step: bool = False, steps_per_call: int = 0) -> dict:
    """steps_per_call: steps of each call of the run that is tuned for (0: all in one call)."""
    import torch
    dev = torch.device(device)
    stream = torch.cuda.current_stream(dev)
    per_call = steps_per_call or steps
    cands = distinct(candidates(grid, dt, patches, ghosts, schedules, placements, tiles), reduce_each_step, per_call)
    if not cands:
        raise ValueError("no compiled kernels for this grid")
    f0 = torch.empty(grid.shape(), dtype=torch.float32, device=dev)
    coef, gx, gk = inputs.packet_factors(grid, packets)
    inputs.fill_separable(f0, coef, gx, gk)
    work = torch.empty_like(f0)
    # most accurate first: largest ghost width, then largest patch
    cands.sort(key=accuracy_order)
    ref = None
    scale = None
    for c in cands:
        work.copy_(f0)
        adv = chasm.Advect(work, grid, c["patch"], c["ghost"], dt, schedule=c["schedule"], graph=True,
                           stream=stream, out_of_place=c["out_of_place"], tile=c["tile"],
                           reduce_each_step=reduce_each_step, history_cap=warmup + steps)
        def run(n):
            for at in range(0, n, per_call):
                adv.step(min(per_call, n - at))
        run(warmup)
        torch.cuda.synchronize()
        work.copy_(f0)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record(stream)
        run(steps)
        ev[1].record(stream)
        torch.cuda.synchronize()
        adv.close()
        c["ms_per_step"] = ev[0].elapsed_time(ev[1]) / steps
        c["point_updates_per_s"] = grid.points / (c["ms_per_step"] * 1e-3)
        if ref is None:
            ref = work.clone()
            scale = float(ref.abs().max())
            c["deviation"] = 0.0
        else:
            c["deviation"] = float((work - ref).abs().max()) / scale
        c["ok"] = c["deviation"] <= tol
        if log:
            log(f"  M={c['patch']:2d} g={c['ghost']} {c['schedule']:5s} t{c['tile']} "
                f"{'oop' if c['out_of_place'] else 'inp'} "
                f"{c['ms_per_step']:8.3f} ms/step "
                f"dev={c['deviation']:.2e}{'' if c['ok'] else '  (over tol)'}")
    del work, f0, ref
    torch.cuda.empty_cache()
    best = choose(cands, margin)
    return {"grid": {"nx": list(grid.nx), "nk": list(grid.nk)}, "dt": dt, "tol": tol, "steps": steps,
            "reduce_each_step": reduce_each_step, "steps_per_call": steps_per_call, "candidates": cands, "best": best}


def cache_key(grid: inputs.Grid, dt: float, reduce_each_step: bool = False, steps_per_call: int = 0) -> str:
    return (f"nx{grid.nx[0]}_nk{grid.nk[0]}x{grid.nk[1]}x{grid.nk[2]}_dt{dt:g}" + ("_red" if reduce_each_step else "")
            + (f"_call{steps_per_call}" if steps_per_call else ""))


def load_cache(path: str) -> Dict[str, dict]:
    if path and os.path.exists(path):
        with open(path) as fh:
            return json.load(fh)
    return {}


def lookup(path: str, grid: inputs.Grid, dt: float, reduce_each_step: bool = False,
           steps_per_call: int = 0) -> Optional[dict]:
    return load_cache(path).get(cache_key(grid, dt, reduce_each_step, steps_per_call))


def store(path: str, grid: inputs.Grid, dt: float, result: dict) -> None:
    c = load_cache(path)
    c[cache_key(grid, dt, bool(result.get("reduce_each_step", False)), result.get("steps_per_call", 0))] = result
    with open(path, "w") as fh:
        json.dump(c, fh, indent=1)


def main():
    ap = argparse.ArgumentParser(description="autotune patch / ghost / schedule for a workload")
    ap.add_argument("--workload", default="C3")
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--tol", type=float, default=1e-5)
    ap.add_argument("--cache", default="")
    ap.add_argument("--reduce-each-step", action="store_true", help="time with the per-step FP64 diagnostics")
    ap.add_argument("--steps-per-call", type=int, default=0, help="steps of each call (0: all of them in one)")
    args = ap.parse_args()
    w = inputs.workload(args.workload)
    res = tune(w.grid, w.dt, w.packets, steps=args.steps, tol=args.tol, log=print,
               reduce_each_step=args.reduce_each_step, steps_per_call=args.steps_per_call)
    print(json.dumps(res["best"]))
    if args.cache:
        store(args.cache, w.grid, w.dt, res)


if __name__ == "__main__":
    main()
