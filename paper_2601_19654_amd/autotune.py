"""Search of the pair kernels' tiles and algorithms, cached per (GPU arch, mode, size class).

For a given batch of systems it times, with HIP events on the context's stream
(nb_time_kernel), the whole force evaluation (force kernel plus the sum of its split
partials) over its candidates, and then whole steps: of the force candidates near the
fastest, of the encounter checks and of the step launches.  A check alone says little
about a step: the sorted check's small kernels run in the gaps of the force beside them,
the direct check's matrix products take their time from it.  The library's automatic
choice (0) is a candidate of both, and is taken unless another is faster by more than
TIE.  The choices are stored in ``tuning.json`` (with every candidate's time) under
``<arch>/<mode>/n<max system size, next power of two>/s<systems, next power of two>``,
and the chosen fields in ``tuning.tsv``, the table the library itself reads
(``nb_params.autotune_path``) whenever the caller leaves the tile fields at 0.

    python -m paper_2601_19654_amd.autotune --workloads c1,c2,c3,c4,c5
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

PKG = os.path.dirname(os.path.abspath(__file__))
CACHE = os.path.join(PKG, "tuning.json")

FORCE_R = (1, 2, 4)
FORCE_J = (256, 512, 1024, 2048, 4096)
FORCE_G = (1, 2, 4)          # super-tile widths of the symmetric force
ENC_J = 1024                 # most sources per item of the direct check (the library halves it)
TIE = 0.04                   # an automatic choice is kept unless another is faster by more
STEP_REPEATS, STEP_REPS = 5, 32   # best of five timings of 32 steps
NEAR, NEAR_MOST = 1.25, 8    # force candidates whose steps are timed: within NEAR of the fastest, at most 8


def _pow2(n: int) -> int:
    p = 1
    while p < n:
        p <<= 1
    return p


def arch() -> str:
    import torch
    name = torch.cuda.get_device_properties(0).gcnArchName
    return name.split(":")[0]


def key(mode: str, off, arch_name: str | None = None, nbig=None) -> str:
    """Size class: largest system and number of systems (next powers of two),
    plus the largest big-body count when some bodies are small."""
    sizes = np.diff(np.asarray(off))
    k = f"{arch_name or arch()}/{mode}/n{_pow2(int(sizes.max()))}/s{_pow2(len(sizes))}"
    if nbig is not None and np.any(np.asarray(nbig) < sizes):
        k += f"/b{_pow2(int(np.max(nbig)))}"
    return k


TABLE = os.path.join(PKG, "tuning.tsv")
TABLE_FIELDS = ("force_algo", "force_r", "force_jchunk", "enc_algo", "enc_jchunk", "step_algo", "force_g")


def write_table(cache: dict, path: str = TABLE) -> None:
    """The table the library reads (nb_params.autotune_path): one line per size
    class, the key then the seven chosen fields (force_g 0: the automatic width)."""
    lines = ["# key " + " ".join(TABLE_FIELDS) + "  (written by autotune.py from tuning.json)"]
    for k in sorted(cache):
        e = cache[k]
        lines.append(k + " " + " ".join(str(int(e.get(f, 0))) for f in TABLE_FIELDS))
    with open(path, "w") as f:
        f.write("\n".join(lines) + "\n")


def load_cache() -> dict:
    if os.path.exists(CACHE):
        with open(CACHE) as f:
            return json.load(f)
    return {}


def _mode_id(mode):
    return 1 if mode == "fp32c" else 0


def tune(w, mode: str, reps: int = 10, verbose: bool = True) -> dict:
    """Time every candidate on workload w; returns the best entry (not saved)."""
    from . import nb
    res_force, res_enc = {}, {}
    all_big = w.nbig is None or np.all(np.asarray(w.nbig) == np.diff(w.off))
    # 4: the symmetric force over the radial order (FP32C only)
    for fa in (((1, 2, 4) if mode == "fp32c" else (1, 2)) if all_big else (1,)):
        for r in FORCE_R:
            # the symmetric tile pairs have no source-chunk parameter, but a
            # super-tile width (tiles per workgroup)
            for j, g in ([(j, 0) for j in FORCE_J] if fa == 1 else [(1024, g) for g in FORCE_G]):
                if j > max(256, _pow2(int(np.diff(w.off).max()))) * 2:
                    continue
                p = nb.default_params(G=w.G, mode=_mode_id(mode), drag=int(w.drag), force_r=r, force_jchunk=j,
                                      force_algo=fa, force_g=g)
                c = nb.Context(w.off, p, enc_cap=1 << 16, device="cuda:0", tuned=False, nbig=w.nbig)
                c.upload(w.m0, w.m, w.x, w.v)
                # ranked by the whole force evaluation: more source chunks or
                # narrower super-tiles mean more split partials for the finalize
                ms = c.time_kernel(nb.NB_K_FORCE_EVAL, reps=reps)
                res_force[(fa, r, j, g)] = ms
                if verbose:
                    print(f"[autotune] {mode} force evaluation algo={fa} r={r} j={j} g={g}: {ms:.4f} ms",
                          file=sys.stderr, flush=True)
                c.close()
    sizes = np.diff(w.off)
    nbig = sizes if w.nbig is None else np.asarray(w.nbig)

    def step_ms(fa_, r_, j_, g_, ea_, sa_):
        p = nb.default_params(G=w.G, mode=_mode_id(mode), drag=int(w.drag), force_r=r_, force_jchunk=j_,
                              force_algo=fa_, force_g=g_, enc_jchunk=ENC_J, enc_algo=ea_, step_algo=sa_)
        c = nb.Context(w.off, p, enc_cap=1 << 18, device="cuda:0", tuned=False, nbig=w.nbig)
        c.upload(w.m0, w.m, w.x, w.v)
        # (the first runs capture their graphs, and raise the clocks of an idle GPU)
        c.step(w.dt, STEP_REPS, allow=(nb.NB_E_CAPACITY, nb.NB_E_KEPLER))
        times = [c.time_kernel(nb.NB_K_STEP, reps=STEP_REPS, dt=w.dt) for _ in range(STEP_REPEATS)]
        c.close()
        if verbose:
            print(f"[autotune] {mode} step, force algo={fa_} r={r_} j={j_} g={g_}, check {ea_}, launch {sa_}: "
                  f"{min(times):.4f} ms", file=sys.stderr, flush=True)
        return min(times)

    def best(times):
        """The fastest candidate, the automatic one (0) on a tie."""
        k = min(times, key=times.get)
        return 0 if 0 in times and times[0] <= (1.0 + TIE) * times[k] else k

    # the force candidates near the fastest, by whole steps of one launch per phase with
    # the automatic check (the super-tile width trades force-kernel time for partial
    # traffic, which the check beside the force shares)
    fms = min(res_force.values())
    near = sorted((k for k in res_force if res_force[k] <= NEAR * fms), key=res_force.get)[:NEAR_MOST]
    res_near = {k: step_ms(*k, 0, 1) for k in near}
    force = min(res_near, key=res_near.get)
    # the encounter checks: automatic, direct, sorted, and (FP32C, every body big, the
    # symmetric force) inside the force pass; and the check alone, for the record
    direct = 3 if np.any(nbig < sizes) and int(nbig.max()) <= 256 else 1
    checks = (0, direct, 2) + ((4,) if mode == "fp32c" and all_big and force[0] == 2 else ())
    res_enc = {ea: step_ms(*force, ea, 1) for ea in checks}
    ea = best(res_enc)
    res_alone = {}
    for a in (direct, 2):
        p = nb.default_params(G=w.G, mode=_mode_id(mode), drag=int(w.drag), enc_jchunk=ENC_J, enc_algo=a)
        c = nb.Context(w.off, p, enc_cap=1 << 18, device="cuda:0", tuned=False, nbig=w.nbig)
        c.upload(w.m0, w.m, w.x, w.v)
        c.drift(w.dt, allow_fail=True)
        res_alone[a] = c.time_kernel(nb.NB_K_ENCOUNTER, reps=reps)
        c.close()
    # the step launches: automatic, per phase, persistent
    persistent = mode == "fp64" and int(sizes.max()) <= 8192
    res_step = {sa: step_ms(*force, ea, sa) for sa in ((0, 1, 2) if persistent else (0, 1))}
    sa = best(res_step)
    name = "a{}_r{}_j{}_g{}".format
    fa, r, j, g = force
    return {"force_algo": fa, "force_r": r, "force_jchunk": j, "force_g": g, "enc_jchunk": ENC_J, "enc_algo": ea,
            "step_algo": sa, "step_ms": round(res_step[sa], 5), "force_ms": round(res_force[force], 5),
            "workload": w.name, "tuned_at": time.strftime("%Y-%m-%d"),
            "force_candidates": {name(*k): round(v, 5) for k, v in res_force.items()},
            "force_candidates_steps": {name(*k): round(v, 5) for k, v in res_near.items()},
            "encounter_candidates_steps": {str(k): round(v, 5) for k, v in res_enc.items()},
            "encounter_alone": {str(k): round(v, 5) for k, v in res_alone.items()},
            "step_candidates": {str(k): round(v, 5) for k, v in res_step.items()}}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--workloads", default="c1,c2,c3,c4,c5,bigsmall")
    ap.add_argument("--modes", default="fp64,fp32c")
    ap.add_argument("--reps", type=int, default=10)
    ap.add_argument("--out", default=CACHE)
    args = ap.parse_args()
    sys.path.insert(0, os.path.dirname(PKG))
    import workloads
    cache = load_cache()
    a = arch()
    for name in args.workloads.split(","):
        w = workloads.by_name(name)
        for mode in args.modes.split(","):
            best = tune(w, mode, reps=args.reps)
            k = key(mode, w.off, a, w.nbig)
            cache[k] = best
            print(f"[autotune] {k} -> force_algo={best['force_algo']} r={best['force_r']} j={best['force_jchunk']} "
                  f"enc_algo={best['enc_algo']} enc_j={best['enc_jchunk']} step_algo={best['step_algo']} "
                  f"(force {best['force_ms']:.4f}, step {best['step_ms']:.4f} ms)",
                  file=sys.stderr, flush=True)
            with open(args.out, "w") as f:
                json.dump(cache, f, indent=1, sort_keys=True)
            write_table(cache, os.path.join(os.path.dirname(os.path.abspath(args.out)), "tuning.tsv"))


if __name__ == "__main__":
    main()
