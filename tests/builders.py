"""Build small hand-specified workloads for the pinned oracle tests.

Input construction only: a JSON-like dict lists the cluster tables and, per
instance, the parent lists, stage attributes and state arrays.  Nothing here
computes a score.
"""

from __future__ import annotations

import numpy as np

from paper_2605_07238_amd import synth


def from_spec(spec: dict, H: int = 1, params: dict | None = None) -> synth.Workload:
    D, M, K = int(spec["D"]), int(spec["M"]), int(spec.get("K", 1))
    insts = []
    for it in spec["instances"]:
        parents = it["parents"]
        n = len(parents)
        cache = np.array(it.get("prefix_cache", [[0] * K for _ in range(D)]), dtype=np.uint64).reshape(D, K)
        insts.append(dict(
            n=n,
            par_lens=np.array([len(p) for p in parents], np.int64),
            par_flat=np.array([p for ps in parents for p in ps], np.int32),
            model=np.array(it["model"], np.int32),
            elig=np.array([int(e) for e in it["elig"]], np.uint64),
            shard=np.array(it.get("shard_max", [1] * n), np.int32),
            hash=np.array([int(h) for h in it.get("prefix_hash", [0] * n)], np.uint64),
            toks=np.array(it.get("prefix_tokens", [0.0] * n), np.float32),
            sigma=np.array(it["out_bytes"], np.float32),
            resident=np.array([int(r) for r in it["resident"]], np.uint64),
            cache=cache,
            holders=np.array([int(h) for h in it["holders"]], np.uint64),
            status=np.array(it["status"], np.uint8),
            tau=np.array(it["tau_free"], np.float32),
            t_now=np.float32(it["t_now"]),
        ))
    cluster = (
        np.array(spec["exec"], np.float32).reshape(M, D),
        np.array(spec["switch_s"], np.float32).reshape(M, D),
        np.array([int(round(x * synth.GB)) for x in spec["weight_gb"]], np.int64),
        np.array([int(round(x * synth.GB)) for x in spec["cap_gb"]], np.int64),
        np.array(spec["beta"], np.float32).reshape(D, D),
    )
    rc = dict(D=D, M=M, H=H)
    w = synth._assemble(spec.get("title", "spec"), rc, cluster, insts, K, int(spec.get("max_shard", 4)))
    if params:
        w.params.update(params)
    return w


def random_batch(sizes, seed: int, D: int = 5, M: int = 3, K: int = 2, fan: int = 3) -> synth.Workload:
    """Instances of the given numbers of stages (0 among them), each stage with
    up to `fan` parents among the 300 before it; a random prefix of up to half
    of an instance is completed, and some of its frontier is running."""
    rng = np.random.default_rng(seed)
    n = np.array(sizes)
    B = len(n)
    stage_off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    N = int(stage_off[-1])
    base = np.repeat(stage_off[:-1], n)
    local = np.arange(N) - base
    far = np.unique(np.geomspace(1, 300, fan + 1).astype(int))  # a parent from each span of distances
    back = np.stack([rng.integers(lo, hi, N) for lo, hi in zip(far[:-1], far[1:])][::-1], 1)
    has = (back <= local[:, None]) & (rng.random(back.shape) < 0.6)
    par, npar = (local[:, None] - back)[has].astype(np.int32), has.sum(1)
    child = np.repeat(np.arange(N), npar)
    done = local < np.repeat(rng.integers(0, n // 2 + 1), n)
    status = done.astype(np.uint8)
    left = np.bincount(child, weights=~done[par + base[child]], minlength=N) if len(par) else np.zeros(N)
    status[~done & (left == 0) & (rng.random(N) < 0.3)] = 2
    return synth.Workload(
        name="random", D=D, M=M, K=K, H=0, max_shard=3, stage_off=stage_off,
        par_off=np.concatenate([[0], np.cumsum(npar)]).astype(np.int64), par_idx=par,
        model=rng.integers(0, M, N).astype(np.int32), elig=np.full(N, (1 << D) - 1, np.uint64),
        shard_max=rng.integers(1, 4, N).astype(np.int32), prefix_hash=rng.integers(0, 5, N).astype(np.uint64),
        prefix_tokens=np.ones(N, np.float32), out_bytes=rng.integers(1, 1000, N).astype(np.float32),
        exec=np.ones((M, D), np.float32), switch_s=np.ones((M, D), np.float32), weight_bytes=np.full(M, 10, np.int64),
        cap_bytes=np.full(D, 25, np.int64), beta=np.full((D, D), 1e-9, np.float32),
        resident=rng.integers(0, 8, (B, D)).astype(np.uint64), prefix_cache=rng.integers(0, 5, (B, D, K)).astype(np.uint64),
        holders=np.where(done, rng.integers(1, 1 << D, N), 0).astype(np.uint64), status=status,
        tau_free=rng.random((B, D)).astype(np.float32), t_now=rng.random(B).astype(np.float32))
