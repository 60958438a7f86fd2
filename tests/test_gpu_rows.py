"""The row kernels (frontiers of single-device candidates, uniform beta, no
variant) against the oracle on shapes that reach their edge cases: k_rows,
one row per lane, in every device-count class (4, 8 and 16 lanes, including
D = 1, 2, 3, 5 and 9), no prefix slots and the most prefix slots, more
completed parents than lanes in a group, instances whose frontier spans
several 128-stage chunks, a parameter set's horizon below the packed one, and
top-k above the one-lane ranking (the group ranks then); k_rows4, one row per
four lanes, for 17 to 64 devices (quads whose upper lanes hold no device,
the largest tables, several chunks, dense parents, top-k up to 64)."""

import dataclasses

import numpy as np
import pytest

from gpu_util import check_against_oracle, run_gpu
from oracle import oracle
from paper_2605_07238_amd import fate, synth

pytestmark = pytest.mark.gpu


def _rows_workload(seed, **kw):
    args = dict(B=3, n=40, H=3, max_shard=1, shard_frac=0.0, uniform_beta=True, p_edge=0.25)
    args.update(kw)
    return synth.make_random_small(seed, **args)


@pytest.mark.parametrize("seed,kw", [
    (1, dict(D=1, M=2, K=2)),
    (2, dict(D=2, M=3, K=0)),
    (3, dict(D=3, M=3, K=1)),
    (4, dict(D=4, M=3, K=4)),
    (5, dict(D=5, M=4, K=8)),
    (6, dict(D=8, M=6, K=32)),
    (7, dict(D=9, M=5, K=3)),
    (8, dict(D=16, M=12, K=16)),
    (9, dict(D=16, M=32, K=32)),
], ids=["d1", "d2-k0", "d3", "d4", "d5", "d8-k32", "d9", "d16", "d16-m32"])
def test_rows_random(seed, kw):
    w = _rows_workload(seed, **kw)
    print("[rows] random", seed, kw, flush=True)
    check_against_oracle(w, run_gpu(w, k=4), k=4)


def test_rows_dense_parents():
    """Up to five completed parents per stage on 4-lane groups."""
    w = _rows_workload(11, D=4, M=3, K=4, n=30, p_edge=0.7)
    print("[rows] dense parents", flush=True)
    check_against_oracle(w, run_gpu(w, k=4), k=4)


def test_rows_several_chunks():
    """Instances whose frontier holds more than 128 stages."""
    w = _rows_workload(12, B=2, n=700, D=16, M=6, K=4, p_edge=0.003)
    g = run_gpu(w, k=4)
    per_inst = np.bincount(np.searchsorted(w.stage_off, g["flat_v"], side="right") - 1, minlength=w.B)
    print("[rows] several chunks, frontier per instance", per_inst.tolist(), flush=True)
    assert per_inst.max() > 128
    check_against_oracle(w, g, k=4)


@pytest.mark.parametrize("H", [0, 1, 2])
def test_rows_horizon_below_packed(H):
    """The descendant lists are packed for H = 3; a parameter set with a
    smaller H takes the prefix of each list within its horizon."""
    w = _rows_workload(13, D=8, M=5, K=4, n=60, p_edge=0.2)
    print("[rows] H", H, "packed 3", flush=True)
    check_against_oracle(w, run_gpu(w, H=H, pack_H=3, k=4), H=H, k=4)


@pytest.mark.parametrize("k", [5, 16, 64])
def test_rows_topk_above_lane_ranking(k):
    w = _rows_workload(14, D=16, M=6, K=4, n=50)
    print("[rows] k", k, flush=True)
    check_against_oracle(w, run_gpu(w, k=k), k=k)


@pytest.mark.parametrize("seed,kw", [
    (21, dict(D=17, M=5, K=4)),
    (22, dict(D=24, M=8, K=2)),
    (23, dict(D=33, M=12, K=8)),
    (24, dict(D=48, M=20, K=16)),
    (25, dict(D=64, M=32, K=16)),
    (26, dict(D=64, M=40, K=0)),
    (27, dict(D=50, M=64, K=4)),
], ids=["d17", "d24", "d33", "d48", "d64", "d64-k0", "d50-m64"])
def test_rows4_random(seed, kw):
    w = _rows_workload(seed, **kw)
    print("[rows4] random", seed, kw, flush=True)
    check_against_oracle(w, run_gpu(w, k=4), k=4)


def test_rows4_dense_parents_and_chunks():
    """Up to five completed parents per stage, and instances of more than 128
    frontier stages, on 64 devices."""
    w = _rows_workload(31, B=2, n=600, D=64, M=16, K=8, p_edge=0.004)
    g = run_gpu(w, k=4)
    per_inst = np.bincount(np.searchsorted(w.stage_off, g["flat_v"], side="right") - 1, minlength=w.B)
    print("[rows4] several chunks, frontier per instance", per_inst.tolist(), flush=True)
    assert per_inst.max() > 128
    check_against_oracle(w, g, k=4)
    w = _rows_workload(32, D=40, M=6, K=4, n=30, p_edge=0.7)
    print("[rows4] dense parents", flush=True)
    check_against_oracle(w, run_gpu(w, k=4), k=4)


@pytest.mark.parametrize("H", [0, 2])
def test_rows4_horizon_below_packed(H):
    w = _rows_workload(33, D=36, M=5, K=4, n=60, p_edge=0.2)
    print("[rows4] H", H, "packed 3", flush=True)
    check_against_oracle(w, run_gpu(w, H=H, pack_H=3, k=4), H=H, k=4)


@pytest.mark.parametrize("k", [1, 16, 64])
def test_rows4_topk(k):
    w = _rows_workload(34, D=64, M=6, K=4, n=50)
    print("[rows4] k", k, flush=True)
    check_against_oracle(w, run_gpu(w, k=k), k=k)


@pytest.mark.parametrize("D,K,M", [(33, 32, 26), (64, 17, 26), (64, 32, 26), (64, 32, 27), (64, 16, 53), (64, 16, 54)])
def test_rows4_most_models(D, K, M):
    """Clusters whose tables just fit k_rows4, and the first that go to the general kernel."""
    w = _rows_workload(90 + M, D=D, M=M, K=K, n=60)
    print("[rows4] most models", D, K, M, flush=True)
    check_against_oracle(w, run_gpu(w, k=4), k=4)


@pytest.mark.parametrize("D,M", [(4, 3), (7, 5), (16, 12), (24, 6), (64, 9)])
def test_rows_variants(D, M):
    """The same-model weight and windows switched off on frontiers without
    windows: the row kernel for 9 to 16 devices, else the general kernel."""
    w = _rows_workload(60 + D, D=D, M=M, K=4, n=60, p_edge=0.08)
    for p in (dict(lam_m=0.3), dict(lam_m=2.0, lam_s=0.5, no_windows=1), dict(no_windows=1)):
        print("[rows] variants", D, p, flush=True)
        check_against_oracle(w, run_gpu(w, k=4, params=p), k=4, params=p)


@pytest.mark.parametrize("D", [1, 3, 4, 6, 8, 13, 16])
@pytest.mark.parametrize("k", [1, 3, 4])
def test_lane_topk(D, k):
    """fate_topk on frontiers of exactly D candidates a stage, aligned or not,
    against the rule (score descending, index ascending), with ties, padding
    and unaligned scores, outputs and strides."""
    import torch
    from paper_2605_07238_amd import parity
    w = _rows_workload(80 + D, B=5, D=D, M=3, K=2, n=300, p_edge=0.005)
    print("[rows] lane top-k", D, k, flush=True)
    pk = fate.fate_pack_dags(w)
    st = fate.fate_pack_state(pk, w)
    F, C = st.n_frontier, st.n_cand
    assert C == F * D and F > 256
    rng = np.random.default_rng(D)
    for shift in (0, 1):
        x = rng.integers(-3, 4, (3, C + 5)).astype(np.float32) * np.float32(0.5)
        x[rng.random(x.shape) < 0.2] = -np.inf
        buf = torch.zeros(x.size + 1, device="cuda")
        scores = buf[shift:shift + x.size].view(x.shape)
        scores.copy_(torch.from_numpy(x))
        out_i = torch.zeros(3 * F * k + 1, dtype=torch.int32, device="cuda")[shift:shift + 3 * F * k].view(3, F, k)
        out_v = torch.zeros(3 * F * k + 1, device="cuda")[shift:shift + 3 * F * k].view(3, F, k)
        fate.fate_topk_sweep(st, scores, k, idx=out_i, val=out_v)
        off = np.arange(F + 1, dtype=np.int64) * D
        for p in range(3):
            want = parity.topk_of_scores(x[p, :C], off, k)
            assert np.array_equal(out_i[p].cpu().numpy(), want)
            vals = np.where(want >= 0, x[p][np.minimum(off[:-1, None] + np.maximum(want, 0), C - 1)], -np.inf)
            assert np.array_equal(out_v[p].cpu().numpy(), vals.astype(np.float32))


def _equal_rows(D, roots, kids, x):
    """`roots` frontier stages, each parent of all `kids` horizon stages, every
    run time x on every device and nothing else in a cost: a row costs x."""
    n = roots + kids
    par_off = np.concatenate([np.zeros(roots + 1), roots * np.arange(1, kids + 1)]).astype(np.int64)
    w = synth.make_random_small(3, B=1, n=n, D=D, M=2, K=1, H=1, max_shard=1, shard_frac=0.0, p_edge=0.0)
    zero = np.zeros(n, np.float32)
    w = dataclasses.replace(
        w, par_off=par_off, par_idx=np.tile(np.arange(roots, dtype=np.int32), kids), model=np.zeros(n, np.int32),
        elig=np.full(n, (1 << D) - 1, np.uint64), status=np.zeros(n, np.uint8), holders=np.zeros(n, np.uint64),
        prefix_hash=np.zeros(n, np.uint64), prefix_tokens=zero, out_bytes=zero, exec=np.full((2, D), x, np.float32),
        weight_bytes=np.full(2, 1, np.int64), cap_bytes=np.full(D, 4, np.int64), resident=np.ones((1, D), np.uint64),
        tau_free=np.zeros((1, D), np.float32), t_now=np.zeros(1, np.float32))
    w.params.update(gamma=1.0, no_windows=1, lam_c=0.0)
    return w


@pytest.mark.parametrize("D,roots,kids", [(3, 128, 1000), (8, 128, 1000), (12, 128, 1000), (16, 128, 1000), (24, 128, 1000),
                                          (64, 128, 1000), (16, 1, 4080), (16, 1, 4081), (16, 3, 2048)])
def test_windows_off_keeps_short_sums(D, roots, kids):
    """A set with windows switched off is summed as the general kernel sums:
    every row in fp64, or sixteen rows in fp32 for 9 to 16 devices.  x loses
    just under half a last place (2^-16 of 2^-15) each time it is added to an
    fp32 sum between 256 and 512, so one sum of all rows is off by 6e-6; x is
    exact in sums below 16, and a row's value and the score are rounded a
    few times each (at most eight), each by 2^-24."""
    x = 1.0 + 2.0 ** -16 - 2.0 ** -19
    w = _equal_rows(D, roots, kids, x)
    print("[rows] windows off, equal rows", D, roots, kids, flush=True)
    got = run_gpu(w, k=4)
    want = -np.float64(x) * (1 + kids)
    bound = (8 + (16 if 8 < D <= 16 else 0)) * 2.0 ** -24
    assert np.abs(got["psi"] / want - 1.0).max() <= bound


@pytest.mark.parametrize("D", [9, 12, 16])
def test_windows_off_over_many_rows(D):
    """Chunks cut where their stages have more rows than sixteen to a task."""
    w = _rows_workload(70 + D, B=3, D=D, M=5, K=4, n=500, p_edge=0.03)
    p = dict(no_windows=1)
    print("[rows] windows off, many rows", D, flush=True)
    for k in (4, 7):
        check_against_oracle(w, run_gpu(w, k=k, params=p), k=k, params=p)
    # through the sweep, beside a plain set and one with the weight: each set as alone
    import torch
    pk = fate.fate_pack_dags(w)
    st = fate.fate_pack_state(pk, w)
    sets = [fate.make_params(w, **q) for q in (dict(), p, dict(lam_m=0.5), dict(no_windows=1, lam_m=0.5))]
    sweep = fate.fate_score_sweep(pk, st, sets)[:, :st.n_cand].cpu().numpy()
    for i, q in enumerate(sets):
        one = fate.fate_score_frontier(pk, st, q)[:st.n_cand].cpu().numpy()
        assert np.array_equal(one.view(np.uint32), sweep[i].view(np.uint32)), i


@pytest.mark.parametrize("D", [4, 8, 20, 64])
@pytest.mark.parametrize("lam_m", [1e3, 1e5])
def test_same_model_weight_leaves_other_terms_exact(D, lam_m):
    """A frontier stage whose Load evicts its child's model on the child's one
    device: placed there, no term of its score holds the same-model weight, and
    the score has the accuracy of its own terms (at most eight roundings of
    2^-24).  (For 9 to 16 devices the cost tables hold a switch term and its
    difference, in which the weight cancels to its own last place.)"""
    import builders
    inst = dict(parents=[[], [0]], model=[0, 1], elig=[(1 << D) - 1, 1], out_bytes=[0.0, 0.0], status=[0, 0], holders=[0, 0],
                resident=[2] + [1] * (D - 1), tau_free=[0.0] * D, t_now=0.0)
    spec = dict(D=D, M=2, K=1, exec=[[1.1] * D, [1.3] * D], switch_s=[[0.7] * D, [0.9] * D], weight_gb=[10, 10], cap_gb=[15] * D,
                beta=[[0.0 if i == j else 1e-10 for j in range(D)] for i in range(D)], max_shard=1, instances=[inst])
    w = builders.from_spec(spec, H=1)
    p = dict(lam_m=lam_m, lam_s=1.0, gamma=0.9)
    print("[rows] same-model weight", D, lam_m, flush=True)
    got = run_gpu(w, k=2, params=p)
    want = oracle.score(w, params=p)["psi"]
    assert abs(want[0]) < 5.0 and abs(got["psi"][0] / want[0] - 1.0) <= 8 * 2.0 ** -24
    check_against_oracle(w, got, k=2, params=p)
