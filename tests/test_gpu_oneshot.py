"""The general scoring kernel on slices with few frontier stages, whose rows
are dealt to all lane groups (one shot), against the oracle: every lane-group
width, uniform and non-uniform transfer coefficients (the transfer table of at
most 32 devices, and past it), windows, workgroups of both sizes (by the number
of instances), frontiers just below and above the number of groups, free
outputs (nothing to move), and plain, planning-state and sweep calls writing
the same bits."""

import numpy as np
import pytest

from gpu_util import check_against_oracle, run_gpu
from paper_2605_07238_amd import fate, synth

pytestmark = pytest.mark.gpu


def _wide_roots(roots, D, seed, **kw):
    """Instances whose frontier is about `roots` stages, with rows below them."""
    return synth.make_random_small(seed, n=roots + 24, D=D, M=5, K=3, H=3, p_edge=1.5 / (roots + 24), shard_frac=0.5,
                                   max_shard=4, **kw)


@pytest.mark.parametrize("D", [3, 4, 5, 8, 9, 16, 17, 24, 32, 33, 64])
@pytest.mark.parametrize("uniform", [True, False], ids=["uniform", "tiered"])
def test_widths(D, uniform):
    w = synth.make_random_small(40 + D, B=3, n=40, D=D, M=6, K=4, H=3, shard_frac=0.5, max_shard=4, p_edge=0.08,
                                uniform_beta=uniform)
    print("[oneshot] D=%d uniform=%d" % (D, uniform), flush=True)
    check_against_oracle(w, run_gpu(w, k=5), k=5)
    p = dict(topo_levels=1, mean_levels=1, lam_m=0.25)
    w.params.update(p)
    check_against_oracle(w, run_gpu(w, k=3, params=p), k=3, params=p)


@pytest.mark.parametrize("roots,D", [(10, 16), (22, 16), (40, 16), (12, 24), (26, 24), (70, 6)])
def test_frontiers_around_the_groups(roots, D):
    w = _wide_roots(roots, D, roots + D, B=4)
    print("[oneshot] roots", roots, "D", D, flush=True)
    check_against_oracle(w, run_gpu(w, k=4), k=4)


@pytest.mark.parametrize("D", [12, 16, 20])
def test_many_instances(D):
    """More instances than wide workgroups fit the chip."""
    w = synth.make_random_small(7, B=520, n=14, D=D, M=4, K=2, H=2, shard_frac=0.5, uniform_beta=D == 16)
    print("[oneshot] 520 instances, D", D, flush=True)
    check_against_oracle(w, run_gpu(w, k=4), k=4)


@pytest.mark.parametrize("n", [447, 448])
def test_large_instances(n):
    """More instances than compute units, just below and from the size where
    they no longer take wide workgroups."""
    w = synth.make_random_small(8, B=257, n=n, D=20, M=4, K=2, H=1, p_edge=0.004, shard_frac=0.1, max_shard=2)
    print("[oneshot] 257 instances of", n, flush=True)
    assert np.diff(w.stage_off).max() == n
    check_against_oracle(w, run_gpu(w, k=4), k=4)


@pytest.mark.parametrize("D,M", [(16, 32), (16, 33), (24, 21), (24, 22), (32, 16), (32, 17), (32, 64)])
@pytest.mark.parametrize("uniform", [True, False], ids=["uniform", "tiered"])
def test_tables(D, M, uniform):
    """Up to 512 (model, device) pairs the workgroup prepares every load's
    residency, with more each stage loads its own; the transfer table is there
    where a set of the launch has a horizon.  Tight capacities, so that loads
    evict; each set of a sweep over the horizons writes its single call's bits."""
    w = synth.make_random_small(60 + D + M, B=5, n=50, D=D, M=M, K=4, H=2, shard_frac=0.5, max_shard=4, p_edge=0.07,
                                uniform_beta=uniform)
    print("[oneshot] tables D=%d M=%d uniform=%d" % (D, M, uniform), flush=True)
    for H in (0, 2):
        check_against_oracle(w, run_gpu(w, H=H, k=4), H=H, k=4)
    pk = fate.fate_pack_dags(w)
    st = fate.fate_pack_state(pk, w)
    sets = [fate.make_params(w, H=h) for h in (0, 1, 2)]
    sweep = fate.fate_score_sweep(pk, st, sets)[:, :st.n_cand].cpu().numpy()
    for p, one in zip(sets, sweep):
        got = fate.fate_score_frontier(pk, st, p)[:st.n_cand].cpu().numpy()
        assert np.array_equal(got.view(np.uint32), one.view(np.uint32))


def test_nothing_to_move():
    w = synth.make_random_small(9, B=3, n=30, D=10, M=4, K=3, H=3, shard_frac=0.5)
    w.out_bytes[::2] = 0.0
    print("[oneshot] zero outputs", flush=True)
    check_against_oracle(w, run_gpu(w, k=4), k=4)
    check_against_oracle(w, run_gpu(w, k=4, params=dict(lam_tr=0.0)), k=4, params=dict(lam_tr=0.0))


@pytest.mark.parametrize("D,uniform", [(16, True), (24, False)])
def test_same_bits_from_every_call(D, uniform):
    w = synth.make_random_small(21, B=40, n=60, D=D, M=6, K=4, H=3, shard_frac=0.4, p_edge=0.06, uniform_beta=uniform)
    print("[oneshot] plain, planning, sweep, D", D, flush=True)
    pk = fate.fate_pack_dags(w)
    st, sa = fate.fate_pack_state(pk, w), fate.fate_pack_state(pk, w, advance=True)
    sets = [fate.make_params(w, lam_tr=0.1 * i) for i in range(16)]
    sweep = fate.fate_score_sweep(pk, st, sets)[:, :st.n_cand].cpu().numpy()
    for i in (0, 7, 15):
        one = fate.fate_score_frontier(pk, st, sets[i])[:st.n_cand].cpu().numpy()
        plan = fate.fate_score_frontier(pk, sa, sets[i])[:st.n_cand].cpu().numpy()
        assert np.array_equal(one.view(np.uint32), sweep[i].view(np.uint32))
        assert np.array_equal(one.view(np.uint32), plan.view(np.uint32))
