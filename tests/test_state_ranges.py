"""Validation of a state on several threads: batches of at least four ranges
of 32,768 stages, with empty instances and an instance larger than a range.
The frontier, its offsets and the completed-parent lists are those of the same
instances packed in pieces too small for a second thread, and of several errors
the one that comes first in (instance, stage) order is returned."""

import ctypes as C
import dataclasses

import numpy as np
import pytest

import builders
from paper_2605_07238_amd import fate

D = 5
# a range border falls on an empty instance, inside the largest one and between two
SIZES = [0, 20000, 0, 12768, 0, 1, 70000, 3, 0, 0, 30000, 2768, 40000, 1, 17000, 0]


def _piece(w, b0, b1):
    """Instances b0 .. b1 of the batch."""
    s = slice(int(w.stage_off[b0]), int(w.stage_off[b1]))
    e = slice(int(w.par_off[s.start]), int(w.par_off[s.stop]))
    over = {f: getattr(w, f)[s] for f in ("model", "elig", "shard_max", "prefix_hash", "prefix_tokens", "out_bytes",
                                          "holders", "status")}
    over.update({f: getattr(w, f)[b0:b1] for f in ("resident", "prefix_cache", "tau_free", "t_now")})
    return dataclasses.replace(w, stage_off=w.stage_off[b0:b1 + 1] - s.start,
                               par_off=w.par_off[s.start:s.stop + 1] - e.start, par_idx=w.par_idx[e], **over)


def _sections(w):
    _, h, _ = fate.fate_layout_dags(w)
    img, st, _ = fate.fate_layout_state(h, w)

    def take(ptr, n):
        off = ptr - img.ctypes.data
        return img[off:off + 4 * n].view(np.uint32).copy()

    F = int(st.n_frontier)
    return dict(frontier=take(st.frontier, 2 * F).reshape(F, 2), cand_off=take(st.cand_off, F + 1),
                fr_off=take(st.fr_off, w.B + 1), done_n=take(st.done_n, w.N), done=take(st.done, 4 * int(h.E)),
                counts=(F, int(st.n_cand)))


def test_ranges_give_the_pieces_image():
    w = builders.random_batch(SIZES, 1, D=D)
    assert w.N >= 4 * 32768
    got = _sections(w)
    F = C0 = 0
    for b0 in range(0, w.B):
        p = _piece(w, b0, b0 + 1)  # one instance: one thread, whatever its size
        if p.N == 0:
            assert got["fr_off"][b0 + 1] == got["fr_off"][b0]
            continue
        x = _sections(p)
        s, e = int(w.stage_off[b0]), int(w.par_off[w.stage_off[b0]])
        f, c = x["counts"]
        assert got["fr_off"][b0] == F and got["fr_off"][b0 + 1] == F + f
        assert np.array_equal(got["frontier"][F:F + f, 0], x["frontier"][:, 0] + s)
        assert np.all(got["frontier"][F:F + f, 1] == b0)
        assert np.array_equal(got["cand_off"][F:F + f + 1], x["cand_off"] + C0)
        assert np.array_equal(got["done_n"][s:s + p.N], x["done_n"])
        assert np.array_equal(got["done"][4 * e:4 * e + len(x["done"])], x["done"])
        F, C0 = F + f, C0 + c
    assert got["counts"] == (F, C0)


def _plant(w, kind, s):
    """An error of the kind at flat stage s (which is pending with a pending
    parent, or completed, as the kind needs); returns the status it gives."""
    if kind == "status":
        w.status[s] = 7
        return fate.FATE_EINVAL
    if kind == "device":
        w.holders[s] = np.uint64(1 << D)
        return fate.FATE_ESTATE
    if kind == "early":  # completed before its parents
        w.status[s], w.holders[s] = 1, 1
        return fate.FATE_ESTATE
    w.par_idx[w.par_off[s]] = 1 << 20  # "parent": a parent that is no earlier stage
    return fate.FATE_ECYCLE


def _where(w, b):
    """Stages of instance b for the kinds: any; pending with a pending parent (which has parents)."""
    s, e = int(w.stage_off[b]), int(w.stage_off[b + 1])
    base = s
    out = []
    for v in range(e - 1, s - 1, -1):
        ps = w.par_idx[w.par_off[v]:w.par_off[v + 1]]
        if w.status[v] == 0 and any(w.status[base + p] != 1 for p in ps):
            out.append(v)
            if len(out) == 2:
                break
    return sorted(out)


@pytest.mark.parametrize("first,second", [(1, 14), (6, 12), (3, 6), (10, 14), (6, 6), (12, 1)])
def test_first_error_in_stage_order(first, second):
    """Two errors in different ranges (or one), either kind first; the state
    calls and the host layout return the earlier one's status."""
    w = builders.random_batch(SIZES, 2, D=D)
    _, h, _ = fate.fate_layout_dags(w)
    lib = fate.load()
    kinds = ("status", "device", "early", "parent")
    for i, ka in enumerate(kinds):
        for kb in kinds[i + 1:] + kinds[:i]:
            x = dataclasses.replace(w, status=w.status.copy(), holders=w.holders.copy(), par_idx=w.par_idx.copy())
            sa, sb = _where(w, first)[0], _where(w, second)[-1]
            want = {sa: _plant(x, ka, sa)}
            want[sb] = _plant(x, kb, sb)
            expect = want[min(want)]
            hi = fate.HostInputs(x)
            n, nf, nc = C.c_size_t(0), C.c_int64(0), C.c_int64(0)
            assert lib.fate_pack_state_size(C.byref(h), C.byref(hi.batch), C.byref(hi.state), 3, C.byref(n), C.byref(nf),
                                            C.byref(nc)) == expect, (ka, kb)
            assert lib.fate_pack_state_advance_size(C.byref(h), C.byref(hi.batch), C.byref(hi.state), 3,
                                                    C.byref(n)) == expect, (ka, kb)
            buf, sh = np.zeros(8, np.uint8), fate.StateH()
            assert lib.fate_layout_state(C.byref(h), C.byref(hi.batch), C.byref(hi.state), 3, buf.ctypes.data, 8,
                                         C.byref(sh)) == expect, (ka, kb)
            assert (n.value, nf.value, nc.value) == (0, 0, 0) and not buf.any()
