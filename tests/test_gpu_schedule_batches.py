"""The per-arrival scheduler's batches where a batch has to end early or look
again: chains that hold one block at different positions or behind different
blocks, repeats inside a chain, zero hashes, caps that bind inside a batch and
instances that are full from the start, tables with holes behind a common
prefix, malformed descriptors among the requests, and pools on both sides of
what the deciding workgroup stages in LDS, batches cut by their positions, and
windows whose batches or rows of hits find no device memory.  Against the in-order scheduler
(every request scored in full) byte for byte, and against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import (DeviceWindow, compare_sequential, edge_window, limit_memory, limit_positions, load_window,
                            nb_cap, reqs_of)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ps():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_33224_amd as ps
    return ps


@pytest.fixture()
def scorer(ps):
    s = ps.Scorer(0)
    yield s
    s.close()


def _run(scorer, w, batch, reqs=None):
    load_window(scorer, w)
    scorer.set_schedule_speculation(batch)
    dw = DeviceWindow(w)
    if reqs is not None:
        import paper_2609_33224_amd as ps
        dw.d_reqs = ps.to_device_bytes(reqs)
    res, sizes, dropped = dw.schedule(scorer)
    plain = None
    if batch:
        load_window(scorer, w)
        plain = dw.schedule(scorer, with_sizes=False)[0].copy()
    return res.copy(), sizes.copy(), dropped, scorer.state(), scorer.schedule_stats(), plain


def _check(scorer, w, label, reqs=None, follow=True):
    a, b = _run(scorer, w, 0, reqs), _run(scorer, w, 256, reqs)
    bad = np.nonzero(a[0] != b[0])[0]
    assert len(bad) == 0, f"{label}: {len(bad)} differ, first {bad[0]}: {a[0][bad[0]]} {b[0][bad[0]]}"
    assert (a[1] == b[1]).all(), f"{label}: set sizes"
    assert a[2] == b[2], f"{label}: dropped {a[2]} {b[2]}"
    for k in a[3]:
        assert (a[3][k] == b[3][k]).all(), f"{label}: {k}"
    assert (b[5] == b[0]).all(), f"{label}: without set sizes"
    valid = w.n_req if reqs is None else int((b[0]["flags"] != 8).sum())
    assert sum(b[4]) == valid, f"{label}: {b[4]} of {valid}"
    if follow and reqs is None:
        o = oracle.Oracle.from_window(w)
        od, dropped = o.window_schedule(w, follow=b[0]["instance"])
        empty = int((w.pre_len + w.tail_len == 0).sum())  # Z = 0: marked near its boundary
        compare_sequential(b[0], b[1], od, label=label, max_nb=nb_cap(w.n_req) + empty)
        assert dropped == b[2]
    return b


def _sessions(seed, n_inst, n_req, n_sess, longest, cap=None, holes=0.0, step=24):
    """Requests that follow their sessions; instances hold prefixes of them,
    some with a hole, so a table may go on behind a common prefix."""
    rng = np.random.default_rng(seed)
    sess = [[(k + 1) * 10**6 + 7 * j for j in range(int(rng.integers(3, longest)))] for k in range(n_sess)]
    at = [int(rng.integers(0, 10)) for _ in sess]
    chains = []
    for r in range(n_req):
        k = int(rng.integers(n_sess))
        at[k] = min(len(sess[k]), at[k] + int(rng.integers(0, step)))
        chains.append((sess[k][:at[k]], [9 * 10**8 + 10 * r + j for j in range(int(rng.integers(0, 3)))]))
    sets = []
    for i in range(n_inst):
        s = sess[int(rng.integers(n_sess))]
        have = s[:int(rng.integers(0, len(s) + 1))]
        if len(have) > 4 and rng.random() < holes:
            cut = int(rng.integers(1, len(have) - 2))
            have = have[:cut] + have[cut + 2:]
        sets.append(have)
    if cap is None:
        cap = max(len(s) for s in sets) + sum(len(a) + len(b) for a, b in chains) + 1
    return edge_window(sets, chains, cap=max(cap, max(len(s) for s in sets), 1), eta=0.31)


@pytest.mark.parametrize("n_inst,n_req,n_sess", [(1, 300, 5), (2, 257, 3), (65, 600, 40), (300, 513, 200)])
@pytest.mark.parametrize("holes", [0.0, 1.0])
def test_batches_follow_sessions(ps, scorer, n_inst, n_req, n_sess, holes):
    w = _sessions(n_inst + n_req, n_inst, n_req, n_sess, 120, holes=holes)
    _check(scorer, w, f"sessions {n_inst} x {n_req}, holes {holes}")


@pytest.mark.parametrize("cap", [1, 30, 90, 140, 400])
def test_batches_cap(ps, scorer, cap):
    _check(scorer, _sessions(cap, 7, 520, 12, 100, cap=cap), f"cap {cap}")


@pytest.mark.parametrize("n_inst", [4095, 4096, 4097, 5003])
def test_batches_pool_sizes(ps, scorer, n_inst):
    _check(scorer, _sessions(n_inst, n_inst, 270, 60, 60), f"pool {n_inst}", follow=n_inst == 4097)


@pytest.mark.parametrize("kind", ["shifted", "behind", "repeats", "all"])
def test_batches_irregular_chains(ps, scorer, kind):
    """Blocks that do not name a prefix: batches end before them (or the
    in-order scheduler takes over), with the same results."""
    rng = np.random.default_rng(len(kind))
    base = [1000 + j for j in range(40)]
    chains = []
    for r in range(400):
        own = [10**7 + 100 * r + j for j in range(6)]
        pre = base[:int(rng.integers(1, 40))]
        x = rng.random()
        if kind in ("shifted", "all") and x < 0.1:
            chains.append((own[:2] + pre, own[2:]))  # the base at other positions
        elif kind in ("behind", "all") and x < 0.2:
            chains.append((own[:1] + pre[1:], own[1:]))  # the same positions behind another block
        elif kind in ("repeats", "all") and x < 0.3:
            chains.append((pre, own + pre[:3] + own[:2]))
        else:
            chains.append((pre, own))
    sets = [base[:int(rng.integers(0, 40))] for _ in range(9)]
    _check(scorer, edge_window(sets, chains, cap=9000, eta=0.31), kind)


def test_batches_mostly_irregular(ps, scorer):
    """Every request breaks the batch: the in-order scheduler takes the rest."""
    chains = [([5000 + (j * 7 + r) % 50 for j in range(20)], [10**6 + r]) for r in range(300)]
    sets = [[5000 + j for j in range(10)], [], [5003, 5010, 5017]]
    _check(scorer, edge_window(sets, chains, cap=2000, eta=0.31), "mostly irregular")


@pytest.mark.parametrize("cap", [9000, 130])
def test_what_batches_leave_is_speculated(ps, scorer, cap):
    """Every chain begins somewhere else in one session, so any two of them end
    a batch: the in-order scheduler takes the window, from speculative results
    too (a launch of up to 256 requests scored in parallel)."""
    rng = np.random.default_rng(11)
    base = [1000 + j for j in range(120)]
    chains = []
    for r in range(500):
        k = int(rng.integers(0, 60))
        chains.append((base[k:k + 60], [10**6 + 10 * r + j for j in range(int(rng.integers(0, 3)))]))
    sets = [base[:int(rng.integers(0, 120))] for _ in range(64)]
    b = _check(scorer, edge_window(sets, chains, cap=cap, eta=0.31), f"one session, cap {cap}")
    assert b[4][0] > 100, f"decided from speculation: {b[4]}"


@pytest.mark.parametrize("max_pos", [1, 130, 1000, 5000])
@pytest.mark.parametrize("cap", [None, 90])
def test_batches_cut_by_positions(ps, scorer, max_pos, cap):
    limit_positions(scorer, max_pos)
    _check(scorer, _sessions(max_pos, 7, 400, 12, 100, cap=cap), f"{max_pos} positions a batch, cap {cap}")


def _limited(ps, scorer, w, room):
    """The schedule of w with `room` bytes of device memory more than the
    loaded context holds, against the one without a limit."""
    dw = DeviceWindow(w)
    load_window(scorer, w)
    want = [x.copy() if hasattr(x, "copy") else x for x in dw.schedule(scorer)]
    state = scorer.state()
    s = ps.Scorer(0)
    load_window(s, w)
    limit_memory(s, 1)
    with pytest.raises(ps.PackServeError):
        dw.score(s)  # gives the load's idle buffers back
    limit_memory(s, limit_memory(s, 0) + room)
    got = dw.schedule(s)
    assert (got[0] == want[0]).all() and (got[1] == want[1]).all() and got[2] == want[2]
    for k, v in s.state().items():
        assert (v == state[k]).all(), k
    s.close()


def test_schedule_without_room_for_batches(ps, scorer):
    """The batches' workspace (28 bytes for each of 4 M positions) does not
    fit: the requests are taken in order, the results are the same."""
    w = edge_window([[5, 6], [7], [], [8]], None, pool=list(range(1, 20_002)), cap=50_000,
                    reqs=[(r % 2, 20_000 - r % 7, 0, 0) for r in range(200)], eta=0.31)
    _limited(ps, scorer, w, 30_000_000)


def test_schedule_rows_for_what_batches_leave(ps, scorer):
    """Chains that end every batch early, on 2,000 instances: what is left to
    the in-order scheduler needs no more memory than the batches took."""
    chains = [([5000 + (j * 7 + r) % 50 for j in range(20)], [10**6 + r]) for r in range(3000)]
    w = edge_window([[5000 + j for j in range(i % 12)] for i in range(2000)], chains, cap=300, eta=0.31)
    _limited(ps, scorer, w, 12_000_000)


def test_schedule_that_runs_out_changes_nothing(ps, scorer):
    w = _sessions(3, 40, 300, 20, 60)
    load_window(scorer, w)
    want = scorer.state()
    dw = DeviceWindow(w)
    limit_memory(scorer, 1)
    with pytest.raises(ps.PackServeError) as e:
        dw.schedule(scorer)
    assert e.value.code == ps.binding.PS_E_NOMEM
    limit_memory(scorer, 0)
    for k, v in scorer.state().items():
        assert (v == want[k]).all(), k
    o = oracle.Oracle.from_window(w)
    assert (dw.hits(scorer, w.n_inst) == o.window_hits(w)).all()


def test_batches_zero_hashes_and_malformed(ps, scorer):
    w = _sessions(77, 20, 600, 30, 80)
    rng = np.random.default_rng(5)
    for k in rng.integers(0, len(w.pool), 40):
        w.pool[k] = 0
    reqs = reqs_of(w)
    for r in rng.integers(0, 600, 30):
        reqs["pre_off"][r] = -1
    for r in rng.integers(0, 600, 10):
        reqs["tail_len"][r] = len(w.pool) + 1
    reqs["pre_off"][0] = reqs["pre_off"][255] = reqs["pre_off"][256] = -1
    b = _check(scorer, w, "zero hashes, malformed", reqs=reqs)
    assert (b[0]["flags"] == 8).sum() >= 30
