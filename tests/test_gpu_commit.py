"""ps_commit against the oracle's entry-by-entry commit, at the sizes where a
batch taken position by position can go wrong: chains that end at and around a
chunk of positions, chunks that hold hundreds of short chains, blocks that
repeat inside a chain and across the chains of one instance, caps that bind
inside a chain, at a repeat and before the first block, empty chains, and
placements that skip entries; commits cut into slices, and commits that run
out of device memory."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import (DeviceWindow, compare_decisions, edge_window, limit_memory, limit_positions, load_window,
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


def _check(scorer, w, inst, label):
    load_window(scorer, w)
    o = oracle.Oracle.from_window(w)
    want = o.commit(w.pool, w.pre_off, w.pre_len, w.tail_off, w.tail_len, inst)
    got = scorer.commit(w.pool, reqs_of(w), np.asarray(inst, np.int32))
    so, sg = o.state(), scorer.state()
    for k in ("D", "Q", "P", "S", "set_size"):
        assert (so[k] == sg[k]).all(), f"{label}: {k} differs"
    assert want == got, f"{label}: dropped {got}, oracle {want}"
    dw = DeviceWindow(w)
    assert (dw.hits(scorer, w.n_inst) == o.window_hits(w)).all(), f"{label}: tables differ"
    res, sizes = dw.score(scorer)  # the index and the rows
    # an empty chain has Z = 0, which the oracle marks near its boundary
    empty = int((w.pre_len + w.tail_len == 0).sum())
    compare_decisions(res, sizes, o.window_score(w), label=label, max_nb=nb_cap(w.n_req) + empty)
    plain, _ = dw.score(scorer, with_sizes=False)
    assert (plain == res).all(), f"{label}: the two scoring paths differ"


def _window(seed, n_inst, n_req, len_lo, len_hi, cap=None, repeats=0.0, shared=0.5, held=40):
    """Chains over a small alphabet of sessions: a request takes a prefix of a
    session's chain and a tail; `repeats` of the tails hold blocks of their own
    chain again; instances hold session prefixes, some with a hole."""
    rng = np.random.default_rng(seed)
    nxt = iter(rng.permutation(1 << 20).astype(np.uint64) + np.uint64(1))
    sess = [[next(nxt) for _ in range(int(rng.integers(max(1, len_lo), len_hi + 1)))]
            for _ in range(max(1, int(n_req * (1 - shared))))]
    chains = []
    for _ in range(n_req):
        s = sess[int(rng.integers(len(sess)))]
        pre = s[:int(rng.integers(0, len(s) + 1))]
        tail = [next(nxt) for _ in range(int(rng.integers(0, 4)))]
        if pre and rng.random() < repeats:
            tail = tail + [pre[int(k)] for k in rng.integers(0, len(pre), 3)] + tail[:1]
        chains.append((pre, tail))
    sets = []
    for _ in range(n_inst):
        have = []
        for _ in range(int(rng.integers(0, 4))):
            s = sess[int(rng.integers(len(sess)))]
            cut = s[:int(rng.integers(0, min(len(s), held) + 1))]
            if len(cut) > 2 and rng.random() < 0.5:
                del cut[int(rng.integers(1, len(cut)))]
            have += cut
        sets.append(sorted(set(have), key=have.index))
    if cap is None:
        cap = 1 + max(len(s) for s in sets) + sum(len(a) + len(b) for a, b in chains)
    else:
        cap = max(cap, max(len(s) for s in sets), 1)
    w = edge_window(sets, chains, cap=cap)
    inst = rng.integers(-1, n_inst, n_req).astype(np.int32)
    return w, inst


@pytest.mark.parametrize("len_lo,len_hi,n_req,n_inst", [
    (1, 3, 700, 3),        # hundreds of chains per chunk of 1,024 positions
    (0, 1, 40, 2),         # empty chains among them
    (1020, 1027, 9, 2),    # chains around one chunk
    (2047, 2049, 5, 1),    # one instance, chains around two chunks
    (30, 300, 150, 70),    # more instances than a wave
])
@pytest.mark.parametrize("repeats", [0.0, 0.6])
def test_commit_chunks(ps, scorer, len_lo, len_hi, n_req, n_inst, repeats):
    w, inst = _window(len_lo * 7 + n_req, n_inst, n_req, len_lo, len_hi, repeats=repeats)
    _check(scorer, w, inst, f"commit {len_lo}-{len_hi} x {n_req} on {n_inst}, repeats {repeats}")


@pytest.mark.parametrize("cap", [1, 41, 64, 500, 1500])
@pytest.mark.parametrize("repeats", [0.0, 0.9])
def test_commit_cap_binds(ps, scorer, cap, repeats):
    w, inst = _window(cap + 3, 3, 120, 5, 90, cap=cap, repeats=repeats, held=40)
    _check(scorer, w, inst, f"commit cap {cap}, repeats {repeats}")


def test_commit_no_placement(ps, scorer):
    w, inst = _window(5, 4, 20, 1, 30)
    inst[:] = -1
    _check(scorer, w, inst, "commit without placements")


def test_commit_empty_chains_only(ps, scorer):
    w = edge_window([[1, 2], [3]], [[], [], []], cap=8)
    _check(scorer, w, np.array([0, 1, 0], np.int32), "commit of empty chains")


def test_commit_twice(ps, scorer):
    """A second commit of the same window finds every block and adds none."""
    w, inst = _window(11, 5, 60, 10, 200)
    load_window(scorer, w)
    scorer.commit(w.pool, reqs_of(w), inst)
    held = scorer.state()["set_size"]
    P = scorer.state()["P"]
    assert scorer.commit(w.pool, reqs_of(w), inst) == 0
    assert (scorer.state()["set_size"] == held).all()
    assert (scorer.state()["P"] == P).all()


@pytest.mark.parametrize("at", [0, 1, 62, 4095, 4096, 12288, 12290])
def test_zero_hash_refused(ps, scorer, at):
    """A zero hash anywhere in a host pool or in the snapshot's lists: refused
    with its index, nothing changed (odd and even lengths, first and last)."""
    n = 12291
    w = edge_window([[5, 6, 7], [8]], [list(range(10, 10 + n))], cap=2 * n)
    load_window(scorer, w)
    before = scorer.state()
    pool = w.pool.copy()
    pool[at] = 0
    for call in (lambda: scorer.score(pool, reqs_of(w)),
                 lambda: scorer.commit(pool, reqs_of(w), np.array([1], np.int32))):
        with pytest.raises(ps.PackServeError, match=rf"zero block hash at pool\[{at}\]") as e:
            call()
        assert e.value.code == -1
    blk = np.arange(1, n + 1, dtype=np.uint64)
    blk[at] = 0
    with pytest.raises(ps.PackServeError, match=rf"zero block hash at blk\[{at}\]"):
        scorer.load(2, n, np.array([0, n // 2, n], np.int64), blk, w.D, w.Q, w.P, w.S, ps.make_model(
            w.alpha, w.seg_ub, w.beta, w.gamma, 0.5, 0.05, 2.0, 556.0, 16, 512, 4_194_304))
    after = scorer.state()
    for k in before:
        assert (before[k] == after[k]).all(), k
    res = scorer.score(w.pool, reqs_of(w))  # the old snapshot still scores
    compare_decisions(res, None, oracle.Oracle.from_window(w).window_score(w))


@pytest.mark.parametrize("n", [300, 65536, 65537, 70001])  # the calling thread looks up to 65,536
def test_zero_hash_comes_first(ps, scorer, n):
    """A zero hash is refused as such whatever else is wrong with the call,
    also where nothing is placed, and a good call goes through."""
    w = edge_window([[5, 6, 7], [8]], [list(range(10, 10 + n))], cap=2 * n)
    load_window(scorer, w)
    reqs = reqs_of(w)
    for at in (0, n // 2, n - 1):
        pool = w.pool.copy()
        pool[at] = 0
        for call in (lambda: scorer.score(pool, reqs),
                     lambda: scorer.commit(pool, reqs, np.array([1], np.int32)),
                     lambda: scorer.commit(pool, reqs, np.array([-1], np.int32)),
                     lambda: scorer.commit(pool, reqs, np.array([2], np.int32))):
            with pytest.raises(ps.PackServeError, match=rf"zero block hash at pool\[{at}\]") as e:
                call()
            assert e.value.code == ps.binding.PS_E_INVAL
    with pytest.raises(ps.PackServeError) as e:
        scorer.commit(w.pool, reqs, np.array([2], np.int32))
    assert e.value.code == ps.binding.PS_E_RANGE
    assert scorer.commit(w.pool, reqs, np.array([-1], np.int32)) == 0
    compare_decisions(scorer.score(w.pool, reqs), None, oracle.Oracle.from_window(w).window_score(w))
    _check(scorer, w, np.array([1], np.int32), f"pool of {n}")


@pytest.mark.parametrize("max_pos", [1, 100, 1024, 3000])
@pytest.mark.parametrize("cap", [None, 41, 300])
def test_commit_slices(ps, scorer, max_pos, cap):
    """A commit cut into slices (blocks that an earlier slice inserted or
    refused come again in later ones) does what one slice does."""
    limit_positions(scorer, max_pos)
    w, inst = _window(max_pos, 3, 150, 5, 90, cap=cap, repeats=0.5, held=40)
    _check(scorer, w, inst, f"commit in slices of {max_pos}, cap {cap}")


def _runs_out(ps, scorer, w, inst, room):
    """A commit with `room` bytes more than the context holds: PS_E_NOMEM."""
    load_window(scorer, w)
    for n_bytes in (1, None):  # 1: gives the load's idle buffers back
        limit_memory(scorer, n_bytes or limit_memory(scorer, 0) + room)
        with pytest.raises(ps.PackServeError) as e:
            scorer.commit(w.pool, reqs_of(w), inst)
        assert e.value.code == ps.binding.PS_E_NOMEM
    limit_memory(scorer, 0)


def _long_last(long):
    """Fifty short chains, then one of `long` blocks, on three instances."""
    chains = [[10 ** 6 + 100 * r + j for j in range(20)] for r in range(50)] + [list(range(1, long + 1))]
    return edge_window([[5, 6], [7], []], chains, cap=2 * long), np.arange(51, dtype=np.int32) % 3


def test_commit_that_runs_out_changes_nothing(ps, scorer):
    """Memory for the first slices, not for a later, larger one: PS_E_NOMEM
    before the first placement, and the same commit works afterwards."""
    w, inst = _long_last(200_000)  # 5.6 MB of workspace for the last chain, 1.6 MB of hashes
    limit_positions(scorer, 400)
    _runs_out(ps, scorer, w, inst, 1_700_000 + 500_000)
    o = oracle.Oracle.from_window(w)
    so, sg = o.state(), scorer.state()
    for k in ("D", "Q", "P", "S", "set_size"):
        assert (so[k] == sg[k]).all(), k
    dw = DeviceWindow(w)
    assert (dw.hits(scorer, w.n_inst) == o.window_hits(w)).all()
    want = o.commit(w.pool, w.pre_off, w.pre_len, w.tail_off, w.tail_len, inst)
    assert scorer.commit(w.pool, reqs_of(w), inst) == want
    assert (dw.hits(scorer, w.n_inst) == o.window_hits(w)).all()


def test_commit_in_smaller_slices_where_memory_is_short(ps, scorer):
    """No room for the workspace of the whole commit (35 MB): slices that fit,
    the same tables."""
    w = edge_window([[5, 6], [7], []], None, pool=list(range(1, 25_002)), cap=50_000,
                    reqs=[(r % 2, 25_000 - r, 0, 0) for r in range(50)])
    inst = (np.arange(50) % 3).astype(np.int32)
    load_window(scorer, w)
    limit_memory(scorer, 1)
    with pytest.raises(ps.PackServeError):
        DeviceWindow(w).score(scorer)  # gives the idle buffers back
    limit_memory(scorer, limit_memory(scorer, 0) + 10_000_000)
    o = oracle.Oracle.from_window(w)
    want = o.commit(w.pool, w.pre_off, w.pre_len, w.tail_off, w.tail_len, inst)
    assert scorer.commit(w.pool, reqs_of(w), inst) == want
    limit_memory(scorer, 0)
    so, sg = o.state(), scorer.state()
    for k in ("D", "Q", "P", "S", "set_size"):
        assert (so[k] == sg[k]).all(), k
    assert (DeviceWindow(w).hits(scorer, w.n_inst) == o.window_hits(w)).all()


def test_commit_whose_index_has_no_room(ps, scorer):
    """Placements made, no memory to rebuild the prefix index: the context has
    no snapshot until the next load."""
    rng = np.random.default_rng(3)
    sets = [list(rng.integers(1, 1 << 40, 20_000).astype(np.uint64)) for _ in range(32)]
    w = edge_window(sets, [[1, 2, 3]], cap=30_000)
    load_window(scorer, w)
    scorer.commit(w.pool, reqs_of(w), np.array([-1], np.int32))  # the host pool's buffers
    _runs_out(ps, scorer, w, np.array([0], np.int32), 100_000)
    for call in (scorer.state, lambda: scorer.score(w.pool, reqs_of(w))):
        with pytest.raises(ps.PackServeError) as e:
            call()
        assert e.value.code == ps.binding.PS_E_STATE
    _check(scorer, w, np.array([0], np.int32), "after the next load")
