"""Device memory of a context: an allocation that fails takes back what lies
idle, in this context and in others, and a call that cannot get its memory
leaves the context as it was."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import DeviceWindow, compare_decisions, leave_error, limit_memory, load_window, reqs_of

pytestmark = pytest.mark.gpu

MIB = 1 << 20


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


def _window(seed, cap=20000):
    return synth.generate("c2", seed=seed, n_req=256, n_sess=64, cap=cap)


def test_growth_takes_back_idle_memory(scorer):
    """A second load leaves the first snapshot's buffers idle; the first
    scoring call then needs its group table (128 MiB and more), which fits
    only where the idle buffers were."""
    w = _window(1, cap=200000)
    load_window(scorer, w)
    load_window(scorer, w)
    held = limit_memory(scorer, 0)
    limit_memory(scorer, held + 16 * MIB)
    res, sizes = DeviceWindow(w).score(scorer)
    compare_decisions(res, sizes, oracle.Oracle.from_window(w).window_score(w))
    limit_memory(scorer, 0)


def test_idle_memory_follows_the_snapshot(scorer):
    """After a small snapshot the context keeps no more than three times what
    it uses, whatever was loaded before."""
    small = _window(2, cap=4096)
    load_window(scorer, small)
    load_window(scorer, small)
    a = limit_memory(scorer, 0)
    load_window(scorer, _window(3, cap=200000))
    load_window(scorer, small)
    b = limit_memory(scorer, 0)
    assert b <= 3 * a, (a, b)


def test_out_of_memory_is_an_error_and_no_more(ps, scorer):
    """Loads and scoring calls that cannot get their memory: PS_E_NOMEM, the
    snapshot as before, and the next call works."""
    w, other = _window(4), _window(5, cap=400000)
    load_window(scorer, w)
    want = scorer.state()
    limit_memory(scorer, 1)
    dw = DeviceWindow(w)
    for call in (lambda: load_window(scorer, other), lambda: dw.score(scorer)):
        with pytest.raises(ps.PackServeError) as e:
            call()
        assert e.value.code == ps.binding.PS_E_NOMEM
    limit_memory(scorer, 0)
    for k, v in scorer.state().items():
        assert (v == want[k]).all(), k
    res, sizes = dw.score(scorer)
    compare_decisions(res, sizes, oracle.Oracle.from_window(w).window_score(w))


@pytest.mark.parametrize("popular", [False, True])
def test_scoring_that_ran_out_scores_again(ps, scorer, popular):
    """A larger window whose tables grow only in part, for a range of limits,
    after windows of both parities: PS_E_NOMEM, then the same decisions as
    without a limit (the half-grown group table is cleared first, and no
    window's leader lists are those of an earlier one)."""
    kw = dict(sp_frac=0.9, sp_blocks=64, n_inst=96) if popular else {}
    large = synth.generate("c2", seed=8, n_req=6000, n_sess=64, cap=20000, **kw)
    small = large.subset(range(64))
    d_small, d_large = DeviceWindow(small), DeviceWindow(large)
    want = oracle.Oracle.from_window(large).window_score(large)
    failed = 0
    for k in range(24):
        s = ps.Scorer(0)
        load_window(s, large)
        limit_memory(s, 1)  # gives the load's idle buffers back
        with pytest.raises(ps.PackServeError):
            d_small.score(s, with_sizes=False)
        limit_memory(s, 0)
        for _ in range(2 + k % 2):
            d_small.score(s, with_sizes=False)
        limit_memory(s, limit_memory(s, 0) + int(1000 * 1.45 ** k))
        try:
            d_large.score(s, with_sizes=False)
        except ps.PackServeError as e:
            assert e.code == ps.binding.PS_E_NOMEM
            failed += 1
        limit_memory(s, 0)
        for sizes in (False, True):
            compare_decisions(*d_large.score(s, with_sizes=sizes), want, label=f"limit {k}")
        s.close()
    assert 0 < failed < 24, failed


def test_idle_memory_of_another_context(ps, scorer):
    """What another context keeps idle is given back where this one runs out
    (a limit no release can meet: every context is asked)."""
    other = ps.Scorer(0)
    w = _window(6, cap=200000)
    load_window(other, w)
    load_window(other, w)
    before = limit_memory(other, 0)
    load_window(scorer, _window(7))
    limit_memory(scorer, 1)
    with pytest.raises(ps.PackServeError):
        DeviceWindow(w).score(scorer)
    assert limit_memory(other, 0) < before
    res, sizes = DeviceWindow(w).score(other)
    compare_decisions(res, sizes, oracle.Oracle.from_window(w).window_score(w))
    other.close()


def test_contexts_in_threads_share_what_lies_idle(ps):
    """One context runs out again and again, which takes back what the other,
    in another thread, has just put aside: that one's loads, commits and windows
    stay the same."""
    import threading
    w = _window(10, cap=60000)
    inst = (np.arange(w.n_req) % w.n_inst).astype(np.int32)
    dw, poor_dw = DeviceWindow(w), DeviceWindow(w)
    o = oracle.Oracle.from_window(w)
    before = o.window_score(w)
    o.commit(w.pool, w.pre_off, w.pre_len, w.tail_off, w.tail_len, inst)
    after = o.window_score(w)
    done, failures = threading.Event(), []

    def run_out():
        s = ps.Scorer(0)
        load_window(s, w)
        limit_memory(s, 1)
        while not done.is_set():
            try:
                poor_dw.score(s)
                failures.append("the call got memory")
                break
            except ps.PackServeError as e:
                if e.code != ps.binding.PS_E_NOMEM:
                    failures.append(str(e))
                    break
        s.close()

    t = threading.Thread(target=run_out)
    t.start()
    try:
        rich = ps.Scorer(0)
        for _ in range(12):
            load_window(rich, w)
            compare_decisions(*dw.score(rich), before)
            rich.commit(w.pool, reqs_of(w), inst)
            compare_decisions(*dw.score(rich), after)
        rich.close()
    finally:
        done.set()
        t.join()
    assert not failures, failures


@pytest.mark.parametrize("what", ["commit", "schedule", "replay", "events", "feedback"])
def test_an_earlier_error_does_not_end_a_call_half_way(ps, scorer, what):
    """A failed HIP call of the program itself, whose error nobody read: a call
    that changes the snapshot reports it before any change, or works."""
    w = _window(9)
    dw = DeviceWindow(w)
    inst = (np.arange(w.n_req) % w.n_inst).astype(np.int32)
    every = np.arange(w.n_inst)
    call = {"commit": lambda: scorer.commit(w.pool, reqs_of(w), inst), "schedule": lambda: dw.schedule(scorer),
            "replay": lambda: dw.replay(scorer, inst),
            "events": lambda: scorer.apply_events(every, 0 * every + ps.PS_EV_DECODE_TOKENS, 100_000 + 0 * every),
            "feedback": lambda: scorer.feedback_decode([4] * 50, [1000] * 50, [0.5] * 50)}[what]

    def seen():
        res, sizes = dw.score(scorer)
        return [*scorer.state().values(), *scorer.model().values(), dw.hits(scorer, w.n_inst), sizes.copy(), res.copy()]

    load_window(scorer, w)
    want = seen()
    leave_error()
    try:
        call()
    except ps.PackServeError:
        assert all((a == b).all() if hasattr(a, "all") else a == b for a, b in zip(want, seen()))
        call()
    assert not (want[-1] == seen()[-1]).all()  # the call had its effect
