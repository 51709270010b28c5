"""The prefix index where its build by sorted runs can go wrong: buckets that
overflow into the next ones, past the table's last bucket and around to its
first, around several chunks of runs, and blocks at both sides of the bitmap
limit.  Scored against the oracle, which knows no index."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import DeviceWindow, compare_decisions, edge_window, load_window

pytestmark = pytest.mark.gpu

M64 = (1 << 64) - 1
XOR = 0x9E3779B97F4A7C15 * 0x10001 & M64
MUL = 0xD6E8FEB86659FD93
INV = pow(MUL, -1, 1 << 64)


def _key(x):
    """The block hash whose index hash is x."""
    return (x * INV & M64) ^ XOR


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


def _score(scorer, sets, chains, label):
    w = edge_window(sets, chains)
    load_window(scorer, w)
    o = oracle.Oracle.from_window(w)
    dw = DeviceWindow(w)
    assert (dw.hits(scorer, w.n_inst) == o.window_hits(w)).all(), label
    res, sizes = dw.score(scorer)
    compare_decisions(res, sizes, o.window_score(w), label=label)
    plain, _ = dw.score(scorer, with_sizes=False)
    assert (plain == res).all(), label


@pytest.mark.parametrize("last,first,spread", [
    (9, 0, 23),      # one bucket too many by one
    (20, 8, 36),     # a full first bucket behind the wrap
    (40, 30, 0),     # every key in two buckets
    (700, 10, 5000),  # a wrap of hundreds, more than one chunk of runs
    (3000, 0, 100),  # the wrap begins a chunk before the last
])
def test_index_wraps(ps, scorer, last, first, spread):
    rng = np.random.default_rng(last + spread)
    keys = [_key(M64 - k) for k in range(last)] + [_key(1 + k) for k in range(first)]
    keys += [_key(int(x)) for x in rng.integers(1 << 40, 1 << 63, spread)]
    keys = [keys[i] for i in rng.permutation(len(keys))]
    absent = [_key(M64 - last - k) for k in range(8)] + [_key(first + 1 + k) for k in range(8)]
    sets = [keys[::2], keys[1::2], keys[::3]]
    pick = [keys[i] for i in rng.permutation(len(keys))[:300]]
    # chains of one, and of eight so that they form prefix groups
    chains = [[k, 5 + i] for i, k in enumerate(pick + absent)]
    chains += [([k] + list(range(100, 108)), [9]) for k in pick[:40]]
    _score(scorer, sets, chains, f"index wrap {last}/{first}/{spread}")


@pytest.mark.parametrize("holders", [1, 63, 64, 65, 66, 129])
def test_index_holder_counts(ps, scorer, holders):
    """Blocks with just under, at and over the bitmap limit, at the head and at
    the end of the sorted pairs."""
    n_inst = 130
    shared = [_key(1), _key(1 << 60), _key(M64)]
    sets = [(shared if i < holders else shared[:1] if i % 3 == 0 else []) + [1000 + i] for i in range(n_inst)]
    chains = [shared + [7, 8, 9], shared[:2], shared[:1] + [11], shared[1:], [1000, 1], [77]]
    chains += [(shared + [1 << 20 | i for i in range(20)], [i + 1]) for i in range(5)]
    _score(scorer, sets, chains, f"holders {holders}")
