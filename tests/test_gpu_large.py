"""The early rounds of one instance above 2^20 states: a second round by labels
and a round by unique hashes, against the ordinary rounds (DFAMIN_NO_LABELS=4)
and the oracle."""
import numpy as np
import pytest

import oracle
from paper_2410_22764_amd import workloads as W

pytestmark = pytest.mark.gpu

N = (1 << 20) + 1  # the smallest size these rounds take


@pytest.fixture(scope="module")
def ctx():
    from paper_2410_22764_amd import dfamin
    c = dfamin.dfamin_create(0)
    yield c
    c.close()


def _redundant(n, k, classes, seed):
    """Every state copies a state of a random automaton of `classes` states."""
    r = np.random.RandomState(seed)
    cls = r.permutation(np.concatenate([np.arange(classes), r.randint(0, classes, n - classes)]))
    order = np.argsort(cls, kind="stable")
    size = np.bincount(cls, minlength=classes)
    start = np.cumsum(size) - size
    base = r.randint(0, classes, (k, classes))
    rows = np.stack([order[start[base[a][cls]] + (r.rand(n) * size[base[a][cls]]).astype(np.int64)] for a in range(k)])
    return W.from_rows(rows.astype(np.uint32), (r.rand(classes) < 0.5)[cls], int(r.randint(n)),
                       f"redundant({n},{k},{classes})")


def _crowd(n, k, seed):
    """Two states in five are copies of one state, the others random: a sample
    of blocks looks unique and one bucket of hashes overflows."""
    r = np.random.RandomState(seed)
    rows = r.randint(0, n, (k, n))
    acc = r.rand(n) < 0.5
    crowd = r.rand(n) < 0.4
    rows[:, crowd] = rows[:, :1]
    acc[crowd] = acc[0]
    return W.from_rows(rows.astype(np.uint32), acc, 3, f"crowd({n},{k})")


def _random(n, k, seed, every=0):
    d = W.random_dfa(n, k, seed)
    if every:
        d.accept = W.pack_accept(np.arange(n) % every == 0)
    return d


CASES = {
    "random3": lambda: _random(N, 3, 1), "random4": lambda: _random(N, 4, 2), "random4b": lambda: _random(3000017, 4, 3),
    "random3b": lambda: _random(4194304, 3, 4), "random5": lambda: _random(2097152, 5, 5),
    "random7": lambda: _random(2097153, 7, 6), "random2": lambda: _random(N, 2, 7), "random8": lambda: _random(N, 8, 8),
    "coarse4": lambda: _random(N + 1023, 4, 9, 97), "coarse5": lambda: _random(2500001, 5, 10, 97),
    "some copies 4": lambda: _redundant(3000000, 4, 2950000, 11), "some copies 5": lambda: _redundant(2100001, 5, 2080000, 12),
    "copies3": lambda: _redundant(4194305, 3, 262000, 13), "copies4": lambda: _redundant(3000000, 4, 1500000, 14),
    "stable after the labels": lambda: _redundant(N, 4, 16, 15), "one class": lambda: _random(N, 4, 16, 1),
    "crowd4": lambda: _crowd(N, 4, 17), "crowd4b": lambda: _crowd(3000000, 4, 18), "crowd6": lambda: _crowd(2200000, 6, 19), "copies6": lambda: _redundant(2100000, 6, 100000, 20),
}


def _both(ctx, monkeypatch, call):
    monkeypatch.setenv("DFAMIN_NO_LABELS", "4")
    want = call()
    monkeypatch.delenv("DFAMIN_NO_LABELS")
    return want, call()


@pytest.mark.parametrize("name", list(CASES))
def test_large(ctx, monkeypatch, name):
    from paper_2410_22764_amd import dfamin
    d = CASES[name]()
    print(f"[case] {name}: {d.n} states, {d.k} letters", flush=True)
    for opts in (dict(closure="auto"), dict(closure="off"), dict(closure="auto", auto_rounds=2, max_levels=1)):
        (a, ra), (b, rb) = _both(ctx, monkeypatch, lambda: dfamin.dfamin_minimize(ctx, d, opts))
        assert np.array_equal(a, b) and ra == rb, (opts, ra, rb)
    if name in ("random4", "some copies 5"):
        want, nb = oracle.hopcroft(d.n, d.k, d.delta, d.accept)
        assert rb["num_blocks"] == nb and np.array_equal(b, want)


@pytest.mark.parametrize("name", ["some copies 4", "some copies 5"])
def test_colliding_hashes_are_redone(monkeypatch, name):
    """The states left by a round of unique hashes meet weak hashes."""
    from paper_2410_22764_amd import dfamin
    d = CASES[name]()
    print(f"[case] weak hashes, {name}", flush=True)
    with dfamin.dfamin_create(0) as c:
        a, ra = dfamin.dfamin_minimize(c, d, "auto")
        monkeypatch.setenv("DFAMIN_HASH_BITS", "34")
        b, rb = dfamin.dfamin_minimize(c, d, "auto")
    assert np.array_equal(a, b) and ra == rb


@pytest.mark.parametrize("name", ["random4", "some copies 5", "copies4"])
def test_minimal_dfa(ctx, monkeypatch, name):
    from paper_2410_22764_amd import dfamin
    d = CASES[name]()
    print(f"[case] minimal DFA, {name}", flush=True)
    want, got = _both(ctx, monkeypatch, lambda: dfamin.dfamin_minimal_dfa(ctx, d, "auto"))
    assert want[0] == got[0] and want[3] == got[3]
    for i in (1, 2, 4):
        assert np.array_equal(want[i], got[i])
