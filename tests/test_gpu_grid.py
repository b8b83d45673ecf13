"""The grid kernel (one instance by co-resident workgroups) against the CPU
oracle and the round engine: same partition, round counts and closure levels.
Sizes sit at the edges of its tiles (1,024 states per workgroup and pass; 1,
2, 4 and 8 states per thread on 256 CUs)."""
import numpy as np
import pytest

import oracle
from paper_2410_22764_amd import dfamin, workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = dfamin.dfamin_create(0)
    yield c
    c.close()


def _both(ctx, d, monkeypatch, **opts):
    """The call as it is, and with the grid kernel turned off."""
    print(f"[case] {d.name} n={d.n} k={d.k} {opts}", flush=True)
    out, res = dfamin.dfamin_minimize(ctx, d, opts or None)
    monkeypatch.setenv("DFAMIN_GRID_MAX_STATES", "0")
    out2, res2 = dfamin.dfamin_minimize(ctx, d, opts or None)
    monkeypatch.delenv("DFAMIN_GRID_MAX_STATES")
    assert np.array_equal(out, out2)
    assert res == res2
    return out, res


def _check(ctx, d, monkeypatch, **opts):
    out, res = _both(ctx, d, monkeypatch, **opts)
    want, nb = oracle.hopcroft(d.n, d.k, d.delta, d.accept)
    assert np.array_equal(out, want) and res["num_blocks"] == nb and res["initial_block"] == want[d.q0]


def _redundant(n, k, classes, seed):
    """Every state copies a state of a random automaton."""
    r = np.random.RandomState(seed)
    cls = r.permutation(np.concatenate([np.arange(classes), r.randint(0, classes, n - classes)]))
    members = [np.nonzero(cls == c)[0] for c in range(classes)]
    base = r.randint(0, classes, (k, classes))
    rows = np.empty((k, n), np.uint32)
    for a in range(k):
        for c in range(classes):
            m = members[c]
            rows[a, m] = r.choice(members[base[a, c]], len(m))
    return W.from_rows(rows, r.rand(classes)[cls] < 0.5, int(r.randint(n)), f"redundant({n},{k},{classes})")


@pytest.mark.parametrize("n", [6145, 7168, 7169, 32769, 262144, 262145, 524289, 1048577])
@pytest.mark.parametrize("k", [2, 5])
def test_random(ctx, n, k, monkeypatch):
    _check(ctx, W.random_dfa(n, k, n + k), monkeypatch)


@pytest.mark.parametrize("closure", ["auto", "off", "on"])
@pytest.mark.parametrize("n,k,c", [(6200, 9, 400), (40001, 3, 5000), (300007, 2, 7)])
def test_redundant(ctx, n, k, c, closure, monkeypatch):
    _check(ctx, _redundant(n, k, c, n), monkeypatch, closure=closure)


@pytest.mark.parametrize("closure", ["auto", "on"])
@pytest.mark.parametrize("n", [6145, 7169, 30001, 270001])
def test_chains(ctx, n, closure, monkeypatch):
    _check(ctx, W.permuted_chain_dfa(n, 3, n), monkeypatch, closure=closure)


@pytest.mark.parametrize("opts", [dict(), dict(max_levels=3), dict(auto_rounds=2), dict(closure="off")])
def test_unary_and_deep(ctx, opts, monkeypatch):
    _check(ctx, W.fib_dfa(16), monkeypatch, **opts)
    _check(ctx, W.bitsplitter_dfa(13), monkeypatch, **opts)
    _check(ctx, W.random_dfa(7000, 1, 3), monkeypatch, **opts)


def test_many_letters(ctx, monkeypatch):
    """Alphabets around the chunks of letters whose loads go out together,
    the widest the kernel validates, and one too wide for it."""
    for k in (7, 8, 9, 32, 33):
        _check(ctx, _redundant(6500, k, 500, k), monkeypatch)


def test_degenerate(ctx, monkeypatch):
    n = 6500
    ident = np.tile(np.arange(n, dtype=np.uint32), (2, 1))
    for rows in (ident, (ident + 1) % n):
        for acc in (np.zeros(n, bool), np.ones(n, bool), np.arange(n) == n - 1, np.arange(n) % 2 == 0):
            _check(ctx, W.from_rows(rows, acc, 17), monkeypatch)


def test_refused_inputs_and_caps(ctx, monkeypatch):
    d = W.random_dfa(70001, 3, 1)
    d.delta[2 * d.n + 69999] = d.n
    for closure in ("auto", "on"):
        _, res = dfamin.dfamin_minimize(ctx, d, dict(closure=closure), check=False)
        assert res["rc"] == dfamin.DFAMIN_E_BAD_DFA and res["status"] == dfamin.DFAMIN_E_BAD_DFA
    c = W.chain_dfa(6200, 2)
    for cap in (1, 5, 12, 13, 14):
        got = dfamin.dfamin_minimize(ctx, c, dict(max_rounds=cap), check=False)[1]
        monkeypatch.setenv("DFAMIN_GRID_MAX_STATES", "0")
        assert dfamin.dfamin_minimize(ctx, c, dict(max_rounds=cap), check=False)[1] == got
        monkeypatch.delenv("DFAMIN_GRID_MAX_STATES")
    _check(ctx, W.random_dfa(70001, 3, 1), monkeypatch)  # the context goes on


def test_weak_hashes_are_redone(ctx, monkeypatch):
    """Few bits of hash: different signatures share one now and then, and
    the round is redone with another salt; with too few, every salt collides
    and the call gives up with an error."""
    d = _redundant(20000, 3, 1200, 5)
    want, nb = oracle.hopcroft(d.n, d.k, d.delta, d.accept)
    monkeypatch.setenv("DFAMIN_GRID_HASH_BITS", "20")
    for _ in range(3):
        out, res = dfamin.dfamin_minimize(ctx, d)
        assert np.array_equal(out, want) and res["num_blocks"] == nb
    monkeypatch.setenv("DFAMIN_GRID_HASH_BITS", "4")
    assert dfamin.dfamin_minimize(ctx, d, check=False)[1]["rc"] == dfamin.DFAMIN_E_INTERNAL
    monkeypatch.delenv("DFAMIN_GRID_HASH_BITS")
    _check(ctx, d, monkeypatch)


def test_minimal_dfa(ctx, monkeypatch):
    for d in (W.random_dfa(30001, 3, 2), _redundant(20001, 2, 3000, 9), W.permuted_chain_dfa(7000, 2, 1),
              W.bitsplitter_dfa(13)):
        print(f"[case] minimal {d.name}", flush=True)
        a = dfamin.dfamin_minimal_dfa(ctx, d)
        monkeypatch.setenv("DFAMIN_GRID_MAX_STATES", "0")
        b = dfamin.dfamin_minimal_dfa(ctx, d)
        monkeypatch.delenv("DFAMIN_GRID_MAX_STATES")
        assert a[0] == b[0] and a[3] == b[3]
        assert all(np.array_equal(a[i], b[i]) for i in (1, 2, 4))


def test_concurrent_calls(monkeypatch):
    """Several contexts at once: the workgroups of all grid kernels in flight
    never exceed the device; calls beyond that take the round engine."""
    import threading
    ds = [W.random_dfa(200003, 2, 1), W.permuted_chain_dfa(150001, 2, 2), W.random_dfa(9001, 3, 3),
          W.fib_dfa(18)]
    want = [oracle.hopcroft(d.n, d.k, d.delta, d.accept)[0] for d in ds]
    bad = []

    def work(i):
        with dfamin.dfamin_create(0) as c:
            for t in range(6):
                d = ds[(i + t) % len(ds)]
                out, _ = dfamin.dfamin_minimize(c, d)
                if not np.array_equal(out, want[(i + t) % len(ds)]):
                    bad.append((i, t))

    ts = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


def _shifts(n, steps, seed):
    """Letters q -> min(q + s, n - 1), one accepting state, ids shuffled:
    deep, with several letters that move."""
    q = np.arange(n)
    rows = np.stack([np.minimum(q + s, n - 1) for s in steps]).astype(np.uint32)
    return W.permute_dfa(W.from_rows(rows, q == n - 1), W.random_permutation(n, seed), f"shifts({n},{steps})")


@pytest.mark.parametrize("closure", ["on", "auto"])
@pytest.mark.parametrize("n,steps", [(120000, [1, 3, 5]), (60000, [1, 2, 3, 4]), (7000, [1, 7])])
def test_noalloc_holds_the_same_levels(ctx, n, steps, closure, monkeypatch):
    """In the fixed region the closure keeps as many levels with the grid
    kernel as with the round engine's rounds, and the results say so."""
    import torch
    d = _shifts(n, steps, n)
    delta = torch.from_numpy(d.delta.view(np.int32)).cuda()
    acc = torch.from_numpy(d.accept).cuda()
    got = []
    for grid in (True, False):
        if not grid:
            monkeypatch.setenv("DFAMIN_GRID_MAX_STATES", "0")
        print(f"[case] noalloc {d.name} {closure} grid={grid}", flush=True)
        out = torch.empty(n, dtype=torch.int32, device="cuda")
        r = dfamin.dfamin_minimize_device_noalloc(ctx, d.n, d.k, delta.data_ptr(), acc.data_ptr(), d.q0, out.data_ptr(),
                                                  opts=closure, stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        got.append((r, out.cpu().numpy()))
    assert got[0][0] == got[1][0]
    assert np.array_equal(got[0][1], got[1][1])
    assert np.array_equal(got[0][1], oracle.hopcroft(d.n, d.k, d.delta, d.accept)[0])


@pytest.mark.parametrize("n,k,tail", [(1 << 19, 4, 0), (400003, 3, 90)])
def test_wide_frontiers_leave_the_grid(ctx, n, k, tail, monkeypatch):
    """Reachability: wide levels run one launch each on all CUs, narrow ones
    (before, between and after them; a path long enough for closure rows)
    many to a launch; the same minimal DFA and level count as level by level."""
    r = np.random.RandomState(n)
    rows = r.randint(tail, n, (k, n)).astype(np.uint32)
    rows[:, :tail] = np.arange(1, tail + 1)  # a path into the wide part
    d = W.from_rows(rows, r.rand(n) < 0.5, 0, f"wide({n},{k},{tail})")
    print(f"[case] minimal {d.name}", flush=True)
    a = dfamin.dfamin_minimal_dfa(ctx, d)
    dfamin.dfamin_set_profiling(ctx, True)
    dfamin.dfamin_minimal_dfa(ctx, d)
    launches = {s["name"]: s["launches"] for s in dfamin.dfamin_get_kernel_stats(ctx)}["bfs_level"]
    dfamin.dfamin_set_profiling(ctx, False)
    monkeypatch.setenv("DFAMIN_GRID_MAX_STATES", "0")
    b = dfamin.dfamin_minimal_dfa(ctx, d)
    assert a[0] == b[0] and a[3] == b[3]
    assert all(np.array_equal(a[i], b[i]) for i in (1, 2, 4))
    assert 3 <= launches < a[3]["bfs_levels"]


def _grid_launches(ctx, call, name="grid"):
    dfamin.dfamin_set_profiling(ctx, True)
    got = call()
    n = sum(s["launches"] for s in dfamin.dfamin_get_kernel_stats(ctx) if s["name"] == name)
    dfamin.dfamin_set_profiling(ctx, False)
    return got, n


@pytest.mark.parametrize("mask", [1, 2, 3])
@pytest.mark.parametrize("d,closure", [(W.random_dfa(40001, 3, 1), "off"), (W.random_dfa(300007, 2, 2), "auto"),
                                       (W.permuted_chain_dfa(30001, 2, 3), "auto"), (W.bitsplitter_dfa(14), "auto"),
                                       (W.bitsplitter_dfa(13), "on")], ids=lambda x: getattr(x, "name", x))
def test_given_up_launches(d, closure, mask, monkeypatch):
    """A launch whose waits run out (the first, the one after the closure was
    built): the call ends as ever through the round engine, also in the fixed
    region, and the next launch finds its barrier in order."""
    import torch
    want, nb = oracle.hopcroft(d.n, d.k, d.delta, d.accept)
    delta = torch.from_numpy(d.delta.view(np.int32)).cuda()
    acc = torch.from_numpy(d.accept).cuda()
    with dfamin.dfamin_create(0) as c:
        for fn in (dfamin.dfamin_minimize_device, dfamin.dfamin_minimize_device_noalloc):
            def call():
                out = torch.full((d.n,), -1, dtype=torch.int32, device="cuda")
                r = fn(c, d.n, d.k, delta.data_ptr(), acc.data_ptr(), d.q0, out.data_ptr(), opts=closure,
                       stream=torch.cuda.current_stream().cuda_stream)
                torch.cuda.synchronize()
                return r, out.cpu().numpy()
            plain = call()
            monkeypatch.setenv("DFAMIN_GRID_ABORT", str(mask))
            print(f"[case] {fn.__name__} {d.name} {closure} launches {mask:b} given up", flush=True)
            given_up = call()
            monkeypatch.delenv("DFAMIN_GRID_ABORT")
            for r, out in (plain, given_up, call(), call(), call()):
                assert r == plain[0] and r["num_blocks"] == nb and np.array_equal(out, want)


def test_given_up_calls_are_remembered(monkeypatch):
    """After a call whose launch gave up, the next takes the round engine at
    once, after a second one in a row the next two, and so on; a launch that
    ends well puts that back."""
    d = W.random_dfa(40001, 3, 1)
    want = oracle.hopcroft(d.n, d.k, d.delta, d.accept)[0]
    launches = []
    with dfamin.dfamin_create(0) as c:
        for i in range(12):
            if i == 0:
                monkeypatch.setenv("DFAMIN_GRID_ABORT", "1")
            if i == 5:
                monkeypatch.delenv("DFAMIN_GRID_ABORT")
            (out, _), n = _grid_launches(c, lambda: dfamin.dfamin_minimize(c, d))
            assert np.array_equal(out, want)
            launches.append(n)
    assert launches == [1, 0, 1, 0, 0, 1, 1, 1, 1, 1, 1, 1]


@pytest.mark.parametrize("mask", [2, 4, 6])
def test_given_up_reachability(mask, monkeypatch):
    """The reachability kernel gives up in its first launch, and in the one
    after closure rows have joined: level by level from the start."""
    n = 20001
    q = np.arange(n)
    rows = np.stack([np.minimum(q + 1, n - 1), np.minimum(q + 2, n - 1)]).astype(np.uint32)
    for d in (W.random_dfa(30001, 3, 2), W.from_rows(rows, np.random.RandomState(1).rand(n) < 0.5, 0, "path")):
        with dfamin.dfamin_create(0) as c:
            a = dfamin.dfamin_minimal_dfa(c, d)
            monkeypatch.setenv("DFAMIN_GRID_ABORT", str(mask))
            print(f"[case] minimal {d.name}, launches {mask:b} given up", flush=True)
            b = dfamin.dfamin_minimal_dfa(c, d)
            monkeypatch.delenv("DFAMIN_GRID_ABORT")
            for x in (b, dfamin.dfamin_minimal_dfa(c, d), dfamin.dfamin_minimal_dfa(c, d)):
                assert a[0] == x[0] and a[3] == x[3]
                assert all(np.array_equal(a[i], x[i]) for i in (1, 2, 4))


def test_given_up_lanes(monkeypatch):
    """Requests whose lane gives up join the resident set."""
    ds = [W.random_dfa(20000 + 5000 * i, 2 + i % 3, i) for i in range(8)] + [W.permuted_chain_dfa(30000, 2, 9)]
    want = [oracle.hopcroft(d.n, d.k, d.delta, d.accept) for d in ds]
    with dfamin.dfamin_create(0) as c:
        for i in range(4):
            if i == 1:
                monkeypatch.setenv("DFAMIN_GRID_ABORT", "1")
            if i == 2:
                monkeypatch.delenv("DFAMIN_GRID_ABORT")
            print(f"[case] serving, lanes {'given up' if i == 1 else 'as ever'}", flush=True)
            tk = [dfamin.dfamin_submit(c, d, "auto") for d in ds]
            for t, d, (w, nb) in zip(tk, ds, want):
                rc, out, res = dfamin.dfamin_wait(c, t, d.n, timeout_us=60_000_000)
                assert rc == dfamin.DFAMIN_OK and res["num_blocks"] == nb and np.array_equal(out, w)


def test_largest_size(ctx, monkeypatch):
    """1,048,576 states on 256 CUs, the last size of the grid kernel."""
    _check(ctx, W.random_dfa(1048576, 2, 1), monkeypatch)
    _check(ctx, W.permuted_chain_dfa(1048576, 2, 2), monkeypatch)
