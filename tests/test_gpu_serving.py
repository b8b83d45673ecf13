"""Serving (continuous batching) through dfamin_submit / dfamin_wait / dfamin_cancel.

Every result must be identical alone and in any mix (tolerance 0: the output
is an exact integer partition) and identical to the CPU oracle.
"""
import hashlib
import json
import os
import time

import numpy as np
import pytest

import oracle
from paper_2410_22764_amd import workloads as W

pytestmark = pytest.mark.gpu

EXPECTED = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "expected_workloads.json")))


def digest(out):
    return hashlib.sha256(np.ascontiguousarray(out, dtype="<u4").tobytes()).hexdigest()[:32]


@pytest.fixture(scope="module")
def ctx():
    from paper_2410_22764_amd import dfamin
    c = dfamin.dfamin_create(0)
    yield c
    c.close()


def _mix(seed, count):
    rng = np.random.default_rng(seed)
    out = []
    for i in range(count):
        n = int(2 ** rng.uniform(4, 15))
        k = int(rng.integers(1, 7))
        kind = rng.choice(["random", "chain", "coarse"], p=[0.6, 0.2, 0.2])
        closure = ["off", "auto", "on"][i % 3]
        if kind == "chain":
            d = W.permuted_chain_dfa(n, k, seed * 1000 + i)
        else:
            d = W.random_dfa(n, k, seed * 1000 + i)
            if kind == "coarse":
                acc = np.zeros(n, bool)
                acc[:: 37] = True
                d.accept = W.pack_accept(acc)
        if kind == "chain" and closure == "off":
            closure = "auto"  # keep plain chain rounds bounded
        out.append((d, closure))
    return out


def test_mix_matches_alone_and_oracle(ctx):
    from paper_2410_22764_amd import dfamin
    reqs = _mix(1, 60)
    print("[case] serving mix of 60", flush=True)
    tickets = [dfamin.dfamin_submit(ctx, d, {"closure": c}) for d, c in reqs]
    for (d, c), t in zip(reqs, tickets):
        rc, out, res = dfamin.dfamin_wait(ctx, t, d.n, timeout_us=20_000_000)
        assert rc == dfamin.DFAMIN_OK, (d.name, rc)
        want, nb = oracle.hopcroft(d.n, d.k, d.delta, d.accept)
        assert res["num_blocks"] == nb and np.array_equal(out, want), d.name
        alone, ra = dfamin.dfamin_minimize(ctx, d, {"closure": c})
        assert np.array_equal(alone, out)
        assert ra["refine_rounds"] == res["refine_rounds"], d.name
        assert res["initial_block"] == want[d.q0]


def test_staggered_arrivals(ctx):
    """Requests submitted while others are resident join the running set."""
    from paper_2410_22764_amd import dfamin
    reqs = _mix(2, 40)
    print("[case] serving staggered", flush=True)
    tickets = []
    for i, (d, c) in enumerate(reqs):
        tickets.append(dfamin.dfamin_submit(ctx, d, {"closure": c}))
        if i % 5 == 0:
            time.sleep(0.002)
    for (d, c), t in zip(reqs, tickets):
        rc, out, res = dfamin.dfamin_wait(ctx, t, d.n)
        assert rc == dfamin.DFAMIN_OK
        want, nb = oracle.hopcroft(d.n, d.k, d.delta, d.accept)
        assert np.array_equal(out, want)


def test_short_request_overtakes_long_one(ctx):
    """Continuous batching: a short request that arrives after a long one
    finishes while the long one is still refining."""
    from paper_2410_22764_amd import dfamin
    long = W.chain_dfa(20000, 1)  # closure off: ~20000 rounds
    short = W.random_dfa(500, 2, 7)
    print("[case] serving overtake", flush=True)
    tl = dfamin.dfamin_submit(ctx, long, {"closure": "off"})
    time.sleep(0.01)
    ts = dfamin.dfamin_submit(ctx, short, None)
    rc, out, res = dfamin.dfamin_wait(ctx, ts, short.n, timeout_us=30_000_000)
    assert rc == dfamin.DFAMIN_OK
    rc_long, _, _ = dfamin.dfamin_wait(ctx, tl, long.n, timeout_us=0)
    assert rc_long == dfamin.DFAMIN_E_TIMEOUT  # still on the device
    rc_long, out_long, res_long = dfamin.dfamin_wait(ctx, tl, long.n)
    assert rc_long == dfamin.DFAMIN_OK
    assert np.array_equal(out_long, np.arange(long.n)) and res_long["refine_rounds"] == long.n - 2
    want, _ = oracle.hopcroft(short.n, short.k, short.delta, short.accept)
    assert np.array_equal(out, want)


def test_cancel_and_errors(ctx):
    from paper_2410_22764_amd import dfamin
    print("[case] serving cancel", flush=True)
    long = W.chain_dfa(20000, 1)
    t = dfamin.dfamin_submit(ctx, long, {"closure": "off"})
    time.sleep(0.01)
    assert dfamin.dfamin_cancel(ctx, t) == dfamin.DFAMIN_OK
    rc, out, _ = dfamin.dfamin_wait(ctx, t, long.n)
    assert rc == dfamin.DFAMIN_E_CANCELLED and out is None
    assert dfamin.dfamin_cancel(ctx, 10 ** 12) == dfamin.DFAMIN_E_INVAL
    bad = W.random_dfa(100, 2, 1)
    bad.delta = bad.delta.copy()
    bad.delta[3] = 100
    t = dfamin.dfamin_submit(ctx, bad, None)
    rc, _, _ = dfamin.dfamin_wait(ctx, t, bad.n)
    assert rc == dfamin.DFAMIN_E_BAD_DFA
    # the loop keeps serving afterwards
    d = W.random_dfa(300, 3, 2)
    t = dfamin.dfamin_submit(ctx, d, None)
    rc, out, _ = dfamin.dfamin_wait(ctx, t, d.n)
    want, _ = oracle.hopcroft(d.n, d.k, d.delta, d.accept)
    assert rc == dfamin.DFAMIN_OK and np.array_equal(out, want)


def test_pageable_staging_when_pinned_cap_is_zero(monkeypatch):
    """With the page-locked staging pool capped at 0 bytes every request is
    staged in ordinary host memory; results are unchanged."""
    from paper_2410_22764_amd import dfamin
    monkeypatch.setenv("DFAMIN_SERVING_PINNED_BYTES", "0")
    c = dfamin.dfamin_create(0)
    try:
        reqs = _mix(7, 12)
        print("[case] serving mix of 12, pageable staging", flush=True)
        tickets = [dfamin.dfamin_submit(c, d, {"closure": cl}) for d, cl in reqs]
        for (d, cl), t in zip(reqs, tickets):
            rc, out, res = dfamin.dfamin_wait(c, t, d.n, timeout_us=20_000_000)
            assert rc == dfamin.DFAMIN_OK, (d.name, rc)
            want, nb = oracle.hopcroft(d.n, d.k, d.delta, d.accept)
            assert res["num_blocks"] == nb and np.array_equal(out, want), d.name
    finally:
        c.close()


def test_serving_pool_at_full_sizes_bit_exact(ctx):
    """Requests of the serving workload at its own sizes (n up to 2^22,
    |Sigma| up to 16, permuted chains of over 2^20 states among them), all
    submitted at once so that they share the device: every result equals
    the oracle's (digest, block count, initial block, written by the golden
    script with the CPU oracle only) and the same DFA minimised alone."""
    from paper_2410_22764_amd import dfamin
    exp = EXPECTED["serving_pool"]
    _, specs = W.serving_stream(exp["seed"], exp["draws"], 1.0)
    reqs = exp["requests"]
    assert any(e["n"] >= 1 << 20 and e["k"] == 16 for e in reqs)
    assert any(e["kind"] == "chain" and e["n"] >= 1 << 20 for e in reqs)
    print(f"[case] serving pool of {len(reqs)} at full sizes: generating", flush=True)
    pool = [W.make_request(specs[e["index"]]) for e in reqs]
    print("[case] serving pool: submitting all", flush=True)
    tickets = [dfamin.dfamin_submit(ctx, d, "auto") for d in pool]
    mixed = []
    for d, e, t in zip(pool, reqs, tickets):
        assert (d.n, d.k) == (e["n"], e["k"])
        rc, out, res = dfamin.dfamin_wait(ctx, t, d.n, timeout_us=60_000_000)
        assert rc == dfamin.DFAMIN_OK, (e, rc)
        assert res["num_blocks"] == e["num_blocks"] and res["initial_block"] == e["initial_block"], e
        assert digest(out) == e["sha"], e
        mixed.append((digest(out), res["refine_rounds"]))
    print("[case] serving pool: each request alone", flush=True)
    for d, e, (dg, rr) in zip(pool, reqs, mixed):
        alone, ra = dfamin.dfamin_minimize(ctx, d, "auto")
        assert digest(alone) == dg and ra["refine_rounds"] == rr, e


def test_doubling_requests_report_as_alone(ctx):
    """Chains under AUTO refine by doubling, in the fused kernel (up to
    16,384 states) or in the resident set: each request's round count and
    closure levels (the highest level a splitting round read) are those of
    the same DFA minimised alone."""
    from paper_2410_22764_amd import dfamin
    ds = [W.permuted_chain_dfa(n, k, n + k) for n, k in [(3, 2), (900, 2), (16384, 3), (16385, 2), (70000, 4)]]
    ds.append(W.random_dfa(3000, 1, 5))
    print("[case] serving doubling requests", flush=True)
    tickets = [dfamin.dfamin_submit(ctx, d, "auto") for d in ds]
    for d, t in zip(ds, tickets):
        rc, out, res = dfamin.dfamin_wait(ctx, t, d.n, timeout_us=20_000_000)
        assert rc == dfamin.DFAMIN_OK, d.name
        alone, ra = dfamin.dfamin_minimize(ctx, d, "auto")
        assert np.array_equal(alone, out), d.name
        for f in ("num_blocks", "initial_block", "refine_rounds", "rounds_executed", "closure_levels",
                  "closure_letters"):
            assert res[f] == ra[f], (d.name, f, res, ra)


def _double_step_chain(n, seed):
    """A chain on which both letters move forward (one or two states): two
    non-identity letters, about n/2 plain rounds, so AUTO gives it the
    closure after its first rounds."""
    ids = np.arange(n, dtype=np.uint32)
    rows = np.stack([np.minimum(ids + 1, n - 1), np.minimum(ids + 2, n - 1)])
    acc = np.zeros(n, bool)
    acc[n - 1] = True
    d = W.from_rows(rows, acc, 0, f"double-step chain(n={n})")
    return W.permute_dfa(d, W.random_permutation(n, seed), f"double-step chain(n={n},seed={seed})")


def test_small_budget_deep_auto_requests():
    """A context whose HBM budget leaves the serving loop a few MB: deep
    requests with two non-identity letters under AUTO all come due for the
    closure at once, and a unary chain refines by doubling beside them.
    Level storage runs short (a closure then keeps the levels it has), and a
    request whose signature records for the new letter count do not fit
    keeps refining on its plain letters: every request still ends with the
    oracle's partition, none fails."""
    from paper_2410_22764_amd import dfamin
    c = dfamin.dfamin_create(0, hbm_budget_bytes=8 << 20)
    try:
        ds = [_double_step_chain(6000, 31 + i) for i in range(10)]
        ds.append(W.permuted_chain_dfa(6000, 2, 41))
        print(f"[case] serving {len(ds)} deep requests under an 8 MB budget", flush=True)
        tickets = [dfamin.dfamin_submit(c, d, "auto") for d in ds]
        for d, t in zip(ds, tickets):
            rc, out, res = dfamin.dfamin_wait(c, t, d.n, timeout_us=60_000_000)
            assert rc == dfamin.DFAMIN_OK, (d.name, rc)
            want, nb = oracle.hopcroft(d.n, d.k, d.delta, d.accept)
            assert res["num_blocks"] == nb and np.array_equal(out, want) and res["initial_block"] == want[d.q0]
    finally:
        c.close()


def test_small_request_batches_beside_rounds(ctx):
    """Small requests run as fused batches on their own stream while the
    resident set refines: a burst of them around a long request, every
    fourth cancelled right after its submit, one invalid and one that the
    fused kernel hands back (two non-identity letters, still splitting after
    the AUTO rounds), which then joins the resident set and takes closure
    letters.  Each result is the oracle's, a cancelled request reports
    success or cancellation, the invalid one E_BAD_DFA."""
    from paper_2410_22764_amd import dfamin
    print("[case] serving: small-request batches beside a long request", flush=True)
    long = W.chain_dfa(3000, 1)
    tl = dfamin.dfamin_submit(ctx, long, {"closure": "off"})  # one round per state
    small = [W.random_dfa(200 + 300 * i, 2 + i % 5, 100 + i) for i in range(48)]
    n = 3000
    ids = np.arange(n)
    rows = np.stack([np.minimum(ids + 1, n - 1), np.minimum(ids + 2, n - 1)])
    acc = np.zeros(n, bool)
    acc[-1] = True
    deep = W.from_rows(rows, acc, 0, "two-letter chain")
    bad = W.random_dfa(500, 2, 7)
    bad.delta = bad.delta.copy()
    bad.delta[10] = 500
    tickets, cancelled = [], set()
    for i, d in enumerate(small):
        t = dfamin.dfamin_submit(ctx, d, {"closure": "auto"})
        tickets.append(t)
        if i % 4 == 1:
            assert dfamin.dfamin_cancel(ctx, t) == dfamin.DFAMIN_OK
            cancelled.add(i)
    td = dfamin.dfamin_submit(ctx, deep, {"closure": "auto"})
    tb = dfamin.dfamin_submit(ctx, bad, {"closure": "auto"})
    for i, (d, t) in enumerate(zip(small, tickets)):
        rc, out, res = dfamin.dfamin_wait(ctx, t, d.n, timeout_us=30_000_000)
        if i in cancelled and rc == dfamin.DFAMIN_E_CANCELLED:
            continue
        assert rc == dfamin.DFAMIN_OK, (i, rc)
        want, nb = oracle.hopcroft(d.n, d.k, d.delta, d.accept)
        assert res["num_blocks"] == nb and np.array_equal(out, want), i
    rc, out, res = dfamin.dfamin_wait(ctx, td, deep.n, timeout_us=30_000_000)
    want, nb = oracle.hopcroft(deep.n, deep.k, deep.delta, deep.accept)
    assert rc == dfamin.DFAMIN_OK and res["num_blocks"] == nb and np.array_equal(out, want)
    assert res["closure_levels"] > 0  # handed back by the fused kernel, closure built by the loop
    rc, _, _ = dfamin.dfamin_wait(ctx, tb, bad.n, timeout_us=30_000_000)
    assert rc == dfamin.DFAMIN_E_BAD_DFA
    rc, out, res = dfamin.dfamin_wait(ctx, tl, long.n, timeout_us=60_000_000)
    assert rc == dfamin.DFAMIN_OK and np.array_equal(out, np.arange(long.n))


def test_larger_requests_on_lanes(monkeypatch):
    """Requests above 16,384 states run on the grid kernel, one per lane: the
    results are those of the resident set (DFAMIN_GRID_MAX_STATES=0) and the
    oracle's, for requests that finish there, that need closure letters, more
    rounds than a lane runs, or a round count that takes AUTO's letters at the
    end; invalid and cancelled ones are reported as ever."""
    from paper_2410_22764_amd import dfamin
    reqs = [(W.random_dfa(n, k, n), {"closure": c}) for n, k, c in
            ((16385, 2, "auto"), (65536, 9, "auto"), (65537, 1, "auto"), (100003, 3, "off"), (262145, 2, "auto"),
             (20000, 32, "auto"), (20000, 33, "auto"), (40000, 2, "on"))]
    reqs += [(W.permuted_chain_dfa(n, k, n), {"closure": "auto"}) for n, k in ((16390, 2), (120000, 5))]
    reqs += [(_double_step_chain(17000, 3), {"closure": "auto"}), (W.bitsplitter_dfa(15), {"closure": "auto"}),
             (W.bitsplitter_dfa(15), {"closure": "off"}), (W.chain_dfa(16400, 1), {"closure": "auto", "max_levels": 3})]
    reqs += [(W.random_dfa(50000, 2, 5), {"closure": "auto", "auto_rounds": r}) for r in (1, 2, 3, 4, 5)]
    n = 17001  # more plain rounds than a lane runs, few enough for the resident set
    ids = np.arange(n)
    step = W.from_rows(np.minimum(ids + 100, n - 1).astype(np.uint32)[None], ids == n - 1, 7, "step chain")
    reqs.append((step, {"closure": "off"}))
    bad = W.random_dfa(30000, 2, 7)
    bad.delta = bad.delta.copy()
    bad.delta[12345] = bad.n
    gone = W.random_dfa(60000, 3, 8)
    ends = []
    for off in (True, False):
        if off:
            monkeypatch.setenv("DFAMIN_GRID_MAX_STATES", "0")
        else:
            monkeypatch.delenv("DFAMIN_GRID_MAX_STATES")
        print(f"[case] serving {len(reqs) + 2} larger requests, lanes {'off' if off else 'on'}", flush=True)
        with dfamin.dfamin_create(0) as c:
            tk = [dfamin.dfamin_submit(c, d, o) for d, o in reqs]
            tb, tg = dfamin.dfamin_submit(c, bad, "auto"), dfamin.dfamin_submit(c, gone, "auto")
            dfamin.dfamin_cancel(c, tg)
            ends.append([dfamin.dfamin_wait(c, t, d.n, timeout_us=60_000_000) for t, (d, _) in zip(tk, reqs)])
            assert dfamin.dfamin_wait(c, tb, bad.n, timeout_us=60_000_000)[0] == dfamin.DFAMIN_E_BAD_DFA
            assert dfamin.dfamin_wait(c, tg, gone.n, timeout_us=60_000_000)[0] in (
                dfamin.DFAMIN_OK, dfamin.DFAMIN_E_CANCELLED)
    for (d, o), (r0, o0, s0), (r1, o1, s1) in zip(reqs, *ends):
        assert r0 == r1 == dfamin.DFAMIN_OK, (d.name, o)
        assert np.array_equal(o0, o1) and s0 == s1, (d.name, o, s0, s1)
        want, nb = oracle.hopcroft(d.n, d.k, d.delta, d.accept)
        assert s1["num_blocks"] == nb and np.array_equal(o1, want) and s1["initial_block"] == want[d.q0], (d.name, o)


def test_lanes_of_several_contexts():
    """Two serving contexts and a thread of single calls share the CUs."""
    import threading
    from paper_2410_22764_amd import dfamin
    ds = [W.random_dfa(20000 + 9000 * i, 2 + i % 3, i) for i in range(12)]
    want = [oracle.hopcroft(d.n, d.k, d.delta, d.accept)[0] for d in ds]
    print("[case] two serving contexts and single calls", flush=True)
    errs = []

    def serve():
        try:
            with dfamin.dfamin_create(0) as c:
                for _ in range(3):
                    tk = [dfamin.dfamin_submit(c, d, "auto") for d in ds]
                    for t, d, w in zip(tk, ds, want):
                        rc, out, _ = dfamin.dfamin_wait(c, t, d.n, timeout_us=60_000_000)
                        assert rc == dfamin.DFAMIN_OK and np.array_equal(out, w), d.name
        except Exception as e:  # reported by the main thread
            errs.append(repr(e))

    def single():
        try:
            with dfamin.dfamin_create(0) as c:
                for _ in range(3):
                    for d, w in zip(ds, want):
                        assert np.array_equal(dfamin.dfamin_minimize(c, d, "auto")[0], w), d.name
        except Exception as e:
            errs.append(repr(e))

    ts = [threading.Thread(target=f) for f in (serve, serve, single)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errs, errs


def _copied_chain(n, length, seed, k=1):
    """Every state copies one of a chain of `length` states: `length` rounds of
    n active states."""
    r = np.random.RandomState(seed)
    cls = r.permutation(np.concatenate([np.arange(length)] * 2 + [r.randint(0, length, n - 2 * length)]))
    order = np.argsort(cls, kind="stable")
    size = np.bincount(cls, minlength=length)
    nxt = np.minimum(cls + 1, length - 1)
    pick = (r.rand(n) * size[nxt]).astype(np.int64)
    row = order[(np.cumsum(size) - size)[nxt] + pick].astype(np.uint32)
    rows = np.concatenate([row[None], np.tile(np.arange(n, dtype=np.uint32), (k - 1, 1))])
    return W.from_rows(rows, cls == length - 1, 0, f"copied chain({n},{length})"), cls

def test_many_requests_beside_a_long_one(ctx):
    """A large request is resident for thirty rounds; three hundred smaller
    ones must not wait for a lane each round of it, but share its rounds (or
    lanes seen to during them), and be done about when it is."""
    from paper_2410_22764_amd import dfamin
    length = 30
    long, cls = _copied_chain(1 << 22, length, 1)
    first = np.unique(cls, return_index=True)[1]
    rank = np.empty(length, np.int64)
    rank[np.argsort(first)] = np.arange(length)
    ds = [W.random_dfa(17000 + 10 * i, 2, i) for i in range(10)]
    want = [oracle.hopcroft(d.n, d.k, d.delta, d.accept)[0] for d in ds]
    for _ in range(2):  # (the first pass fills the pools)
        print("[case] serving: 300 requests beside a long one", flush=True)
        tl = dfamin.dfamin_submit(ctx, long, {"closure": "off"})
        tk = [dfamin.dfamin_submit(ctx, ds[i % 10], "auto") for i in range(300)]
        rc, out, res = dfamin.dfamin_wait(ctx, tl, long.n, timeout_us=60_000_000)
        ends = [dfamin.dfamin_wait(ctx, t, ds[i % 10].n, timeout_us=0) for i, t in enumerate(tk)]
        late = [i for i, e in enumerate(ends) if e[0] == dfamin.DFAMIN_E_TIMEOUT]
        for i in late:
            ends[i] = dfamin.dfamin_wait(ctx, tk[i], ds[i % 10].n, timeout_us=60_000_000)
        for i, (r, o, _) in enumerate(ends):
            assert r == dfamin.DFAMIN_OK and np.array_equal(o, want[i % 10]), i
        assert rc == dfamin.DFAMIN_OK and res["num_blocks"] == length and res["refine_rounds"] == length - 2
        assert np.array_equal(out, rank[cls])
    assert len(late) <= 60, len(late)


def test_cancelled_while_waiting_for_a_lane(ctx):
    """A cancelled request that waits for a lane ends as cancelled without
    being looked at: these are invalid, and would otherwise say so."""
    from paper_2410_22764_amd import dfamin
    good = _copied_chain(20000, 60, 1)[0]
    bad = W.random_dfa(20000, 1, 2)
    bad.delta = bad.delta.copy()
    bad.delta[777] = bad.n
    print("[case] serving: 300 requests for lanes, the last 10 cancelled", flush=True)
    tk = [dfamin.dfamin_submit(ctx, good, {"closure": "off"}) for _ in range(290)]
    tb = [dfamin.dfamin_submit(ctx, bad, {"closure": "off"}) for _ in range(10)]
    time.sleep(0.005)  # admitted, their inputs on the device
    for t in tb:
        dfamin.dfamin_cancel(ctx, t)
    for t in tb:
        assert dfamin.dfamin_wait(ctx, t, bad.n, timeout_us=60_000_000)[0] == dfamin.DFAMIN_E_CANCELLED
    for t in tk:
        rc, _, res = dfamin.dfamin_wait(ctx, t, good.n, timeout_us=60_000_000)
        assert rc == dfamin.DFAMIN_OK and res["num_blocks"] == 60
