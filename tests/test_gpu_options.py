"""GPU tests of the options and error paths: the default closure policy, the
memory-capped closure (a context's HBM budget, max_levels, auto_rounds),
E_NOMEM, and outputs left untouched on E_BAD_DFA.

The partition must always equal the oracle's; round counts follow from the
oracle's Moore partitions and closure levels (Section 3.4: every closure
letter is a word over Sigma, so any subset of levels gives the same classes
and only the number of rounds changes).
"""
import numpy as np
import pytest

import oracle
from paper_2410_22764_amd import workloads as W

pytestmark = pytest.mark.gpu

SENTINEL = 0x5A5A5A5A


@pytest.fixture(scope="module")
def ctx():
    from paper_2410_22764_amd import dfamin
    c = dfamin.dfamin_create(0)
    yield c
    c.close()


def shift_dfa(n, shifts, name):
    """Letter s sends i to min(i + s, n - 1); only state n - 1 accepts.  With
    several shifts every letter is a non-identity letter (no doubling), and
    plain refinement needs about n / max(shift) rounds."""
    ids = np.arange(n, dtype=np.int64)
    rows = np.stack([np.minimum(ids + s, n - 1) for s in shifts]).astype(np.uint32)
    acc = np.zeros(n, bool)
    acc[n - 1] = True
    return W.from_rows(rows, acc, name=name)


def _hop(d):
    return oracle.hopcroft(d.n, d.k, d.delta, d.accept)


def test_null_options_mean_auto(ctx):
    """A NULL options pointer and a zeroed struct select closure AUTO: on a
    chain (one non-identity letter) the rounds double from the first one,
    ceil(log2(n - 1)) of them instead of the n - 2 of plain refinement."""
    from paper_2410_22764_amd import dfamin
    d = W.permuted_chain_dfa(5000, 3, 17)
    print("[case] NULL options on a 5000-state chain", flush=True)
    a, ra = dfamin.dfamin_minimize(ctx, d, None)
    z, rz = dfamin.dfamin_minimize(ctx, d, dfamin.Opts())
    e, re = dfamin.dfamin_minimize(ctx, d, "auto")
    assert np.array_equal(a, np.arange(d.n)) and np.array_equal(z, a) and np.array_equal(e, a)
    assert ra == rz == re
    assert ra["refine_rounds"] == 13 and ra["closure_levels"] > 0


def test_max_levels_caps_the_closure(ctx):
    """max_levels = 3: closure ON builds levels 0..3 only, and the rounds are
    Moore's on the closure automaton with L = 3; AUTO on a unary instance
    doubles with steps of at most 2^3."""
    from paper_2410_22764_amd import dfamin
    d = shift_dfa(3000, [1, 3], "shift(1,3) n=3000")
    want, nb = _hop(d)
    print("[case] max_levels=3, closure on", flush=True)
    out, r = dfamin.dfamin_minimize(ctx, d, dict(closure="on", max_levels=3))
    _, _, rr = oracle.moore_closure(d.n, d.k, d.delta, d.accept, L=3)
    assert np.array_equal(out, want) and r["num_blocks"] == nb
    assert r["closure_levels"] == 3 and r["refine_rounds"] == rr
    c = W.chain_dfa(3000, 2)
    print("[case] max_levels=3, AUTO on a chain", flush=True)
    out, r = dfamin.dfamin_minimize(ctx, c, dict(closure="auto", max_levels=3))
    assert np.array_equal(out, np.arange(c.n))
    # doubling with t = 2^min(floor(log2(j+1)), 3): P_j for j = 0, 1, 3, 7, 15, 23, ...
    j = r_want = 0
    while j < c.n - 2:
        j += 2 ** min(oracle.floor_log2(j + 1), 3)
        r_want += 1
    assert r["refine_rounds"] == r_want and r["closure_levels"] == 3


@pytest.mark.parametrize("auto_rounds", [0, 3, 5])
def test_auto_rounds_before_the_closure(ctx, auto_rounds):
    """A deep instance with two non-identity letters under AUTO: plain rounds
    until auto_rounds (0 = the default, 8), then the closure's letters from
    that partition on.  r* = A + Moore's refining rounds on the closure
    automaton started from P_A."""
    from paper_2410_22764_amd import dfamin
    d = shift_dfa(4000, [1, 2], "shift(1,2) n=4000")
    A = auto_rounds or 8
    print(f"[case] auto_rounds={auto_rounds}", flush=True)
    out, r = dfamin.dfamin_minimize(ctx, d, dict(closure="auto", auto_rounds=auto_rounds))
    want, nb = _hop(d)
    assert np.array_equal(out, want) and r["num_blocks"] == nb
    pa, _, ra = oracle.moore_partial(d.n, d.k, d.delta, d.accept, A)
    assert ra == A  # still refining after A rounds
    L = oracle.floor_log2(d.n)
    rows = oracle.closure(d.n, d.k, d.delta, L)
    _, _, rc = oracle.moore_from(d.n, rows.shape[0], rows.reshape(-1), pa)
    assert r["refine_rounds"] == A + rc
    assert r["closure_levels"] > 0


def test_hbm_budget_caps_the_closure_and_reports_nomem():
    """Closure storage is capped at half of a context's remaining budget.
    Over a range of budgets each call either fails with E_NOMEM or returns
    the oracle's partition with L' <= floor(log2 n) closure levels and
    exactly the rounds of Moore's refinement on the closure cut at L'.  Some
    budget must stop the closure early, a large one must build every level,
    and a budget below the base buffers must give E_NOMEM."""
    from paper_2410_22764_amd import dfamin
    d = shift_dfa(20000, [1, 7, 31, 127], "shift(1,7,31,127) n=20000")
    want, nb = _hop(d)
    L = oracle.floor_log2(d.n)
    rounds_at = {}
    seen = {"nomem": 0, "capped": 0, "full": 0}
    for mib in [64, 32, 16, 12, 10, 8, 7, 6, 5, 4, 3, 2, 1, 0.25]:
        budget = int(mib * (1 << 20))
        print(f"[case] closure on, budget {budget} bytes", flush=True)
        with dfamin.dfamin_create(0, budget) as c:
            out, r = dfamin.dfamin_minimize(c, d, "on", check=False)
        if r["rc"] == dfamin.DFAMIN_E_NOMEM:
            seen["nomem"] += 1
            continue
        assert r["rc"] == dfamin.DFAMIN_OK, (mib, r)
        assert np.array_equal(out, want) and r["num_blocks"] == nb, mib
        lv = r["closure_levels"]
        assert lv <= L
        if lv not in rounds_at:
            rounds_at[lv] = oracle.moore_closure(d.n, d.k, d.delta, d.accept, L=lv)[2]
        assert r["refine_rounds"] == rounds_at[lv], (mib, lv)
        seen["full" if lv == L else "capped"] += 1
    assert seen["full"] and seen["capped"] and seen["nomem"], seen


def test_bad_dfa_leaves_device_outputs_untouched(ctx):
    """E_BAD_DFA is found on the device before anything is written: a
    sentinel-filled output stays as it was, alone and in a batch (where no
    instance is minimized when one is bad)."""
    import torch
    from paper_2410_22764_amd import dfamin
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream().cuda_stream
    for n, k in [(300, 2), (5000, 3), (70000, 2)]:
        d = W.random_dfa(n, k, n)
        delta = torch.from_numpy(d.delta.view(np.int32)).to(dev)
        delta[(k - 1) * n + n // 3] = n  # letter k-1, state n/3: out of range
        accept = torch.from_numpy(d.accept).to(dev)
        out = torch.full((n,), SENTINEL, dtype=torch.int32, device=dev)
        print(f"[case] bad DFA n={n} device entry", flush=True)
        r = dfamin.dfamin_minimize_device(ctx, n, k, delta.data_ptr(), accept.data_ptr(), 0, out.data_ptr(),
                                          stream=stream, check=False)
        torch.cuda.synchronize()
        assert r["rc"] == dfamin.DFAMIN_E_BAD_DFA
        assert bool((out == SENTINEL).all())
    good = [W.random_dfa(n, 2, n + 1) for n in (100, 4000, 30000)]
    bad = W.random_dfa(2000, 3, 9)
    bad.delta = bad.delta.copy()
    bad.delta[-1] = 2000
    ds = good[:2] + [bad] + good[2:]
    tens = [(torch.from_numpy(x.delta.view(np.int32)).to(dev), torch.from_numpy(x.accept).to(dev)) for x in ds]
    outs = [torch.full((x.n,), SENTINEL, dtype=torch.int32, device=dev) for x in ds]
    specs = [(x.n, x.k, t[0].data_ptr(), t[1].data_ptr(), x.q0) for x, t in zip(ds, tens)]
    print("[case] bad DFA in a device batch", flush=True)
    res = dfamin.dfamin_minimize_batch_device(ctx, specs, [o.data_ptr() for o in outs], stream=stream, check=False)
    torch.cuda.synchronize()
    assert res[0]["rc"] == dfamin.DFAMIN_E_BAD_DFA
    assert [r["status"] for r in res] == [0, 0, dfamin.DFAMIN_E_BAD_DFA, 0]
    for o in outs:
        assert bool((o == SENTINEL).all())
    # host entry point: the caller's buffer keeps its contents too
    h = np.full(bad.n, SENTINEL, np.uint32)
    s, keep = dfamin._host_dfa(bad)
    rr = dfamin.Result()
    rc = dfamin.load().dfamin_minimize(ctx.handle, dfamin.ctypes.byref(s), None, h.ctypes.data,
                                       dfamin.ctypes.byref(rr))
    assert rc == dfamin.DFAMIN_E_BAD_DFA and bool((h == SENTINEL).all())


def test_small_budgets_take_calls_in_a_row():
    """One context of a small budget: what the kernels of one call keep gives
    way to the next call's needs.  Every call here fits its budget in a context
    of its own, and has to in this one, in any order, with the same partition."""
    from paper_2410_22764_amd import dfamin
    ds = [W.random_dfa(300000, 2, 1), W.random_dfa(100000, 12, 1), W.permuted_chain_dfa(200000, 2, 1),
          shift_dfa(20000, [1, 7], "shift(1,7) n=20000")]
    want = [oracle.hopcroft(d.n, d.k, d.delta, d.accept) for d in ds]
    batch = [W.random_dfa(17000 + 13 * i, 3, i) for i in range(60)]
    bwant = [oracle.hopcroft(d.n, d.k, d.delta, d.accept)[0] for d in batch]
    for mib in (72, 128, 176):
        with dfamin.dfamin_create(0, mib << 20) as c:
            for t in range(3):
                for i in (0, 1, 2, 3) if t % 2 == 0 else (1, 0, 3, 2):
                    d = ds[i]
                    print(f"[case] budget {mib} MiB, pass {t}: {d.name} n={d.n} k={d.k}", flush=True)
                    out, r = dfamin.dfamin_minimize(c, d, "auto", check=False)
                    if mib < 100 and i == 1 and r["rc"] == dfamin.DFAMIN_E_NOMEM:
                        continue  # (its buffers beside the largest call's)
                    assert r["rc"] == dfamin.DFAMIN_OK, (mib, t, i, r)
                    assert np.array_equal(out, want[i][0]) and r["num_blocks"] == want[i][1]
                if mib >= 176:
                    print(f"[case] budget {mib} MiB, pass {t}: batch of {len(batch)}", flush=True)
                    outs, _ = dfamin.dfamin_minimize_batch(c, batch, "auto")
                    for o, w in zip(outs, bwant):
                        assert np.array_equal(o, w)


def test_small_budget_after_calls_that_did_not_fit():
    """64 MiB: a chain of 200,000 states has room after other calls, some of
    which may have been refused."""
    from paper_2410_22764_amd import dfamin
    ds = [(W.random_dfa(100000, 12, 1), True), (shift_dfa(60000, [1, 7], "shift(1,7) n=60000"), True),
          (W.random_dfa(300000, 2, 1), False), (W.permuted_chain_dfa(200000, 2, 1), True)]
    with dfamin.dfamin_create(0, 64 << 20) as c:
        for d, fits in ds:
            want, nb = oracle.hopcroft(d.n, d.k, d.delta, d.accept)
            for closure in ("auto", "on"):
                print(f"[case] budget 64 MiB: {d.name} closure {closure}", flush=True)
                out, r = dfamin.dfamin_minimize(c, d, closure, check=False)
                assert r["rc"] == dfamin.DFAMIN_OK or (not fits and r["rc"] == dfamin.DFAMIN_E_NOMEM), (d.name, closure, r)
                if r["rc"] == dfamin.DFAMIN_OK:
                    assert np.array_equal(out, want) and r["num_blocks"] == nb


@pytest.mark.parametrize("mib", [22, 24.66, 30, 40])
def test_small_budget_keeps_the_levels_of_the_round_engine(mib, monkeypatch):
    """A deep instance of sixteen letters under AUTO: no fewer closure levels
    with the grid kernel than with the round engine's rounds."""
    from paper_2410_22764_amd import dfamin
    d = shift_dfa(40000, list(range(1, 17)), "shift(1..16) n=40000")
    want, nb = _hop(d)
    levels = []
    for grid in (True, False):
        if not grid:
            monkeypatch.setenv("DFAMIN_GRID_MAX_STATES", "0")
        print(f"[case] {d.name}, budget {mib} MiB, grid {grid}", flush=True)
        with dfamin.dfamin_create(0, int(mib * (1 << 20))) as c:
            out, r = dfamin.dfamin_minimize(c, d, "auto", check=False)
        assert r["rc"] == dfamin.DFAMIN_OK
        assert np.array_equal(out, want) and r["num_blocks"] == nb
        levels.append(r["closure_levels"])
    assert levels[0] >= levels[1], levels


def test_handed_back_instances_have_the_scratch_of_the_others():
    """A batch of larger instances, most done in a workgroup each, some handed
    back for their closure: the scratch of the others gives way to its levels."""
    from paper_2410_22764_amd import dfamin
    ds = [W.random_dfa(17000 + 13 * i, 3, i) for i in range(60)]
    ds += [shift_dfa(17500, [1, 2, 3, 4], "shift(1,2,3,4) n=17500")] * 3
    want, nb = _hop(ds[-1])
    levels = {}
    for mib in (90, 400):
        print(f"[case] batch of {len(ds)}, budget {mib} MiB", flush=True)
        with dfamin.dfamin_create(0, mib << 20) as c:
            outs, res = dfamin.dfamin_minimize_batch(c, ds, "auto")
        assert np.array_equal(outs[-1], want) and res[-1]["num_blocks"] == nb
        levels[mib] = [r["closure_levels"] for r in res[-3:]]
    assert levels[90] == levels[400], levels
