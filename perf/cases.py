"""Performance cases: what a user of the library has it do.

Each case is one call (or, for serving, one set of requests) through the
public binding ``paper_2410_22764_amd.dfamin``: single DFAs in device memory
from a few hundred states to 2^24, deep automata that need the closure, a
batch of thousands, host-memory calls, the minimal DFA, and the request loop.
Inputs are synthetic and seeded; sizes follow the repository's workloads, its
tests, or are generic.
"""
import types

import numpy as np
import torch

from paper_2410_22764_amd import dfamin, workloads

_FIELDS = ("num_blocks", "initial_block", "refine_rounds", "rounds_executed", "closure_levels", "closure_letters")
_CTX = {}


def _ctx(which="calls"):
    """A program's context: made once and kept (the request loop has its own)."""
    if which not in _CTX:
        _CTX[which] = dfamin.dfamin_create(0)
    return _CTX[which]


def listed():
    return [
        # a lexer- or pattern-sized automaton: launch and wait latency
        {"name": "random_tiny", "kind": "random", "n": 701, "k": 3, "closure": "auto"},
        # the repository's plain_single workload: the largest size one workgroup holds
        {"name": "random_small", "kind": "random", "n": 16384, "k": 2, "closure": "auto"},
        # Fib_20 of the paper's Table 2: a unary cycle, 15 doubling rounds
        {"name": "fib20", "kind": "fib", "m": 20, "closure": "auto"},
        # an automaton with redundant states (each class about 16 of them), as
        # constructions produce them: blocks stay large to the end
        {"name": "redundant_mid", "kind": "redundant", "n": 200003, "k": 5, "classes": 12500, "closure": "auto"},
        # the repository's plain_large workload (its bench headline)
        {"name": "random_large", "kind": "random", "n": 1 << 24, "k": 4, "closure": "auto"},
        # the repository's deep_chain workload: closure letters in every round
        {"name": "deep_chain_on", "kind": "chain", "n": 1 << 20, "k": 2, "permuted": False, "closure": "on"},
        # a deep automaton of odd size with shuffled ids under the default policy
        {"name": "chain_auto", "kind": "chain", "n": 300007, "k": 3, "permuted": True, "closure": "auto"},
        # the paper's bit-splitter family: many letters, many rounds
        {"name": "bitsplitter20", "kind": "bitsplitter", "m": 20, "closure": "auto"},
        # the repository's batch_mixed workload: 4,096 uneven instances in one call
        {"name": "batch_mixed", "kind": "batch", "count": 4096, "n_max": 65536, "mix": 1},
        # host buffers in and out, an odd size
        {"name": "host_mid", "kind": "host", "n": 1000003, "k": 3},
        # the minimal DFA of the reachable part, host buffers in and out
        {"name": "minimal_mid", "kind": "minimal", "n": 1 << 18, "k": 4},
        # the request loop: 64 requests submitted at once, then all waited for
        {"name": "serving_64", "kind": "serving", "count": 64, "log2_max": 17, "mix": 1},
    ]


def _log_int(rng, lo, hi):
    return int(lo * (hi / lo) ** rng.random())


def draw(rng):
    kind = rng.choice(["random", "random", "random", "redundant", "redundant", "coarse", "chain", "fib",
                       "bitsplitter", "leader", "batch", "host", "minimal", "serving", "noalloc"])
    if kind in ("random", "coarse"):
        n = _log_int(rng, 64, 1 << 23)
        k = rng.randint(1, max(1, min(12, (1 << 26) // n)))
        closure = rng.choice(["auto", "auto", "off"]) if n > 4096 else rng.choice(["auto", "off", "on"])
        return {"kind": kind, "n": n, "k": k, "closure": closure if kind == "random" else "auto"}
    if kind == "redundant":
        n = _log_int(rng, 1000, 1 << 22)
        return {"kind": kind, "n": n, "k": rng.randint(2, 8), "classes": max(16, n // rng.randint(2, 64)),
                "closure": rng.choice(["auto", "off"])}
    if kind == "chain":
        on = rng.random() < 0.3
        return {"kind": kind, "n": _log_int(rng, 64, 1 << (17 if on else 21)), "k": rng.randint(2, 6),
                "permuted": rng.random() < 0.7, "closure": "on" if on else "auto"}
    if kind == "fib":
        return {"kind": kind, "m": rng.randint(10, 28), "closure": "auto", "turn": rng.randint(0, 99)}
    if kind == "bitsplitter":
        return {"kind": kind, "m": rng.randint(6, 20), "closure": "auto", "turn": rng.randint(0, 99)}
    if kind == "leader":
        return {"kind": "bitsplitter", "m": rng.randint(6, 16), "closure": "off", "method": "leader",
                "turn": rng.randint(0, 99)}
    if kind == "batch":
        return {"kind": kind, "count": _log_int(rng, 16, 2048), "n_max": _log_int(rng, 512, 65537),
                "mix": rng.randint(2, 1 << 20)}
    if kind == "host":
        return {"kind": kind, "n": _log_int(rng, 256, 1 << 21), "k": rng.randint(1, 6)}
    if kind == "minimal":
        return {"kind": kind, "n": _log_int(rng, 256, 1 << 20), "k": rng.randint(2, 6)}
    if kind == "serving":
        return {"kind": kind, "count": rng.randint(8, 64), "log2_max": rng.randint(12, 17),
                "mix": rng.randint(2, 1 << 20)}
    return {"kind": "random", "n": _log_int(rng, 64, 250000), "k": rng.randint(2, 4), "closure": "auto",
            "entry": "noalloc"}


# ---------------------------------------------------------------- sizes
def _mix_sizes(case):
    """(n, k, is_chain) per instance of a batch or request set; fixed by the
    case (the contents come from the seed)."""
    rs = np.random.RandomState(case["mix"])
    c = case["count"]
    if case["kind"] == "batch":  # as workloads.batch_mixed
        n = np.floor(64 * (case["n_max"] / 64.0) ** rs.rand(c)).astype(np.int64)
        k = rs.randint(2, 9, c)
        chain = np.arange(c) < round(0.25 * c)
        rs.shuffle(chain)
    else:  # as workloads.serving_stream
        n = np.floor(2.0 ** (8 + (case["log2_max"] - 8) * rs.rand(c))).astype(np.int64)
        k = rs.randint(2, 17, c)
        chain = rs.rand(c) < 0.2
    return n, k.astype(np.int64), chain


def _single_size(case):
    if case["kind"] == "fib":
        return len(workloads.fib_word(case["m"] + 1)), 1
    if case["kind"] == "bitsplitter":
        return 1 << case["m"], max(case["m"] - 1, 1)
    return case["n"], case["k"]


def work(case):
    """Every transition and accept bit read once, every class id written once
    (and the minimal DFA's transitions, where it is asked for)."""
    if case["kind"] in ("batch", "serving"):
        n, k, _ = _mix_sizes(case)
        return {"bytes": float((4 * n * k + (n + 7) // 8 + 4 * n).sum()), "flops": 0.0}
    n, k = _single_size(case)
    b = 4.0 * n * k + (n + 7) // 8 + 4.0 * n
    if case["kind"] == "minimal":
        b += 4.0 * n * k + (n + 7) // 8
    return {"bytes": b, "flops": 0.0}


# ---------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)
    return g


def _bits(acc):
    """LSB-first bitmap of a bool vector."""
    n = acc.numel()
    pad = torch.zeros((n + 7) // 8 * 8, dtype=torch.int32, device=acc.device)
    pad[:n] = acc.to(torch.int32)
    w = torch.tensor([1, 2, 4, 8, 16, 32, 64, 128], dtype=torch.int32, device=acc.device)
    return (pad.view(-1, 8) * w).sum(1).to(torch.uint8)


def _chain_rows(n, k, pi):
    dev = pi.device
    rows = torch.arange(n, device=dev, dtype=torch.int32).repeat(k, 1)
    rows[0, pi] = pi[torch.clamp(torch.arange(n, device=dev) + 1, max=n - 1)].to(torch.int32)
    acc = torch.zeros(n, dtype=torch.bool, device=dev)
    acc[pi[n - 1]] = True
    return rows, acc


def _single(case, seed):
    """(rows int32[k, n], accept bool[n], q0) on the GPU."""
    g, dev = _gen(seed), "cuda"
    kind = case["kind"]
    n, k = _single_size(case)
    q0 = int(torch.randint(0, n, (1,), generator=g, device=dev))
    if kind in ("random", "coarse", "host", "minimal"):
        rows = torch.randint(0, n, (k, n), generator=g, device=dev, dtype=torch.int32)
        if kind == "minimal":  # trimmed input: one letter runs through every state, so all are reachable
            pi = torch.randperm(n, generator=g, device=dev)
            rows[0, pi] = pi.roll(-1).to(torch.int32)
        if kind == "coarse":  # few accepting states: skewed classes
            acc = torch.arange(n, device=dev) % 97 == 0
        else:
            acc = torch.randint(0, 2, (n,), generator=g, device=dev).bool()
        return rows, acc, q0
    if kind == "redundant":
        # every state copies a state of a random automaton of `classes`
        # states; a transition leads to any copy of the class it leads to
        c = case["classes"]
        cls = torch.cat([torch.arange(c, device=dev), torch.randint(0, c, (n - c,), generator=g, device=dev)])
        cls = cls[torch.randperm(n, generator=g, device=dev)]
        order = torch.argsort(cls, stable=True)
        size = torch.bincount(cls, minlength=c)
        start = torch.cumsum(size, 0) - size
        base = torch.randint(0, c, (k, c), generator=g, device=dev)
        rows = torch.empty((k, n), dtype=torch.int32, device=dev)
        for a in range(k):
            t = base[a][cls]
            pick = (torch.rand(n, generator=g, device=dev, dtype=torch.float64) * size[t]).long()
            rows[a] = order[start[t] + pick].to(torch.int32)
        acc = torch.randint(0, 2, (c,), generator=g, device=dev).bool()[cls]
        return rows, acc, q0
    if kind == "chain":
        pi = torch.randperm(n, generator=g, device=dev) if case["permuted"] else torch.arange(n, device=dev)
        rows, acc = _chain_rows(n, k, pi)
        return rows, acc, q0
    if kind == "fib":
        d = workloads.fib_dfa(case["m"])
    else:
        d = workloads.bitsplitter_dfa(case["m"])
    rows = torch.from_numpy(d.rows().view(np.int32)).to(dev)
    return rows, torch.from_numpy(d.accept_bool()).to(dev), q0


def _mixed(case, seed):
    """Flat transitions (each instance from a 16-byte boundary), flat accept
    bytes, and per instance (n, k, offset, accept offset, q0, is_chain)."""
    g, dev = _gen(seed), "cuda"
    n, k, chain = _mix_sizes(case)
    words = (n * k + 3) // 4 * 4
    off = np.concatenate([[0], np.cumsum(words)])
    aoff = np.concatenate([[0], np.cumsum((n + 7) // 8)])
    nw = torch.repeat_interleave(torch.from_numpy(n).to(dev), torch.from_numpy(words).to(dev))
    flat = torch.randint(0, 1 << 31, (int(off[-1]),), generator=g, device=dev)
    flat = ((flat * nw) >> 31).to(torch.int32)
    acc = torch.randint(0, 256, (int(aoff[-1]),), generator=g, device=dev, dtype=torch.uint8)
    q0 = np.random.RandomState(int(seed) & 0x7FFFFFFF).randint(0, 1 << 30, len(n)) % n
    for i in np.nonzero(chain)[0]:
        m = int(n[i])
        rows, fin = _chain_rows(m, int(k[i]), torch.randperm(m, generator=g, device=dev))
        flat[int(off[i]):int(off[i]) + m * int(k[i])] = rows.reshape(-1)
        acc[int(aoff[i]):int(aoff[i + 1])] = _bits(fin)
    return flat, acc, n, k, off, aoff, q0, chain


def _host_dfa(rows, acc, q0):
    k, n = rows.shape
    return workloads.DFA(n, k, rows.reshape(-1).cpu().numpy().view(np.uint32), _bits(acc).cpu().numpy(), q0)


def prepare(case, seed):
    s = types.SimpleNamespace(kind=case["kind"], entry=case.get("entry", "device"))
    if s.kind == "batch":
        s.ctx = _ctx()
        s.flat, s.acc, n, k, off, aoff, q0, _ = _mixed(case, seed)
        ooff = np.concatenate([[0], np.cumsum(n)])
        s.out = torch.empty(int(ooff[-1]), dtype=torch.int32, device="cuda")
        dp, ap, op = s.flat.data_ptr(), s.acc.data_ptr(), s.out.data_ptr()
        specs = [(n[i], k[i], dp + 4 * off[i], ap + aoff[i], q0[i]) for i in range(len(n))]
        s.batch = dfamin.BatchDevice(specs, [op + 4 * o for o in ooff[:-1]])
        return s
    if s.kind == "serving":
        s.ctx = _ctx("serving")
        flat, acc, n, k, off, aoff, q0, _ = _mixed(case, seed)
        flat, acc = flat.cpu().numpy().view(np.uint32), acc.cpu().numpy()
        s.requests = [workloads.DFA(int(n[i]), int(k[i]), flat[off[i]:off[i] + n[i] * k[i]], acc[aoff[i]:aoff[i + 1]],
                                    int(q0[i])) for i in range(len(n))]
        return s
    s.ctx = _ctx()
    rows, acc, q0 = _single(case, seed)
    if s.kind in ("host", "minimal"):
        s.dfa = _host_dfa(rows, acc, q0)
        return s
    s.n, s.k, s.q0 = rows.shape[1], rows.shape[0], q0
    s.rows, s.acc = rows.contiguous(), _bits(acc)
    s.out = torch.empty(s.n, dtype=torch.int32, device="cuda")
    s.opts = dfamin.make_opts(closure=case["closure"], method=case.get("method", "signature"))
    return s


# ---------------------------------------------------------------- one pass
def _ints(res):
    return {f: int(res[f]) for f in _FIELDS}


def run(s):
    if s.kind == "batch":
        s.batch.run(s.ctx, "auto", torch.cuda.current_stream().cuda_stream)
        return {"out": s.out, **{f: s.batch.field(f).astype(np.int64) for f in _FIELDS}}
    if s.kind == "serving":
        tickets = [dfamin.dfamin_submit(s.ctx, d, "auto") for d in s.requests]
        done = [dfamin.dfamin_wait(s.ctx, t, d.n) for t, d in zip(tickets, s.requests)]
        if any(rc != 0 for rc, _, _ in done):
            raise RuntimeError("a request failed")
        return {"out": np.concatenate([o for _, o, _ in done]).view(np.int32),
                **{f: np.array([r[f] for _, _, r in done]) for f in _FIELDS}}
    if s.kind == "host":
        out, res = dfamin.dfamin_minimize(s.ctx, s.dfa, "auto")
        return {"out": out.view(np.int32), **_ints(res)}
    if s.kind == "minimal":
        m, delta, accept, info, out = dfamin.dfamin_minimal_dfa(s.ctx, s.dfa, "auto")
        return {"out": out.view(np.int32), "delta": delta.view(np.int32), "accept": accept, "n": m,
                "q0": info["q0"], "reachable": info["reachable"], "bfs_levels": info["bfs_levels"]}
    call = dfamin.dfamin_minimize_device_noalloc if s.entry == "noalloc" else dfamin.dfamin_minimize_device
    res = call(s.ctx, s.n, s.k, s.rows.data_ptr(), s.acc.data_ptr(), s.q0, s.out.data_ptr(), s.opts,
               torch.cuda.current_stream().cuda_stream)
    return {"out": s.out, **_ints(res)}


# ---------------------------------------------------------------- exact results
def _refine(rows, lab):
    """Coarsest stable refinement of lab under the successor rows (a list of
    int64 vectors), labels in no particular order."""
    lab = torch.unique(lab, return_inverse=True)[1]
    count = int(lab.max()) + 1
    while True:
        new = lab
        for r in rows:
            new = torch.unique(new * (count + 1) + lab[r], return_inverse=True)[1]
        c = int(new.max()) + 1
        if c == count:
            return lab, count
        lab, count = new, c


def _canonical(lab, count):
    """Class numbers in order of each class's least member."""
    n = lab.numel()
    least = torch.full((count,), n, dtype=torch.int64, device=lab.device)
    least.scatter_reduce_(0, lab, torch.arange(n, device=lab.device), "amin")
    rank = torch.empty_like(least)
    rank[torch.argsort(least)] = torch.arange(count, device=lab.device)
    return rank[lab]


def exact(case, seed):
    none = {f: None for f in _FIELDS}
    if case["kind"] in ("batch", "serving"):
        # one union automaton; a chain's states are all different
        flat, acc, n, k, off, aoff, q0, chain = _mixed(case, seed)
        dev = "cuda"
        N = int(n.sum())
        base = np.concatenate([[0], np.cumsum(n)])
        tn = torch.from_numpy(n).to(dev)
        inst = torch.repeat_interleave(torch.arange(len(n), device=dev), tn)
        g = torch.arange(N, device=dev)
        first = torch.from_numpy(base[:-1]).to(dev)[inst]
        q = g - first
        bit = (acc[torch.from_numpy(aoff[:-1]).to(dev)[inst] + (q >> 3)].long() >> (q & 7)) & 1
        at = torch.from_numpy(off[:-1]).to(dev)[inst]
        kk = torch.from_numpy(k).to(dev)[inst]
        rows = []
        for a in range(int(k.max())):
            has = kk > a
            where = torch.where(has, at + a * tn[inst] + q, torch.zeros_like(at))
            rows.append(torch.where(has, first + flat[where].long(), g))
        alone = torch.from_numpy(chain).to(dev)[inst]
        lab, count = _refine(rows, torch.where(alone, 2 * len(n) + g, 2 * inst + bit))
        out = _canonical(lab, count)
        return {"out": out - out[first], **none}
    rows, acc, q0 = _single(case, seed)
    n = rows.shape[1]
    if case["kind"] in ("chain", "fib", "bitsplitter"):  # all states differ, by construction
        out = torch.arange(n, device="cuda")
        return {"out": out, **none, "num_blocks": n, "initial_block": q0}
    lab, count = _refine([r.long() for r in rows], acc.long())
    out = _canonical(lab, count)
    if case["kind"] == "minimal":
        return {"out": out, "delta": None, "accept": None, "n": None, "q0": None, "reachable": None,
                "bfs_levels": None}
    return {"out": out, **none, "num_blocks": count, "initial_block": int(out[q0])}
