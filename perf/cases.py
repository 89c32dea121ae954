"""The calls this framework is timed on: which they are, their inputs, one pass
of each, the work a pass cannot do without, and their results in plain torch.

A case is one prepared call of the package on device tensors, as an allocator
or a planner keeps it: the window search (integer and real-valued costs), first
fit, and the replay of Algorithm 1 under both policies.  Four pool shapes occur:

  iid        free, evictable and pinned blocks drawn independently, sizes
             log-uniform, requests log-uniform in bytes;
  clustered  heavy-tailed sizes, pinned blocks in stretches, requests at the
             median and the 95th percentile of a snapshot's open runs, a tenth
             of them infeasible;
  long       parameters pinned at the two ends of one pool, everything between
             them one run, requests from one block to the whole run;
  trace      (replay) pools that start empty between their parameters and the
             allocations of a training iteration.

Inputs come from the seed alone and are drawn on the GPU.  All results are
whole numbers, so every output has to match exactly.
"""
import math

import torch

import paper_2311_00591_amd as coop

KiB, MiB, GiB = 1 << 10, 1 << 20, 1 << 30
GRAIN = 512
FREE, EVICTABLE, PINNED = 0, 1, 2
BIG = (1 << 63) - 1
EXACT_LIMIT = 1 << 30  # (block, request) pairs a plain search takes a few seconds for


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def _iid(name, op, segments, lo, hi, requests, size_hi, req_lo, req_hi, p_free, p_pinned,
         cost_hi, log_cost):
    return {"name": name, "op": op, "shape": "iid", "segments": segments, "lo": lo, "hi": hi,
            "requests": requests, "size_hi": size_hi, "req_lo": req_lo, "req_hi": req_hi,
            "p_free": p_free, "p_pinned": p_pinned, "cost_hi": cost_hi, "log_cost": log_cost}


def _clustered(name, op, segments, lo, hi, requests):
    return {"name": name, "op": op, "shape": "clustered", "segments": segments, "lo": lo,
            "hi": hi, "requests": requests}


def _long(name, blocks, requests):
    return {"name": name, "op": "window", "shape": "long", "segments": 1, "lo": blocks,
            "hi": blocks, "requests": requests}


def _replay(name, policy, pools, layers, iterations, budget, pattern):
    return {"name": name, "op": "replay", "shape": "trace", "policy": policy, "pools": pools,
            "layers": layers, "iterations": iterations, "budget": budget, "pattern": pattern}


def listed():
    return [
        # one allocation that found no chunk: the call an allocator makes itself
        _iid("window_one", "window", 1, 1000, 1000, 1, 64 * MiB, 1 * MiB, 256 * MiB,
             0.10, 0.05, 10**6, False),
        # what-if planning on one small pool: many sizes, one snapshot
        _iid("window_tiny", "window", 1, 1000, 1000, 1000, 64 * MiB, 1 * MiB, 256 * MiB,
             0.10, 0.05, 10**6, False),
        # one request from each of many replicas' pools
        _iid("window_mid", "window", 1024, 4096, 4096, 1, 64 * MiB, 4 * MiB, 1 * GiB,
             0.10, 0.05, 10**6, False),
        # large pools, the requests of a whole layer at once
        _iid("window_large", "window", 256, 65536, 65536, 16, 256 * MiB, 16 * MiB, 4 * GiB,
             0.15, 0.03, 10**9, True),
        # the mixed batch of a cluster: ragged pools, heavy-tailed sizes
        _clustered("window_ragged", "window", 4096, 64, 32768, 4),
        # one pool of a very large memory, a long list of sizes
        _iid("window_huge", "window", 1, 1 << 24, 1 << 24, 4096, 64 * MiB, 64 * MiB, 16 * GiB,
             0.20, 0.01, 10**12, True),
        # activations between the parameters: one run without a pinned block
        _long("window_long", 1 << 24, 16),
        # the free-chunk lookup ahead of any eviction, on the ragged batch
        _clustered("first_fit_ragged", "first_fit", 4096, 64, 32768, 4),
        # costs as the paper defines them, cost over staleness
        _iid("real_mid", "real", 1024, 4096, 4096, 1, 64 * MiB, 4 * MiB, 1 * GiB,
             0.10, 0.05, 10**6, False),
        _iid("real_large", "real", 256, 65536, 65536, 16, 256 * MiB, 16 * MiB, 4 * GiB,
             0.15, 0.03, 10**9, True),
        # one training iteration on many pools, under both eviction policies
        _replay("replay_window", "window", 512, 1024, 1, 0.85, "gpt"),
        _replay("replay_greedy", "greedy", 512, 1024, 1, 0.85, "gpt"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["window"] * 6 + ["first_fit", "real", "real", "replay", "replay"])
    if op == "replay":
        layers = _log(rng, 12, 1024)
        return _strip(_replay("", rng.choice(["window", "greedy"]), _log(rng, 4, 512), layers,
                              rng.choice([1, 2]) if layers <= 512 else 1,
                              rng.choice([0.6, 0.75, 0.85]), rng.choice(["gpt", "resnet"])))
    shape = rng.choice(["iid", "iid", "clustered", "long"] if op == "window" else ["iid", "clustered"])
    if shape == "long":
        return _strip(_long("", _log(rng, 10_000, 1 << 24), rng.choice([1, 2, 5, 16])))
    pairs_cap = 1 << (28 if op == "real" else 32)
    segments = _log(rng, 1, 4096)
    blocks = _log(rng, max(64 * segments, 1000), 1 << (24 if op == "real" else 26))
    mean = max(64, blocks // segments)
    requests = min(_log(rng, 1, 4096 if segments == 1 else 64), max(1, pairs_cap // blocks))
    requests = min(requests, max(1, (1 << 18) // segments))
    lo, hi = (max(1, mean // 4), mean + mean // 2 + 1) if rng.random() < 0.6 else (mean, mean)
    if shape == "clustered":
        return _strip(_clustered("", op, segments, lo, hi, requests))
    size_hi = rng.choice([64, 256]) * MiB
    req_lo = rng.choice([1, 4, 16]) * MiB
    return _strip(_iid("", op, segments, lo, hi, requests, size_hi, req_lo, 256 * req_lo,
                       rng.choice([0.10, 0.15, 0.20]), rng.choice([0.01, 0.03, 0.05]),
                       rng.choice([10**6, 10**9]), rng.random() < 0.5))


def _strip(case):
    del case["name"]
    return case


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _rand(gen, *n):
    return torch.rand(*n, generator=gen, device="cuda", dtype=torch.float64)


def _log_uniform(gen, lo, hi, *n):
    return torch.exp(math.log(lo) + _rand(gen, *n) * (math.log(hi) - math.log(lo)))


def _grains(x):
    return (torch.ceil(x / GRAIN).clamp(min=1) * GRAIN).to(torch.int64)


def _geometric(gen, p, n):
    u = 1.0 - _rand(gen, n)
    return torch.ceil(torch.log(u) / math.log(1.0 - p)).clamp(min=1).to(torch.int64)


def _run_requests(gen, size, kind, seg_of, segments, requests):
    """Requests at the median and the 95th percentile of each snapshot's open
    runs, one in ten just above the largest run."""
    open_ = kind != PINNED
    before = torch.cat([open_.new_zeros(1), open_[:-1]])
    new_seg = torch.cat([open_.new_ones(1), seg_of[1:] != seg_of[:-1]])
    starts = open_ & (~before | new_seg)
    run = torch.cumsum(starts, 0) - 1
    n_runs = int(starts.sum())
    totals = torch.zeros(n_runs + 1, dtype=torch.int64, device="cuda")
    totals.index_add_(0, torch.where(open_, run, n_runs), size)
    totals, owner = totals[:n_runs], seg_of[starts]
    order = torch.argsort(totals, stable=True)
    order = order[torch.argsort(owner[order], stable=True)]
    totals = torch.cat([totals[order], totals.new_full((1,), GRAIN)])
    count = torch.bincount(owner, minlength=segments)
    first = torch.cumsum(count, 0) - count
    pct = torch.where(torch.arange(requests, device="cuda") % 2 == 0, 0.50, 0.95)
    rank = torch.ceil(pct[None] * count[:, None]).to(torch.int64).clamp(min=1) - 1
    none = (count == 0)[:, None]
    req = totals[torch.where(none, n_runs, first[:, None] + rank)]
    top = totals[torch.where(none, n_runs, (first + count - 1)[:, None])] + GRAIN
    return torch.where((_rand(gen, segments, requests) < 0.1) & ~none, top, req)


def _pools(case, seed):
    """Device tensors of a batch: blocks, offsets, requests (segments x requests)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B, R, lo, hi = case["segments"], case["requests"], case["lo"], case["hi"]
    nb = torch.randint(lo, hi + 1, (B,), generator=gen, device="cuda")
    seg = torch.zeros(B + 1, dtype=torch.int64, device="cuda")
    seg[1:] = torch.cumsum(nb, 0)
    n = int(seg[-1])
    seg_of = torch.repeat_interleave(torch.arange(B, device="cuda"), nb)
    if case["shape"] == "clustered":
        size = _grains((GRAIN * torch.exp(-torch.log(1.0 - _rand(gen, n)) / 1.2)).clamp(max=GiB))
        p_pin, p_open = 0.3, 9 / 70
        pairs = int(n / (1 / p_pin + 1 / p_open) * 1.05) + 1000
        lens = torch.stack([_geometric(gen, p_open, pairs), _geometric(gen, p_pin, pairs)], 1).view(-1)
        label = torch.tensor([False, True], device="cuda").repeat(pairs)
        pinned = torch.repeat_interleave(label, lens)
        if pinned.numel() < n:  # (practically never: five percent to spare)
            pinned = torch.cat([pinned, pinned.new_zeros(n - pinned.numel())])
        kind = torch.where(_rand(gen, n) < 1 / 7, FREE, EVICTABLE)
        kind = torch.where(pinned[:n], PINNED, kind).to(torch.uint8)
        cost = torch.randint(0, (1 << 40) + 1, (n,), generator=gen, device="cuda")
        req = _run_requests(gen, size, kind, seg_of, B, R)
    elif case["shape"] == "long":
        size = _grains(_log_uniform(gen, 512, 64 * MiB, n))
        kind = torch.where(_rand(gen, n) < 0.2, FREE, EVICTABLE).to(torch.uint8)
        kind[:37] = PINNED
        kind[-53:] = PINNED
        cost = torch.floor(_log_uniform(gen, 1, 10**12, n)).to(torch.int64)
        run = int(size[37:-53].sum())
        mean = int(size.sum()) // n
        # one block, the mean block, 100 and 5000 of them, then parts of the run
        sizes = [512, mean, 100 * mean, min(5000 * mean, run)] + [run * k // 12 for k in range(1, 13)]
        pick = [run // 2, run, 100 * mean, mean, run // 3] if R < len(sizes) else sizes
        req = torch.tensor(pick[:R], dtype=torch.int64, device="cuda").view(1, R)
    else:
        size = _grains(_log_uniform(gen, 512, case["size_hi"], n))
        u = _rand(gen, n)
        pf, pp = case["p_free"], case["p_pinned"]
        kind = torch.where(u < pf, FREE, torch.where(u < pf + pp, PINNED, EVICTABLE)).to(torch.uint8)
        if case["log_cost"]:
            cost = torch.floor(_log_uniform(gen, 1, case["cost_hi"], n)).to(torch.int64)
        else:
            cost = torch.randint(1, case["cost_hi"] + 1, (n,), generator=gen, device="cuda")
        req = torch.ceil(_log_uniform(gen, case["req_lo"], case["req_hi"], B, R)).to(torch.int64)
    cost[kind != EVICTABLE] = 0
    req_off = torch.arange(B + 1, dtype=torch.int64, device="cuda") * R
    batch = {"size": size, "cost": cost, "kind": kind, "seg": seg, "seg_of": seg_of,
             "req": req.reshape(-1).contiguous(), "req_off": req_off}
    if case["op"] == "real":
        stale = torch.randint(1, 4097, (n,), generator=gen, device="cuda")
        batch["h"] = cost.to(torch.float64) / stale
    return batch


# microseconds of recomputation per MiB of each layer kind, and whether its
# cost grows faster than its size
LAYERS = {"gpt": ((33.5, 1), (4.2, 0), (3.8, 0)), "resnet": ((35.6, 1), (3.9, 0))}
PARAMS = 4  # unevictable blocks at each end of a pool


def _trace(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    P, L, its = case["pools"], case["layers"], case["iterations"]
    pattern = LAYERS[case["pattern"]]
    cap, T = 2 * PARAMS + 2 * L + 16, its * 4 * L
    acts = _grains(_log_uniform(gen, 1 * MiB, 64 * MiB, P, L))
    params = _grains(_log_uniform(gen, 4 * MiB, 256 * MiB, P, 2 * PARAMS))
    free = (acts.sum(1).to(torch.float64) * case["budget"] / GRAIN).ceil().to(torch.int64) * GRAIN
    n = 2 * PARAMS + 1
    size = torch.zeros(P, cap, dtype=torch.int64, device="cuda")
    size[:, :n] = torch.cat([params[:, :PARAMS], free[:, None], params[:, PARAMS:]], 1)
    kind = torch.full((P, cap), PINNED, dtype=torch.uint8, device="cuda")
    kind[:, PARAMS] = FREE
    ids = torch.zeros(P, cap, dtype=torch.int32, device="cuda")
    ids[:, :n] = torch.tensor([*range(1, PARAMS + 1), 0, *range(PARAMS + 1, 2 * PARAMS + 1)],
                              dtype=torch.int32, device="cuda")
    state = {"size": size.view(-1), "cost": torch.zeros_like(size).view(-1), "kind": kind.view(-1),
             "id": ids.view(-1), "len": torch.full((P,), n, dtype=torch.int64, device="cuda"),
             "capacity": cap}
    # one row of operations for all pools: (release?, id, layer or -1)
    rows, nid = [], 2 * PARAMS + 1
    for _ in range(its):
        act = list(range(nid, nid + L))
        rows += [(0, act[i], i) for i in range(L)]
        nid += L
        for i in reversed(range(L)):
            rows += [(0, nid, i), (1, act[i], -1), (1, nid, -1)]
            nid += 1
    op, op_id, layer = (torch.tensor(c, device="cuda") for c in zip(*rows))
    alloc = (layer >= 0)[None]
    density = torch.tensor([pattern[i % len(pattern)][0] for i in range(L)], dtype=torch.float64,
                           device="cuda")
    flags = torch.tensor([pattern[i % len(pattern)][1] for i in range(L)], device="cuda")
    at = layer.clamp(min=0)
    op_size = torch.where(alloc, acts[:, at], 0)
    op_cost = torch.where(alloc, (density[None] * acts / MiB * 1000).round().to(torch.int64)[:, at], 0)
    op_flags = torch.where(alloc, flags[at][None], 0).expand(P, T)
    trace = {"op": op.to(torch.uint8).expand(P, T).contiguous().view(-1),
             "op_id": op_id.to(torch.int32).expand(P, T).contiguous().view(-1),
             "op_size": op_size.contiguous().view(-1), "op_cost": op_cost.contiguous().view(-1),
             "op_flags": op_flags.to(torch.uint8).contiguous().view(-1)}
    return state, trace


def prepare(case, seed):
    if case["op"] == "replay":
        policy = coop.POLICY_WINDOW if case["policy"] == "window" else coop.POLICY_GREEDY
        return coop.Replay(*_trace(case, seed), policy=policy)
    b = _pools(case, seed)
    tail = (b["seg"], b["req"], b["req_off"])
    if case["op"] == "first_fit":
        return coop.FirstFit(b["size"], b["kind"], *tail)
    if case["op"] == "real":
        return coop.WindowSearchReal(b["size"], b["h"], b["kind"], *tail)
    return coop.WindowSearch(b["size"], b["cost"], b["kind"], *tail)


def run(state):
    if isinstance(state, coop.Replay):
        # (a training iteration leaves the pools as it found them)
        state.launch()
        return [state.block, state.window, state.cost, state.free, state.status,
                *(state.state[k] for k in ("size", "cost", "kind", "id", "len"))]
    out = state()
    return [out, state.status] if isinstance(state, coop.WindowSearchReal) else out


def work(case):
    if case["op"] == "replay":
        ops = case["pools"] * case["iterations"] * 4 * case["layers"]
        used = case["pools"] * (2 * PARAMS + 1)
        # an operation's record and its outcome, the pools in and out
        return {"bytes": ops * (22 + 40) + used * 2 * 21, "flops": ops}
    blocks = case["segments"] * (case["lo"] + case["hi"]) // 2
    queries = case["segments"] * case["requests"]
    per_block = {"first_fit": 9, "window": 17, "real": 17}[case["op"]]
    per_query = {"first_fit": 8 + 8, "window": 8 + 24, "real": 8 + 40}[case["op"]]
    # each block's bytes, cost and pinned count summed once, or compared once
    adds = {"first_fit": 1, "window": 3, "real": 4}[case["op"]]
    return {"bytes": blocks * per_block + queries * per_query, "flops": blocks * adds}


def tolerance(case):
    return "exact"


# ---------------------------------------------------------------------------
# The same results in plain torch
# ---------------------------------------------------------------------------

def _segment_min(value, seg_of, segments):
    out = torch.full((segments,), BIG, dtype=torch.int64, device="cuda")
    return out.scatter_reduce_(0, seg_of, value, "amin")


def _least(keys, valid, seg_of, segments):
    """Per segment, the lexicographic minimum of the key columns over the valid rows."""
    rows = valid.nonzero().squeeze(1)
    owner, cols = seg_of[rows], [k[rows] for k in keys]
    best = []
    for c in range(len(cols)):
        m = _segment_min(cols[c], owner, segments)
        best.append(m)
        keep = (cols[c] == m[owner]).nonzero().squeeze(1)
        owner, cols = owner[keep], [k[keep] for k in cols]
    return best


def _prefix(x):
    return torch.cat([x.new_zeros(1), torch.cumsum(x, 0)])


def _exact_search(case, seed):
    b = _pools(case, seed)
    n, B, R = b["size"].numel(), case["segments"], case["requests"]
    if n * R > EXACT_LIMIT:
        return None
    seg, seg_of, pinned = b["seg"], b["seg_of"], b["kind"] == PINNED
    req = b["req"].view(B, R)
    index = torch.arange(n, device="cuda")
    if case["op"] == "first_fit":
        free = b["kind"] == FREE
        cols = [_least([index], free & (b["size"] >= req[:, r][seg_of]), seg_of, B)[0]
                for r in range(R)]
        out = torch.stack(cols, 1)
        return torch.where(out == BIG, -1, out - seg[:-1, None]).view(-1)
    # where each block's run ends: the next pinned block or the snapshot's end
    wall = torch.where(pinned, index, BIG)
    wall = torch.flip(torch.cummin(torch.flip(wall, [0]), 0)[0], [0])
    run_end = torch.minimum(wall, seg[1:][seg_of])
    P = _prefix(b["size"])
    if case["op"] == "real":
        # h in units of 2^-64: the whole part and two halves of the fraction
        # (exact: every nonzero h is at least 2^-12)
        whole = torch.floor(b["h"])
        frac = (b["h"] - whole) * 2.0**32
        top = torch.floor(frac)
        limbs = [whole, top, (frac - top) * 2.0**32]
        sums = [_prefix(x.to(torch.int64)) for x in limbs]
    else:
        sums = [_prefix(b["cost"])]
    out = torch.empty(B, R, 5 if case["op"] == "real" else 3, dtype=torch.int64, device="cuda")
    mask = (1 << 32) - 1
    for r in range(R):
        end = torch.searchsorted(P, P[:-1] + req[:, r][seg_of])
        valid = (end <= run_end) & ~pinned
        e = end.clamp(max=n)
        d = [s[e] - s[:-1] for s in sums]
        if len(d) == 3:
            d[1] = d[1] + (d[2] >> 32)
            d[2] = d[2] & mask
            d[0] = d[0] + (d[1] >> 32)
            d[1] = d[1] & mask
        best = _least([*d, P[e] - P[:-1], index], valid, seg_of, B)
        start, none = best[-1], best[-1] == BIG
        local = start.clamp(max=n - 1)
        out[:, r, 0] = start - seg[:-1]
        out[:, r, 1] = e[local] - seg[:-1]
        if len(d) == 3:
            out[:, r, 2] = (best[1] << 32) | best[2]
            out[:, r, 3] = best[0]
            exact = [(h << 64) | (m << 32) | l for h, m, l in
                     zip(*(torch.where(none, 0, x).tolist() for x in best[:3]))]
            cost = torch.tensor([x / 2**64 for x in exact], dtype=torch.float64, device="cuda")
            out[:, r, 4] = torch.where(none, math.inf, cost).view(torch.int64)
        else:
            out[:, r, 2] = best[0]
        out[none, r, :4 if len(d) == 3 else 3] = -1
    out = out.view(B * R, -1)
    if case["op"] == "real":
        return [out, torch.zeros(1, dtype=torch.int32, device="cuda")]
    return out


class _Pools:
    """All pools of a replay side by side, one row each; every operation is
    of the same kind in all of them."""

    def __init__(self, state):
        P, cap = state["len"].numel(), state["capacity"]
        self.size, self.cost, self.id = (state[k].view(P, cap).to(torch.int64)
                                         for k in ("size", "cost", "id"))
        self.kind, self.len = state["kind"].view(P, cap).to(torch.int64), state["len"].clone()
        self.slots = torch.arange(cap, device="cuda")[None]
        self.rows = torch.arange(P, device="cuda")

    def at(self, x, k):
        return x.gather(1, k.clamp(0, x.shape[1] - 1)[:, None]).squeeze(1)

    def first(self, mask):
        """The first slot of each row where mask holds (BIG: none)."""
        return torch.where(mask, self.slots, BIG).amin(1)

    def replace(self, act, lo, hi, blocks):
        """Slots [lo, hi) of the rows in act become `blocks`, a list of
        (present, size, cost, kind, id) per row."""
        lo, hi = torch.where(act, lo, 0)[:, None], torch.where(act, hi, 0)[:, None]
        m = sum((act & b[0]).to(torch.int64) for b in blocks)[:, None]
        src = torch.where(self.slots < lo + m, self.slots, self.slots - m - lo + hi)
        past = src >= self.slots.shape[1]
        src = src.clamp(0, self.slots.shape[1] - 1)
        pos = lo.clone()
        new = []
        for x, empty in ((self.size, 0), (self.cost, 0), (self.kind, PINNED), (self.id, 0)):
            new.append(torch.where(past, empty, x.gather(1, src)))
        for present, *values in blocks:
            here = (self.slots == pos) & (act & present)[:, None]
            for k, v in enumerate(values):
                v = v[:, None] if isinstance(v, torch.Tensor) else v
                new[k] = torch.where(here, v, new[k])
            pos = pos + (act & present)[:, None].to(torch.int64)
        self.size, self.cost, self.kind, self.id = new
        self.len = self.len + (m - (hi - lo)).squeeze(1)

    def free_up(self, act, lo, hi):
        """Blocks [lo, hi) and their free neighbours become one free chunk;
        returns its slot."""
        lo = lo - ((lo > 0) & (self.at(self.kind, lo - 1) == FREE)).to(torch.int64)
        hi = hi + ((hi < self.len) & (self.at(self.kind, hi) == FREE)).to(torch.int64)
        inside = (self.slots >= lo[:, None]) & (self.slots < hi[:, None])
        total = torch.where(inside, self.size, 0).sum(1)
        self.replace(act, lo, hi, [(act, total, 0, FREE, 0)])
        return lo

    def free_bytes(self):
        return torch.where(self.kind == FREE, self.size, 0).sum(1)

    def fit(self, S):
        return self.first((self.kind == FREE) & (self.size >= S[:, None]))

    def window(self, S):
        zero = self.size.new_zeros(self.size.shape[0], 1)
        evict = torch.where(self.kind == EVICTABLE, self.cost, 0)
        P, C, R = (torch.cat([zero, torch.cumsum(x, 1)], 1)
                   for x in (self.size, evict, (self.kind == PINNED).to(torch.int64)))
        end = torch.searchsorted(P[:, 1:].contiguous(), P[:, :-1] + S[:, None]) + 1
        e = end.clamp(max=self.size.shape[1])
        valid = (end == e) & (R.gather(1, e) == R[:, :-1])
        for key in (C.gather(1, e) - C[:, :-1], P.gather(1, e) - P[:, :-1]):
            k = torch.where(valid, key, BIG)
            valid &= k == k.amin(1, keepdim=True)
        start = self.first(valid)
        return start, self.at(e, start), self.at(C, self.at(e, start)) - self.at(C, start)


def _exact_replay(case, seed):
    state, trace = _trace(case, seed)
    p = _Pools(state)
    P, T = p.len.numel(), trace["op"].numel() // state["len"].numel()
    kinds = trace["op"].view(P, T)[0].tolist()
    tr = {k: v.view(P, T).to(torch.int64) for k, v in trace.items()}
    block = torch.full((P, T), -1, dtype=torch.int64, device="cuda")
    window = torch.full((P, T, 2), -1, dtype=torch.int64, device="cuda")
    cost = torch.zeros(P, T, dtype=torch.int64, device="cuda")
    free = torch.full((P, T), -1, dtype=torch.int64, device="cuda")
    for t in range(T):
        oid = tr["op_id"][:, t]
        if kinds[t]:
            j = p.first((p.kind != FREE) & (p.id == oid[:, None]))
            act = j != BIG
            lo = p.free_up(act, torch.where(act, j, 0), torch.where(act, j + 1, 0))
            block[:, t] = torch.where(act, lo, -1)
            continue
        S = tr["op_size"][:, t]
        k = p.fit(S)
        need = k == BIG
        if bool(need.any()):
            before = p.free_bytes()
            if case["policy"] == "window":
                w0, w1, wc = p.window(S)
                need &= w0 != BIG
                lo = p.free_up(need, torch.where(need, w0, 0), torch.where(need, w1, 0))
                window[:, t] = torch.where(need[:, None], torch.stack([w0, w1], 1), -1)
                cost[:, t] = torch.where(need, wc, 0)
                free[:, t] = torch.where(need, before, -1)
                k = torch.where(need, lo, k)
            else:
                count, spent = torch.zeros_like(k), torch.zeros_like(k)
                while True:
                    # least cost over size times staleness; distinct ratios of
                    # these integers (sizes in grains) are distinct in binary64
                    stale = (oid[:, None] - p.id).clamp(min=1)
                    h = p.cost.to(torch.float64) / ((p.size // GRAIN).clamp(min=1) * stale)
                    h = torch.where(p.kind == EVICTABLE, h, math.inf)
                    v = p.first(h == h.amin(1, keepdim=True))
                    act = need & (h.amin(1) < math.inf)
                    if not bool(act.any()):
                        break
                    count += act
                    spent += torch.where(act, p.at(p.cost, v), 0)
                    lo = p.free_up(act, torch.where(act, v, 0), torch.where(act, v + 1, 0))
                    done = act & (p.at(p.size, lo) >= S)
                    k = torch.where(done, lo, k)
                    need &= ~done
                window[:, t, 0] = torch.where(count > 0, count, -1)
                cost[:, t] = spent
                free[:, t] = torch.where(count > 0, before, -1)
        ok = k != BIG
        at = torch.where(ok, k, 0)
        rest = p.at(p.size, at) - S
        split, left = rest != 0, tr["op_flags"][:, t] == 1
        tensor = (S, tr["op_cost"][:, t], EVICTABLE, oid)
        p.replace(ok, at, at + 1, [(split & ~left, rest, 0, FREE, 0), (ok, *tensor),
                                   (split & left, rest, 0, FREE, 0)])
        block[:, t] = torch.where(ok, at + (split & ~left).to(torch.int64), -1)
    return [block.view(-1), window.view(-1), cost.view(-1), free.view(-1),
            torch.zeros(1, dtype=torch.int32, device="cuda"),
            p.size.reshape(-1), p.cost.reshape(-1), p.kind.to(torch.uint8).reshape(-1),
            p.id.to(torch.int32).reshape(-1), p.len]


def exact(case, seed):
    if case["op"] == "replay":
        return _exact_replay(case, seed)
    return _exact_search(case, seed)
