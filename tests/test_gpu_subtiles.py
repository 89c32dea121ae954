"""The window search on batches large enough for its search on subtiles: the
kernel takes a batch by the blocks it samples, so both answers of that look
are tested (and which one it gave, from its word in the workspace), at the
edges of subtiles (512 starts, 64 blocks past them), tiles and request groups,
with windows left to the second kernel and blocks too large for packed keys.
Bit for bit against the oracle, eagerly and replayed from a graph."""
import os

import numpy as np
import pytest

import oracle
import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EDGES = [1, 7, 8, 9, 511, 512, 513, 575, 576, 577, 1599, 1600, 1601, 4095, 4096, 4097, 4671, 4672,
         8191, 8192, 8193]


def _batch(pinned, cost, seed, every=4):
    """Snapshots at the edges, and one long one per edge that brings the
    average to more than 8192 blocks; one long one in `every` has no pinned
    block (one in two of those a huge block), one in four a huge block."""
    rng = np.random.default_rng(seed)
    long_ = (1 << 25) // 1200
    lens = []
    for i in range(1230):
        lens += [EDGES[i % len(EDGES)]] if i < 4 * len(EDGES) else []
        lens.append(long_ + int(rng.integers(0, 700)))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
    n = int(off[-1])
    size = (rng.integers(1, 1 << 12, size=n) * 512).astype(np.uint64)
    u = rng.random(n)
    kind = np.where(u < pinned, 2, np.where(u < pinned + 0.15, 0, 1)).astype(np.uint8)
    c = np.exp(rng.random(n) * np.log(1e12)) if cost == "log" else rng.integers(0, 4, n) \
        if cost == "ties" else rng.integers(0, 10**6, n)
    c = np.where(kind == 1, c, 0).astype(np.uint64)
    reqs = []
    for b, (s, e) in enumerate(zip(off[:-1].astype(int), off[1:].astype(int))):
        if e - s > 10000 and b % every == 0:
            kind[s:e] = np.minimum(kind[s:e], 1)
            if every > 4 and b % (2 * every) == 0:
                size[s + int(rng.integers(0, e - s))] = 1 << 40
        if e - s > 10000 and b % 4 == 1:
            size[s + int(rng.integers(0, e - s))] = 1 << 40
        total = int(size[s:e].sum())
        mean = total // (e - s)
        r = [mean * 3, min(total, mean * 500)] if e - s > 10000 else [mean, total, total + 1]
        if b % 97 == 0 or b % every == 0 and every > 4 and e - s > 10000:
            r = [0, 1, mean * 700, mean * 9000] + [int(mean * x) for x in rng.random(126) * 40]
        reqs.append(r)
    req = np.array([x for r in reqs for x in r], dtype=np.uint64)
    roff = np.concatenate([[0], np.cumsum([len(r) for r in reqs])]).astype(np.uint64)
    return workloads.Pools(size, c, kind, off, req, roff)


@pytest.mark.parametrize("pinned, cost, every, subtiles", [
    (0.3, "uniform", 4, 0), (0.3, "log", 4, 0), (0.5, "ties", 4, 0), (0.02, "uniform", 4, 0),
    (0.3, "uniform", 300, 1), (0.3, "log", 300, 1), (0.5, "ties", 300, 1), (0.15, "uniform", 300, 1)])
def test_large_batches(pinned, cost, every, subtiles):
    import paper_2311_00591_amd as coop
    a = _batch(pinned, cost, 7, every)
    info = coop.plan_info(a.num_blocks, a.num_segments, a.num_requests)
    assert info["units"] >= 16 * info["workgroups"] and a.num_blocks >= 8192 * a.num_segments
    print(f"[gpu case] subtiles {subtiles}: pinned {pinned}, {cost} costs, {a.num_blocks} blocks "
          f"{a.num_requests} requests", flush=True)
    want = oracle.window_search(*a.arrays(), threads=min(16, len(os.sched_getaffinity(0))))
    # memory with the least keys in the partial slots and every deferral bit set
    nbytes = coop.workspace_size(a.num_blocks, a.num_segments, a.num_requests)
    memory = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    memory[nbytes * 9 // 10:] = 255
    ws = coop.WindowSearch(*coop.to_device(a, "cuda"), workspace=memory)
    at = coop._pick_offset(a.num_blocks, a.num_segments, a.num_requests)

    def check(label):
        torch.cuda.synchronize()
        assert memory[at:at + 8].tolist() == [subtiles] + [0] * 7, f"{label}: the other kernel"
        got = ws.out.cpu().numpy().view(np.uint64)
        bad = np.flatnonzero((got != want).any(axis=1))
        assert len(bad) == 0, f"{label}: {len(bad)} differ, first {int(bad[0])}"

    ws.launch()
    check("eager")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ws.launch()
    for r in range(2):
        ws.out.fill_(-1)
        g.replay()
        check(f"replay {r}")
        ws.launch()
        check(f"eager after replay {r}")


# Lengths around the shortest snapshot with windows left to the second kernel
# (512 starts and a walk of 8192 blocks, less 7 before the snapshot start when
# a subtile ends without its 64 blocks past the starts; 64 more with them),
# and where the huge block lies that takes those away: among the starts (plain
# prefixes), or among the blocks past them.  (Blocks, place of the huge block,
# snapshot start mod 8; few enough that the batch still counts as short runs.)
FAR = [(8697, 0, 7), (8698, None, 7), (8698, 0, 7), (8698, 511, 7), (8698, 512, 7), (8698, 575, 7),
       (8705, 0, 0), (8705, 575, 0), (8730, 511, 0), (8761, 512, 7), (8762, None, 7), (8762, 575, 7)]


def _far_batch():
    rng = np.random.default_rng(11)
    lens, far = [], []
    for n, at, lead in FAR:
        lens += [4_000_000 + (lead - sum(lens)) % 8, n]
        far.append((len(lens) - 1, at))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
    n = int(off[-1])
    short = 1 << 20  # short runs between: 30% pinned
    u = rng.random(short)
    kind = np.resize(np.where(u < 0.3, 2, np.where(u < 0.45, 0, 1)).astype(np.uint8), n)
    size = np.resize((rng.integers(1, 1 << 12, short) * 512).astype(np.uint64), n)
    cost = np.resize(rng.integers(0, 1 << 40, short).astype(np.uint64), n)
    mean = 1 << 20
    reqs = [[mean * 3, mean * 10] for _ in lens]
    for b, at in far:
        s, e = int(off[b]), int(off[b + 1])
        kind[s:e] = np.minimum(kind[s:e], 1)
        if at is not None:
            size[s + at] = 1 << 40
        total = int(size[s:e].sum())
        reqs[b] = [total, total - 1, total - int(size[e - 1]) + 1, mean * 3]
    cost[kind != 1] = 0
    req = np.array([x for r in reqs for x in r], dtype=np.uint64)
    roff = np.concatenate([[0], np.cumsum([len(r) for r in reqs])]).astype(np.uint64)
    return workloads.Pools(size, cost, kind, off, req, roff)


def test_shortest_snapshots_with_windows_past_the_walk():
    import paper_2311_00591_amd as coop
    a = _far_batch()
    print(f"[gpu case] windows past the walk: {a.num_blocks} blocks {a.num_requests} requests", flush=True)
    want = oracle.window_search(*a.arrays(), threads=min(16, len(os.sched_getaffinity(0))))
    dev = coop.to_device(a, "cuda")
    nbytes = coop.workspace_size(a.num_blocks, a.num_segments, a.num_requests)
    for fill in (0, 255):  # no deferral bit set beforehand, and every one
        memory = torch.full((nbytes,), fill, dtype=torch.uint8, device="cuda")
        ws = coop.WindowSearch(*dev, workspace=memory)
        ws.out.fill_(-7)
        ws.launch()
        torch.cuda.synchronize()
        got = ws.out.cpu().numpy().view(np.uint64)
        bad = np.flatnonzero((got != want).any(axis=1))
        at = coop._pick_offset(a.num_blocks, a.num_segments, a.num_requests)
        assert memory[at].item() == 1
        assert len(bad) == 0, f"memory of {fill}: {len(bad)} differ, first {int(bad[0])}: {got[bad[0]]}, {want[bad[0]]}"


def test_the_stepwise_replay_stays_on_tiles():
    """Pools too large for LDS, enough of them for the search on subtiles: an
    operation's search makes no look at the batch (the word keeps what the
    memory held before)."""
    import paper_2311_00591_amd as coop
    P, cap = 4096, 8192
    print(f"[gpu case] stepwise replay: {P} pools of {cap} slots", flush=True)
    n = P * cap
    assert coop.plan_info(n, P, P)["units"] >= 16 * 512
    st = {k: torch.zeros(n, dtype=t, device="cuda") for k, t in
          (("size", torch.int64), ("cost", torch.int64), ("id", torch.int32))}
    st["kind"] = torch.full((n,), 2, dtype=torch.uint8, device="cuda")
    for k, v in (("size", 8192), ("kind", 0)):
        st[k].view(P, cap)[:, 1] = v
    st["size"].view(P, cap)[:, 0], st["id"].view(P, cap)[:, 0] = 512, 1
    st["len"], st["capacity"] = torch.full((P,), 2, dtype=torch.int64, device="cuda"), cap
    row = lambda t, *v: torch.tensor([*v] * P, dtype=t, device="cuda")
    # an allocation that fits, one that finds no window, one that evicts the first
    tr = {"op": row(torch.uint8, 0, 0, 0), "op_id": row(torch.int32, 2, 3, 4),
          "op_size": row(torch.int64, 512, 1 << 40, 8192), "op_cost": row(torch.int64, 7, 7, 7),
          "op_flags": row(torch.uint8, 1, 1, 1)}
    need = coop.replay_workspace_size(P, cap)
    ws = torch.full((need,), 0xab, dtype=torch.uint8, device="cuda")
    rep = coop.Replay(st, tr, workspace=ws)
    rep.launch()
    torch.cuda.synchronize()
    assert (rep.block.view(P, 3) == torch.tensor([1, -1, 1], device="cuda")).all()
    assert (rep.window.view(P, 3, 2)[:, 2] == torch.tensor([1, 3], device="cuda")).all()
    search = need - (coop.workspace_size(n, P, P) + 255) // 256 * 256
    at = search + coop._pick_offset(n, P, P)
    assert ws[at:at + 8].tolist() == [0xab] * 8


# Batches by what they hold -> whether the search on subtiles takes them.
LOOKS = {"short runs": 1, "few pinned": 0, "pinned at every pool's start": 0, "every other pool open": 0,
         "pinned at both ends": 0, "one pool in 64 open": 0, "costs half zero": 1, "costs mostly zero": 0,
         "mostly free": 0, "many requests, short runs": 1, "many requests, few pinned": 0,
         "many requests, uneven costs": 1, "many requests, uneven costs, longer runs": 0,
         "many requests, uneven costs, one long run": 0, "all pinned": 1}


@pytest.mark.parametrize("what", LOOKS)
def test_the_look_at_a_batch(what):
    """The pick on batches of every kind, the kinds at an odd address too.
    (Requests of 0 bytes: the look does not depend on them.)"""
    import paper_2311_00591_amd as coop
    print(f"[gpu case] look: {what}", flush=True)
    many = what.startswith("many")
    B, n = (16, 1 << 21) if many else (512, 65536)
    gen = torch.Generator(device="cuda").manual_seed(5)
    rand = lambda: torch.rand(B * n, generator=gen, device="cuda")
    pos, pool = torch.arange(B * n, device="cuda") % n, torch.arange(B * n, device="cuda") // n
    share = {"short runs": 0.3, "few pinned": 0.03, "every other pool open": 0.5, "one pool in 64 open": 0.3,
             "pinned at both ends": 0, "costs half zero": 0.3, "costs mostly zero": 0.3, "mostly free": 0.3,
             "many requests, short runs": 0.05, "many requests, uneven costs, longer runs": 0.002,
             "all pinned": 1}.get(what, 0.01)
    pinned = rand() < share
    if what == "pinned at every pool's start": pinned |= pos < 8
    if what == "every other pool open": pinned &= pool % 2 == 0
    if what == "one pool in 64 open": pinned &= pool % 64 != 0
    if what == "pinned at both ends": pinned = (pos < n // 12) | (pos >= n - n // 12)
    if what.endswith("one long run"): pinned[B * n // 2:B * n // 2 + 400_000] = False
    free = rand() < (0.8 if what == "mostly free" else 0.15)
    cost = torch.exp(rand() * 27).long() if "uneven" in what else torch.randint(
        1, 1000, (B * n,), generator=gen, device="cuda")
    cost[rand() < {"costs half zero": 0.4, "costs mostly zero": 0.7}.get(what, 0)] = 0
    kind = torch.where(pinned, 2, torch.where(free, 0, 1)).to(torch.uint8)
    size = torch.full((B * n,), 512, dtype=torch.int64, device="cuda")
    off = torch.arange(B + 1, device="cuda")
    R = 64 if many else 1
    req = torch.zeros(B * R, dtype=torch.int64, device="cuda")
    for shift in (0, 5):
        memory = torch.empty(B * n + shift, dtype=torch.uint8, device="cuda")
        memory[shift:] = kind
        ws = coop.WindowSearch(size, cost, memory[shift:], off * n, req, off * R)
        assert (ws() == 0).all()
        at = coop._pick_offset(B * n, B, B * R)
        assert ws.workspace[at].item() == LOOKS[what], f"kinds shifted by {shift}"


def test_many_requests_on_one_pool():
    """Requests in passes of 64 over every tile, slices of them, bounds shared
    by all workgroups, and costs so uneven that the look takes the pool with
    few pinned blocks; one run longer than the walk."""
    import paper_2311_00591_amd as coop
    rng = np.random.default_rng(3)
    n, R = 1 << 22, 4096
    print(f"[gpu case] subtiles: one pool of {n} blocks, {R} requests", flush=True)
    size = (rng.integers(1, 1 << 12, n) * 512).astype(np.uint64)
    u = rng.random(n)
    kind = np.where(u < 0.01, 2, np.where(u < 0.2, 0, 1)).astype(np.uint8)
    kind[3_000_000:3_009_500] = np.minimum(kind[3_000_000:3_009_500], 1)
    cost = np.where(kind == 1, np.exp(rng.random(n) * np.log(1e12)), 0).astype(np.uint64)
    req = (np.exp(rng.random(R) * np.log(9400)) * (1 << 20)).astype(np.uint64)
    a = workloads.Pools(size, cost, kind, np.array([0, n], np.uint64), req, np.array([0, R], np.uint64))
    ws = coop.WindowSearch(*coop.to_device(a, "cuda"))
    got = ws().cpu().numpy().view(np.uint64)
    assert ws.workspace[coop._pick_offset(n, 1, R)].item() == 1
    want = oracle.window_search(*a.arrays(), threads=min(16, len(os.sched_getaffinity(0))))
    assert (want[:, 1] - want[:, 0])[want[:, 0] != (1 << 64) - 1].max() > 8192
    bad = np.flatnonzero((got != want).any(axis=1))
    assert len(bad) == 0, f"{len(bad)} differ, first {int(bad[0])}"
