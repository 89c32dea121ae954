"""The resident replay at the edges of its rounds: pools of as many blocks as
a round scans or moves, one less and one more, so that tails move by one round
or several, both ways; operation counts around the batch the kernel reads
ahead; equal costs and sizes, so that windows and victims tie.  Whole numbers:
every outcome equals the CPU oracle's."""
import numpy as np
import pytest

import oracle
import test_gpu_replay as replay

pytestmark = pytest.mark.gpu

GRAIN = 512
OUT_OF_SLOTS = -5  # the oracle's code for it


def pools(blocks, ops, seed, ties, cap=None):
    """Random pools of `blocks` blocks each and `ops` operations on them."""
    rng = np.random.default_rng(seed)
    P, cap = 3, cap or blocks + 2 * ops + 2
    st = {"size": np.zeros((P, cap), np.uint64), "cost": np.zeros((P, cap), np.uint64),
          "kind": np.full((P, cap), 2, np.uint8), "id": np.zeros((P, cap), np.uint32)}
    tr = {k: np.zeros((P, ops), t) for k, t in
          (("op", np.uint8), ("op_id", np.uint32), ("op_size", np.uint64),
           ("op_cost", np.uint64), ("op_flags", np.uint8))}
    for p in range(P):
        kind = rng.choice([0, 1, 2], blocks, p=[0.2, 0.77, 0.03]).astype(np.uint8)
        # a pool holds no two adjacent free chunks (a released one merges)
        for k in range(1, blocks):
            if kind[k] == 0 and kind[k - 1] == 0:
                kind[k] = 1
        st["kind"][p, :blocks] = kind
        st["size"][p, :blocks] = GRAIN * rng.integers(1, 3 if ties else 200, blocks)
        st["cost"][p, :blocks] = np.where(kind == 1, rng.integers(0, 2 if ties else 1 << 50, blocks), 0)
        st["id"][p, :blocks] = np.where(kind != 0, np.arange(1, blocks + 1), 0)
        held = list(range(1, blocks + 1))
        for t in range(ops):
            if rng.random() < 0.4:
                # the first, the last or any tensor, held or evicted or never there
                i = int(rng.choice([0, -1, rng.integers(len(held))]))
                tr["op"][p, t], tr["op_id"][p, t] = 1, held[i]
                continue
            nid = blocks + 1 + t
            held.append(nid)
            big = int(rng.choice([1, 2, 5, 40, blocks]))
            tr["op_id"][p, t] = nid
            tr["op_size"][p, t] = GRAIN * big * (1 if ties else int(rng.integers(1, 100)))
            tr["op_cost"][p, t] = 1 if ties else int(rng.integers(0, 1 << 50))
            tr["op_flags"][p, t] = int(rng.integers(0, 4))
    state = {k: v.reshape(-1) for k, v in st.items()}
    state["len"] = np.full(P, blocks, np.uint64)
    state["capacity"] = cap
    return state, {k: v.reshape(-1) for k, v in tr.items()}


@pytest.mark.parametrize("policy", [replay.WINDOW, replay.GREEDY])
@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("blocks,ops", [(1, 1), (2, 7), (63, 8), (64, 9), (255, 17), (257, 33),
                                        (1023, 40), (1024, 41), (1026, 47), (2047, 40), (2050, 63),
                                        (4000, 31)])
def test_edges_of_rounds_and_batches(blocks, ops, ties, policy):
    label = f"edges: {blocks} blocks, {ops} operations, ties {ties}, policy {policy}"
    replay._announce(label)
    state, trace = pools(blocks, ops, 1000 * blocks + ops, ties)
    assert (state["capacity"] * 31) < 150 * 1024  # held in LDS
    replay.assert_same(state, trace, label, policy)


@pytest.mark.parametrize("policy", [replay.WINDOW, replay.GREEDY])
@pytest.mark.parametrize("cap", [1040, 1046, 2620, 2628, 2632, 2633, 2640])
def test_pools_close_to_a_share_of_the_lds(cap, policy):
    """Around a fifth and a half of a CU's LDS, the kernel has a form that
    keeps costs and outcomes in registers."""
    label = f"{cap} slots, policy {policy}"
    replay._announce(label)
    for ops in (7, 41):
        replay.assert_same(*pools(900, ops, cap + ops, False, cap), f"{label}, {ops} operations", policy)


@pytest.mark.parametrize("policy", [replay.WINDOW, replay.GREEDY])
@pytest.mark.parametrize("blocks,ops", [(1, 6), (2, 16), (64, 24), (257, 24), (1030, 24)])
def test_pools_that_fill_their_slots(blocks, ops, policy):
    """The fewest slots that the replay can do with, so that some operation
    leaves the pool with no slot to spare."""
    for seed in range(4):
        for cap in range(blocks, blocks + ops + 2):
            state, trace = pools(blocks, ops, seed, False, cap)
            try:
                oracle.replay(state, trace, threads=8, policy=policy)
                break
            except oracle.OracleError as e:  # it refuses a replay that runs out of slots
                assert e.code == OUT_OF_SLOTS
                continue
        label = f"full: {blocks} blocks in {cap} slots, {ops} operations, seed {seed}, {policy}"
        replay._announce(label)
        replay.assert_same(state, trace, label, policy)


@pytest.mark.parametrize("policy", [replay.WINDOW, replay.GREEDY])
@pytest.mark.parametrize("cap", [4, 5400])
def test_an_eviction_that_leaves_no_slot(cap, policy):
    """A full pool whose one evictable block is larger than the request: the
    eviction stays done, the allocation fails for want of a slot for the rest,
    and so does one that would fill the chunk exactly; once a neighbour is
    released there is room.  Worked by hand (the oracle refuses a replay that
    runs out of slots), in LDS and step by step."""
    replay._announce(f"no slot left after an eviction: {cap} slots, policy {policy}")
    MB, none = 1 << 20, (1 << 64) - 1
    state = {"size": np.full(cap, MB, np.uint64), "cost": np.zeros(cap, np.uint64),
             "kind": np.full(cap, 2, np.uint8), "id": np.arange(1, cap + 1, dtype=np.uint32),
             "len": np.array([cap], np.uint64), "capacity": cap}
    state["size"][1], state["cost"][1], state["kind"][1] = 8 * MB, 5, 1
    a, b, c, d = cap + 1, cap + 2, cap + 3, cap + 4
    trace = {"op": np.array([0, 0, 1, 0, 0], np.uint8), "op_id": np.array([a, b, 3, c, d], np.uint32),
             "op_size": np.array([MB, 8 * MB, 0, 9 * MB, MB], np.uint64),
             "op_cost": np.array([1, 1, 0, 6, 1], np.uint64), "op_flags": np.array([1, 1, 0, 1, 1], np.uint8)}
    got_state, got, status = replay.gpu_replay(state, trace, policy)
    assert status == 1
    assert got["block"][0].tolist() == [none, none, 1, 1, 1]
    evicted = [1, 2] if policy == replay.WINDOW else [1, none]
    assert got["window"][0].tolist() == [evicted, [none] * 2, [none] * 2, [none] * 2, evicted]
    assert got["cost"][0].tolist() == [5, 0, 0, 0, 6]
    assert got["free"][0].tolist() == [0, none, none, none, 0]
    # the last allocation's megabyte at the left end of the nine, the rest free
    assert got_state["len"].tolist() == [cap]
    assert got_state["size"].tolist() == [MB, MB, 8 * MB] + [MB] * (cap - 3)
    assert got_state["kind"].tolist() == [2, 1, 0] + [2] * (cap - 3)
    assert got_state["id"].tolist() == [1, d, 0] + list(range(4, cap + 1))
    assert got_state["cost"].tolist() == [0, 1, 0] + [0] * (cap - 3)
