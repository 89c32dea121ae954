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
@pytest.mark.parametrize("blocks,ops", [(1, 6), (2, 16), (64, 24), (257, 24), (1030, 24)])
def test_pools_that_fill_their_slots(blocks, ops, policy):
    """The fewest slots that the replay can do with: with no room at one end
    the blocks at the other have to move, and with none at either end the pool
    fills its slots."""
    for seed in range(4):
        for cap in range(blocks, blocks + ops + 2):
            state, trace = pools(blocks, ops, seed, False, cap)
            try:
                oracle.replay(state, trace, threads=8, policy=policy)
                break
            except Exception:  # the oracle refuses a replay that runs out of slots
                continue
        label = f"full: {blocks} blocks in {cap} slots, {ops} operations, seed {seed}, {policy}"
        replay._announce(label)
        replay.assert_same(state, trace, label, policy)
