"""The bound on walks that a wave's lanes share (the four-way query kernel): in
a damaged tree, whose records may form cycles, every walk ends.

A model of one wave: lanes with stacks, idle lanes taking the lowest entry of
a walking lane's stack, each lane's count of visited records checked every 64
node-step rounds.  The count that a lane starts with when it takes an entry,
and which lanes end with one that is past the bound, are read from the
kernel's source, so the model follows the code.
"""
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LANES, SHARE_MIN, DEFER, STACK = 64, 8, 32, 286


def rules():
    """(a lane that takes an entry starts from the giver's count, a lane past
    the bound ends its segment on every lane) in query.hip."""
    with open(os.path.join(ROOT, "paper_2209_02878_amd", "csrc", "query.hip")) as f:
        text = f.read()
    body = text.split("void share_walks(")[1].split("\n}\n")[0]
    name = re.search(r"int32_t (\w+) = __shfl\(vis, from, 64\)", body)
    start = re.search(r"\bvis = (\w+);", body).group(1)
    cut = text.split(" void k_query(QArgs a)")[1].split("\n}\n")[0].split("max_steps")[1].split("kWalkCut")[0]
    return name is not None and start == name.group(1), "L.own ==" in cut


def wave_rounds(children, segments, bound, from_giver, by_segment, most):
    """Node-step rounds until the wave's segments are walked, None past
    `most`; children[n]: the references of record n (negative: a leaf, tested
    and dropped)."""
    cur = [0] * segments + [None] * (LANES - segments)
    own = list(range(LANES))
    role = ["item"] * segments + ["idle"] * (LANES - segments)
    stack = [[] for _ in range(LANES)]
    vis = [0] * LANES
    rounds = 0
    while True:
        # ended helpers are idle again; a segment is done with its last part
        for i in range(LANES):
            if role[i] == "helps" and cur[i] is None:
                role[i], own[i] = "idle", i
        walked = {own[i] for i in range(LANES) if role[i] == "helps"}
        for i in range(LANES):
            if role[i] == "item" and cur[i] is None and i not in walked:
                role[i] = "idle"
        if "item" not in role:
            return rounds
        idle = [i for i in range(LANES) if role[i] == "idle"]
        if len(idle) >= SHARE_MIN:
            gives = [i for i in range(LANES) if role[i] != "idle" and cur[i] is not None and stack[i]]
            for i, d in zip(idle, gives):
                cur[i], stack[i], own[i], role[i] = stack[d].pop(0), [], own[d], "helps"
                vis[i] = vis[d] if from_giver else 0
        enough = 0
        while True:
            steps = [i for i in range(LANES) if cur[i] is not None and cur[i] >= 0]
            if not steps:
                break
            enough = enough or ((len(steps) + 1) // 2 if len(steps) < DEFER else DEFER)
            for i in steps:
                vis[i] += 1
                stack[i].extend(children[cur[i]])
                del stack[i][STACK:]
                cur[i] = stack[i].pop() if stack[i] else None
            rounds += 1
            if rounds > most:
                return None
            if rounds % 64 == 0:
                late = [i for i in range(LANES) if vis[i] > bound]
                past = {own[i] for i in late}
                for i in range(LANES):
                    if i in late or (by_segment and own[i] in past):
                        cur[i], stack[i] = None, []
            if len(steps) < enough:
                break
        # leaf phase: up to four leaves from the top of each stack
        for i in range(LANES):
            for _ in range(4):
                if cur[i] is not None and cur[i] < 0:
                    cur[i] = stack[i].pop() if stack[i] else None


def damaged(rng, n, leaves):
    """n records whose references go anywhere, `leaves` of them to leaves."""
    refs = rng.integers(0, n, (n, 4))
    refs[rng.random((n, 4)) < leaves] = -1
    return [list(map(int, r)) for r in refs]


@pytest.mark.parametrize("leaves", [0.0, 0.3, 0.6, 0.7])
@pytest.mark.parametrize("segments", [1, 20, 64])
def test_walks_of_a_damaged_tree_end(leaves, segments):
    """Every lane's count covers the steps of its line of descent, and lanes
    with a node on top step together, so a segment's lanes reach the bound at
    about the same time: a small multiple of it bounds the wave."""
    n = 600
    children = damaged(np.random.default_rng(segments), n, leaves)
    rounds = wave_rounds(children, segments, n, *rules(), 8 * n)
    assert rounds is not None


def _four_way(n):
    """A valid tree of n records: record i's children are 4 i + 1 .. 4 i + 4."""
    return [[c if c < n else -1 for c in range(4 * i + 1, 4 * i + 5)] for i in range(n)]


@pytest.mark.parametrize("segments", [1, 5, 64])
def test_valid_walks_are_never_cut(segments):
    """Parts of one walk are disjoint, so a line of descent visits each record
    at most once: with the bound at the number of records no walk is cut
    (a lower bound would cut the walk of one lane alone)."""
    n = 341
    seen = []
    children = _four_way(n)

    class Counting(list):
        def __getitem__(self, i):
            seen.append(i)
            return list.__getitem__(self, i)

    assert wave_rounds(Counting(children), segments, n, True, True, 100 * n) is not None
    assert len(seen) == segments * n  # every record, once per segment
