"""Progress of the gated delta rule's walks, which wait for each other inside one launch: a model of how workgroups are started.

Workgroups of a launch go round-robin over 8 XCDs (id = y * columns + x); every XCD starts its share of each launch when a compute
unit is free, in some order, and which launch it serves first is its own affair.  A started workgroup holds its compute unit until
all segments that it waits for are done.  A workgroup's place in the walk's order is its ticket, the number of workgroups of its column
that have started before it; with its block id in the place of the ticket (the mistake) the same model stops."""
import ctypes
import os
import random
import re
import subprocess

import pytest

import paper_2511_00413_amd as T
import workloads as W

CSRC = os.path.join(os.path.dirname(T.__file__), "csrc")
XCDS = 8


@pytest.fixture(scope="module")
def reverse_segment(tmp_path_factory):
    """reverse_walk_segment of the kernels' header, compiled for the host."""
    d = tmp_path_factory.mktemp("order")
    (d / "order.cpp").write_text('#include "tt_gdn_order.h"\n'
                                 'extern "C" int seg(int p, int n, int l, const int* off) { return tt::reverse_walk_segment(p, n, l, off); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(d / "order.cpp"), "-o", str(d / "order.so")], check=True)
    f = ctypes.CDLL(str(d / "order.so")).seg
    return lambda place, n, levels, off: f(place, n, levels, off.ctypes.data_as(ctypes.c_void_p))


def _spine(n):
    parent, seg, at = [-1], [3], 0
    for i in range(n):
        parent += [at, at]
        seg += [1 + i % 3, 2 + (i % 5) * 31]
        at = len(parent) - 1
    return T.tree_gdn_plan(parent, seg)


def _plans():
    return [_spine(12), _spine(40)] + [T.tree_gdn_plan(t.parent, t.seg_len) for t in
                                       (W.random_tree(910 + s, n_nodes=30, lo=1, hi=150, n_roots=1 + s % 3, p_zero=0.1) for s in range(3))]


def _walks(plan, reverse_segment):
    """(segment of every place, what every segment waits for) of the forward and of the reverse walk."""
    n = plan.n_segments
    saver = {int(plan.chunk_dst[c]): s for s in range(n) for c in range(plan.seg_chunk0[s], plan.seg_chunk1[s]) if plan.chunk_dst[c] >= 0}
    src = [int(plan.chunk_src[c]) for c in plan.seg_chunk0]
    fwd = {s: [saver[src[s]]] if src[s] >= 0 else [] for s in range(n)}
    rev = {s: [r for r in range(n) if fwd[r] == [s]] for s in range(n)}
    levels = plan.n_levels if plan.n_levels <= 32 else 0
    return [(list(range(n)), fwd), ([reverse_segment(p, n, levels, plan.level_off) for p in range(n)], rev)]


def test_a_segment_comes_behind_all_it_waits_for(reverse_segment):
    for plan in _plans():
        for order, waits in _walks(plan, reverse_segment):
            place = {s: p for p, s in enumerate(order)}
            assert sorted(order) == list(range(plan.n_segments))
            assert all(place[r] < place[s] for s in order for r in waits[s])
            assert any(waits.values())


def test_the_kernels_take_their_places_by_ticket():
    """All three walks start the same way, and the row of the block id counts only where nobody waits: what the model below stands for."""
    src = re.sub(r"//.*", "", open(os.path.join(CSRC, "tt_gdn.hip")).read())
    assert len(re.findall(r"\bwalk_start<(?:false|true)>\(a, ", src)) == 3
    assert re.findall(r".*blockIdx\.y.*", src) == [
        "  const int place = __builtin_amdgcn_readfirstlane(a.tickets ? place_of_all : a.seg_base + (int)blockIdx.y);"]


def _drains(launches, columns, cus, by_ticket, rng, in_order):
    """Runs the launches, each (order, waits), side by side; False if a state is reached in which nothing can go on."""
    share = [[[] for _ in launches] for _ in range(XCDS)]            # not yet started, by XCD and launch
    for li, (order, _) in enumerate(launches):
        for wg in range(len(order) * columns):
            share[wg % XCDS][li].append(wg)
    if not in_order:
        for x in range(XCDS):
            for ids in share[x]:
                rng.shuffle(ids)
    first = [rng.randrange(len(launches)) for _ in range(XCDS)]      # the launch that an XCD serves first
    tickets, done, running = {}, set(), [[] for _ in range(XCDS)]
    while True:
        moved = False
        for x in rng.sample(range(XCDS), XCDS):
            while len(running[x]) < cus and any(share[x]):
                li = first[x] if share[x][first[x]] else next(i for i, ids in enumerate(share[x]) if ids)
                wg, moved = share[x][li].pop(0), True
                col = wg % columns
                place = tickets.get((li, col), 0) if by_ticket else wg // columns
                tickets[li, col] = place + 1
                running[x].append((li, col, launches[li][0][place]))
            for it in list(running[x]):
                li, col, s = it
                if all((li, col, r) in done for r in launches[li][1][s]):
                    running[x].remove(it)
                    done.add(it)
                    moved = True
        if len(done) == columns * sum(len(order) for order, _ in launches):
            return True
        if not moved:
            return False


@pytest.mark.parametrize("columns", [1, 2, 4, 8, 12, 20])
def test_two_walks_side_by_side_always_end(reverse_segment, columns):
    """Few compute units stand for many segments: 2 per XCD.  Every order of starting workgroups must do, in order or not."""
    plans, rng = _plans(), random.Random(columns)
    walks = [w for p in plans for w in _walks(p, reverse_segment)]
    for trial in range(60):
        pair = rng.sample(walks, 2)
        assert _drains(pair, columns, 2, True, rng, in_order=trial % 2 == 0)


def test_the_model_sees_the_mistake(reverse_segment):
    """Places from block ids: one walk that is started in order ends, two walks of 4 columns stand still, and so does one that is
    started in another order."""
    rng, walks = random.Random(7), _walks(_spine(40), reverse_segment)
    assert all(_drains([w], 4, 2, False, rng, in_order=True) for w in walks)
    assert not all(_drains([walks[0], walks[0]], 4, 2, False, rng, in_order=True) for _ in range(200))
    assert not all(_drains([w], 4, 2, False, rng, in_order=False) for w in walks for _ in range(20))
