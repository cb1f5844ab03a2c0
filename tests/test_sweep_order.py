"""The order in which the sweep's slices read, count and store, by enumeration (CPU).

A model of the sweep kernel's wavefronts: wavefront w takes slices w, w + W, ...; a slice
waits until the slices of all earlier levels are counted, then counts, then stores its
results to memory, then makes that known.  A slow slice reads older results from memory
before it counts and waits beforehand until the earlier levels' slices are stored.  Every
interleaving is visited: with the rule that the kernel uses (every wavefront's first slice
that is not stored yet lies at or behind the level's first) no slow slice reads a result
that is not stored, and every run ends; with the number of stored slices instead there are
interleavings in which one does, as soon as a level mixes slow slices with others."""
import pytest


def explore(levels, waves, rule):
    """levels: a string per level, a letter per slice (f: fast, s: slow).  Returns (a slow slice
    can read too early, some run cannot end)."""
    kind = "".join(levels)
    dep = [sum(map(len, levels[:k])) for k, lv in enumerate(levels) for _ in lv]
    n = len(kind)
    # per wavefront: its slice and what that has done (0: nothing, 1: counted, 2: stored)
    start = tuple((w, 0) for w in range(waves))
    seen, todo, early, stuck = {start}, [start], False, False
    while todo:
        state = todo.pop()
        counted = sum(min(len(range(i % waves, i, waves)), n) + (at > 0) for i, at in state)
        known = sum(len(range(i % waves, min(i, n), waves)) for i, _ in state)
        stored = {j for i, at in state for j in range(i % waves, min(i, n), waves)} | {i for i, at in state if at == 2}
        moved = False
        for w, (i, at) in enumerate(state):
            if i >= n:
                continue
            if at == 0:
                if counted < dep[i]:
                    continue
                if kind[i] == "s":
                    ready = known >= dep[i] if rule == "sum" else all(j >= dep[i] for j, _ in state)
                    if not ready:
                        continue
                    early |= any(j not in stored for j in range(dep[i]))
            moved = True
            new = state[:w] + (((i, at + 1) if at < 2 else (i + waves, 0)),) + state[w + 1:]
            if new not in seen:
                seen.add(new)
                todo.append(new)
        stuck |= not moved and any(i < n for i, _ in state)
    return early, stuck


MIXED = [["ff", "fs"], ["f", "sf", "fss"], ["ff", "ffs", "sf"], ["fff", "sfff", "fs"], ["ffff", "ssff", "s"], ["ss", "sf", "fsf"]]


@pytest.mark.parametrize("waves", [1, 2, 3, 4])
@pytest.mark.parametrize("levels", MIXED + [["ff", "ss", "ss"], ["fff", "fff"]])
def test_slow_slices_read_stored_results(levels, waves):
    assert explore(levels, waves, "each") == (False, False)


@pytest.mark.parametrize("levels", MIXED)
def test_a_sum_of_stored_slices_is_not_enough(levels):
    early = [explore(levels, w, "sum")[0] for w in (2, 3, 4)]
    assert any(early)
    assert not explore(levels, 1, "sum")[0]


def test_a_sum_is_enough_where_all_slices_of_a_level_are_slow():
    for w in (2, 3, 4):
        assert explore(["ff", "ss", "ss"], w, "sum") == (False, False)
