"""Systems whose work groups take the branches of the group-size rule and of
the choice between two, three and four launches per iteration."""

import functools

import numpy as np

import synth


def _grid(m):
    """Edges of an m x m grid with one diagonal per cell."""
    k = np.arange(m * m).reshape(m, m)
    pairs = [(k[:, :-1], k[:, 1:]), (k[:-1], k[1:]), (k[:-1, :-1], k[1:, 1:])]
    return np.concatenate([np.stack([a.ravel(), b.ravel()], 1) for a, b in pairs])


# grid, hub (node 0 coupled with that many others, evenly spread), clique (so
# many nodes of the first rows all coupled) -> domains per group, unit lists
# (two launches; else three)
SYSTEMS = {
    "even": ((112, 0, 0), 2, True),
    "wide": ((112, 3000, 0), 2, False),        # node 0's group reads more units than the lists hold
    "wide_heavy": ((112, 9000, 0), 1, False),  # and its window halves the groups
    "heavy": ((112, 0, 160), 1, True),         # the window alone does
}


@functools.lru_cache(maxsize=None)
def system(name):
    m, hub, clique = SYSTEMS[name][0]
    n, grid = m * m, _grid(m)
    e = [grid]
    if hub:
        e.append(np.stack([np.zeros(hub, int), 1 + np.arange(hub) * ((n - 1) // hub)], 1))
    if clique:
        side = int(clique ** 0.5) + 1
        near = (np.arange(side)[:, None] * m + np.arange(side)).ravel()[:clique]
        a, b = np.triu_indices(clique, 1)
        e.append(np.stack([near[a], near[b]], 1))
    e = np.unique(np.sort(np.concatenate(e), axis=1), axis=0)
    s = synth.bcsr.spd_system_from_edges(n, e, seed=n + hub + clique)
    s.gptr, s.gadj = synth.bcsr.graph_from_edges(n, grid)  # the couplings come later than the partition
    return s


# nodes of a line, 16 to a domain -> domains per group: both sides of 384,
# 1,536 and 4,096 domains
EDGES = [(6144, 1), (6160, 2), (24576, 2), (24592, 4), (65536, 4), (65552, 8)]


@functools.lru_cache(maxsize=2)
def line(n):
    """A line with some second neighbours."""
    i = np.arange(n)
    e = np.concatenate([np.stack([i[:-1], i[1:]], 1), np.stack([i[:-5:3], i[5::3]], 1)])
    return synth.bcsr.spd_system_from_edges(n, e, seed=n)
