"""Optimal connected subgraph of graphs too large to enumerate on the CPU: forests, whose optimum, mask and number of connected
sets a recursion over the trees gives.  Both searches of the GPU, over all their tables and several pairs a thread."""
import numpy as np
import pytest
import torch

DEV = "cuda:0"


def forest_graph(N, window, roots, counts, parents=(0, 64), seed=0):
    """Random forest of N nodes under shuffled numbers: a node that is not root-level has its one parent among the last
    `window` nodes.  `parents` = range for the number of nodes with such a child; rows that change nothing are mixed in.
    counts: "ties", "wide", "high" (the best set reaches a parent with 24 parents of lower number) or the sum of |count|."""
    for seed in range(seed, seed + 1000):
        r = np.random.default_rng(seed)
        label = r.permutation(N)
        first = sorted({0} | {int(q) for q in r.choice(np.arange(1, N), roots - 1, replace=False)})
        parent = [-1] * N
        for i in range(N):
            if i not in first:
                parent[label[i]] = int(label[r.integers(max(0, i - window), i)])
        order = sorted({p for p in parent if p >= 0})
        if parents[0] <= len(order) <= parents[1]:
            break
    else:
        raise AssertionError("no such forest")
    level = np.array([3 + i % 4 if p >= 0 else 1 + i % 2 for i, p in enumerate(parent)], np.int32)
    is_root = [q for q in range(N) if parent[q] < 0]
    edges = [(p, q) for q, p in enumerate(parent) if p >= 0]
    edges += [(int(r.integers(N)), q) for q in is_root] + [(is_root[0], is_root[0]), edges[0], (-1, 2), (1, N)]
    edges = np.asarray([edges[i] for i in r.permutation(len(edges))], np.int32)
    if counts == "ties":
        count = r.integers(0, 3, N)
    elif isinstance(counts, str):
        count = r.integers(-1000, 10 ** 6, N)
    else:
        share = r.random(N)
        count = np.floor(share / share.sum() * counts).astype(np.int64)
        count[0] += counts - int(count.sum())
        count *= np.where(r.random(N) < 0.2, -1, 1)
        assert int(np.abs(count).sum()) == counts
    count = count.astype(np.int64)
    if counts == "high":
        def path(q):
            return [q] + (path(parent[q]) if parent[q] >= 0 else [])
        count[min((path(q) for q in order[24:]), key=len)] += 10 ** 7
    return count, level, edges, parent


def forest_search(count, parent, D):
    """What the oracle's subgraph_search returns, by recursion: per subtree and size the best (sum, -mask) of the sets that
    hold its top, both parts adding up over disjoint subtrees, and their number."""
    N = len(count)
    kids = [[q for q in range(N) if parent[q] == p] for p in range(N)]

    def join(a, b):
        out = {}
        for i, (s, m, n) in a.items():
            for j, (s2, m2, n2) in b.items():
                if i + j <= D:
                    best, had = out.get(i + j, (None, 0))
                    new = (s + s2, m + m2)
                    out[i + j] = (new if best is None or new > best else best, had + n * n2)
        return {k: (v[0][0], v[0][1], v[1]) for k, v in out.items()}

    def top(q):
        t = {1: (int(count[q]), -(1 << q), 1)}
        for c in kids[q]:
            t = join(t, {0: (0, 0, 1), **top(c)})
        return t

    total = {0: (0, 0, 1)}
    for q in range(N):
        if parent[q] < 0:
            total = join(total, {0: (0, 0, 1), **top(q)})
    if D not in total:
        return dict(best_nodes=[], best_mask=0, best_sum=0, n_connected=0)
    s, m, n = total[D]
    return dict(best_nodes=[q for q in range(N) if -m >> q & 1], best_mask=-m, best_sum=s, n_connected=n)


@pytest.mark.parametrize("N,window,roots,D,counts", [(9, 1, 1, 4, "wide"), (12, 2, 3, 5, "ties"), (14, 3, 4, 6, "ties"),
                                                     (16, 2, 2, 5, 1 << 40), (13, 13, 1, 13, "wide"), (8, 1, 1, 9, "ties")])
def test_forest_recursion_equals_the_oracle(N, window, roots, D, counts):
    from oracle import spiffy_oracle as O
    count, level, edges, parent = forest_graph(N, window, roots, counts)
    assert forest_search(count, parent, D) == O.subgraph_search(count, level, edges, D)


@pytest.mark.gpu
@pytest.mark.parametrize("N,window,roots,D,counts,parents", [
    # sets one by one (more than 30 parents): several workgroups, several (top, middle) pairs a thread
    (36, 1, 5, 6, "ties", (31, 64)), (40, 1, 9, 8, "wide", (31, 64)), (45, 1, 13, 9, "ties", (31, 64)),
    (50, 2, 12, 7, "wide", (31, 64)), (64, 1, 24, 6, "ties", (31, 64)), (64, 3, 20, 5, "wide", (31, 64)),
    # ... and 32-bit sums while |count| adds up to less than 2^30
    (40, 1, 8, 7, 1 << 29, (31, 64)), (40, 1, 8, 7, (1 << 30) - 1, (31, 64)), (40, 1, 8, 7, 1 << 30, (31, 64)),
    (40, 1, 8, 7, 1 << 41, (31, 64)),
    # choices of 25 to 30 parents: all four tables
    (40, 2, 8, 9, "high", (25, 26)), (40, 2, 8, 9, "ties", (25, 26)), (42, 2, 7, 9, "high", (27, 28)),
    (45, 2, 7, 10, "high", (29, 30)), (45, 2, 8, 10, 1 << 45, (29, 30)), (45, 2, 8, 10, "ties", (29, 30))])
def test_subgraph_search_of_forests(N, window, roots, D, counts, parents):
    from paper_2509_18085_amd import spiffy as sp
    count, level, edges, parent = forest_graph(N, window, roots, counts, parents)
    ref = forest_search(count, parent, D)
    assert ref["n_connected"] > 0
    if counts == "high":
        order = sorted({p for p in parent if p >= 0})
        assert any(q in order[24:] for q in ref["best_nodes"])
    out = sp.subgraph_search(torch.from_numpy(count).to(DEV), torch.from_numpy(level).to(DEV),
                             torch.from_numpy(edges).to(DEV), D)
    torch.cuda.synchronize()
    got = dict(best_nodes=[q for q in out["nodes"].cpu().tolist()[:D] if q >= 0],
               best_mask=int(out["best_mask"].cpu().numpy().view(np.uint64)[0]), best_sum=int(out["best_sum"].item()),
               n_connected=int(out["n_connected"].item()))
    assert got == ref, (got, ref)
