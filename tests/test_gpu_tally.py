"""The read statistics of smore_sample_negatives (stats) on graphs small enough
to count every read by hand: bytes of each kind of read, per draw and per
intersected list."""
import numpy as np
import pytest

import oracle
import paper_2110_14890_amd as sm
from gpu_common import require_gpu, to_numpy

pytestmark = pytest.mark.gpu

TAG_NEG = 2


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def pairs(heads, r, tails):
    h, t = np.meshgrid(heads, tails, indexing="ij")
    return np.stack([h.ravel(), np.full(h.size, r), t.ravel()], 1)


def run_caller_queries(g, qt, batch, n_neg, neg_tries, seed, anchors, relations, positive):
    """Rows and statistics of `batch` caller-built queries that are all alike."""
    import torch
    dag = sm.query_preset(qt)
    args = sm.make_args(batch, n_neg, seed=seed, neg_tries=neg_tries)
    out = sm.alloc_outputs(batch, n_neg)
    out["anchors"][:] = torch.tensor(anchors, dtype=torch.int32, device="cuda")
    out["relations"][:] = torch.tensor(relations, dtype=torch.int32, device="cuda")
    out["positive"][:] = positive
    stats = torch.zeros((batch, 4), dtype=torch.int64, device="cuda")
    sm.sample_negatives(g, dag, args, out, stats)
    return to_numpy(out), stats.cpu().numpy()


def search_reads(n):
    """Reads of one key's bisection in a list of n entries: a probe per
    halving and the last comparison."""
    probes = 0
    while n > 1:
        n -= n >> 1
        probes += 1
    return probes + 1


def hub_draws(V, seed, batch, tries, hubs):
    d = np.array([[oracle.pick(oracle.draw(seed, TAG_NEG, q, 0, j), V) for j in range(tries)]
                  for q in range(batch)])
    return np.isin(d, hubs)


# Anchors 0 and 1 have the forward lists F0, F1 under relation 0; the
# candidates of C have the same 2,000 heads under relation 1, none of them in
# F0 or F1, and nothing else has an in-edge under relation 1.  So of a query's
# draws exactly those in C go past the first test, each meets a list too long
# for the wavefront that drew it, and all of them cost the same reads.
V, HEADS, C = 8192, np.arange(2048, 4048), np.arange(4096, 4496)
F0, F1 = np.arange(16, 716), np.arange(720, 1520)
NODE_PAIR, ONE_GROUP = 8, 16     # a node entry and the next; a group and the next


@pytest.mark.parametrize("qt", ["2p", "ip", "up"])
def test_long_lists_are_counted_one_by_one(qt):
    tr = np.concatenate([pairs([0], 0, F0), pairs([1], 0, F1), pairs(HEADS, 1, C)]).astype(np.int32)
    g = sm.Graph(tr, V, 2)
    batch, tries, seed = 64, 300, 11     # one range of draws: [0, tries)
    two = qt != "2p"
    out, st = run_caller_queries(g, qt, batch, tries, tries, seed, [0, 1, -1] if two else [0, -1, -1],
                                 [0, 0, 1] if two else [0, 1, -1], int(C[0]))
    k = hub_draws(V, seed, batch, tries, C).sum(1)
    assert k.min() >= 2          # several long lists per query, or nothing is tested
    lookup = NODE_PAIR + ONE_GROUP
    cached = lookup + 4 * len(F0) + (lookup + 4 * len(F1) if two else 0)
    assert np.array_equal(st[:, 0], cached + 4 * tries + lookup * k)
    # the forward list's entries are the keys, 256 per step (the last step is
    # padded), each searched in the 2,000 heads; a union searches both lists
    steps = -(-len(F0) // 256) + (-(-len(F1) // 256) if qt == "up" else 0)
    searches = 256 * steps * search_reads(len(HEADS))
    assert np.array_equal(st[:, 2], (lookup + 4 * searches) * k)
    # a line per probe; the node pair and the group may straddle a line each
    assert ((searches + 2) * k <= st[:, 3]).all() and (st[:, 3] <= (searches + 4) * k).all()


# Half of the entities are candidates with 600 heads under relation 1, which
# hold the forward list: answers.  A query is short after its first range of
# draws and takes further ones, with long lists of their own.
@pytest.mark.parametrize("batch", [5, 64, 4096])
def test_further_draws_are_counted_alike(batch):
    V, f0, heads, c = 2048, np.arange(16, 536), np.arange(16, 616), np.arange(1024, 2048)
    tr = np.concatenate([pairs([0], 0, f0), pairs(heads, 1, c)]).astype(np.int32)
    g = sm.Graph(tr, V, 2)
    n_neg, tries, seed = 300, 1200, 12
    out, st = run_caller_queries(g, "2p", batch, n_neg, tries, seed, [0, -1, -1], [0, 1, -1], int(c[0]))
    rows = min(batch, 64)
    hub = np.concatenate([np.zeros((rows, 1), int), hub_draws(V, seed, rows, tries, c).cumsum(1)], 1)
    st, end = st[:rows], out["neg_draws"][:rows]
    lookup = NODE_PAIR + ONE_GROUP
    # every list is met within the first 256 of the forward list's entries
    each = lookup + 4 * 256 * search_reads(len(heads))
    k = st[:, 2] // each
    assert (k * each == st[:, 2]).all()
    taken = (st[:, 0] - (lookup + 4 * len(f0)) - lookup * k) // 4     # draws
    assert (4 * taken + lookup * k + lookup + 4 * len(f0) == st[:, 0]).all()
    assert (taken >= end).all() and (taken <= tries).all() and (taken > 400).all()
    assert np.array_equal(hub[np.arange(rows), taken], k)


def lines(first, nbytes):
    """64-byte lines of nbytes from byte offset first of a device array."""
    return (first + nbytes - 1) // 64 - first // 64 + 1


def rev_list(g, node, grp, v):
    """First edge and length of an entity's only in-group, and the lines of
    looking it up."""
    i = int(node[v])
    assert node[v + 1] == i + 1
    beg, end = int(grp[i, 1]), int(grp[i + 1, 1])
    return beg, end - beg, lines(4 * v, NODE_PAIR) + lines(8 * i, ONE_GROUP)


# A list that a wavefront walks is one contiguous read of its entries, not a
# line per entry.  2p: 64 heads per candidate, a forward list of 200 without
# them; 3p: 8 in-neighbours per candidate with 16 heads each, few enough steps
# for a wavefront of any call.
@pytest.mark.parametrize("qt,tries", [("2p", 100), ("3p", 12)])
def test_walked_lists_are_counted_in_lines(qt, tries):
    V, batch, seed = 4096, 64, 13
    f0, c = np.arange(16, 216), np.arange(2048, 2448)
    if qt == "2p":
        tr = [pairs([0], 0, f0), pairs(np.arange(512, 576), 1, c)]
    else:
        ys = np.arange(600, 608)
        tr = [pairs([0], 0, f0), pairs(np.arange(512, 528), 1, ys), pairs(ys, 2, c)]
    g = sm.Graph(np.concatenate(tr).astype(np.int32), V, 3)
    out, st = run_caller_queries(g, qt, batch, tries, tries, seed, [0, -1, -1],
                                 [0, 1, -1] if qt == "2p" else [0, 1, 2], int(c[0]))
    node, grp = g.copy(3, V + 1), g.copy(4, 2 * (g.S_rev + 1)).reshape(-1, 2)
    draws = [[oracle.pick(oracle.draw(seed, TAG_NEG, q, 0, j), V) for j in range(tries)] for q in range(batch)]
    checked = 0
    for q in range(batch):
        if st[q, 2]:              # lists left to another kernel (more than a wavefront may walk)
            continue
        want_b = NODE_PAIR + ONE_GROUP + 4 * len(f0) + 4 * tries
        want_l = 1 + 1 + lines(0, 4 * len(f0)) + tries
        hubs = [d for d in draws[q] if d >= c[0] and d <= c[-1]]
        checked += len(hubs)
        for d in hubs:
            beg, n, look = rev_list(g, node, grp, d)
            want_b += NODE_PAIR + ONE_GROUP + 4 * n
            want_l += look + lines(4 * beg, 4 * n)
            for y in ys if qt == "3p" else []:
                ybeg, yn, ylook = rev_list(g, node, grp, y)
                want_b += 1 + NODE_PAIR + ONE_GROUP + 4 * yn      # the signature byte first
                want_l += 1 + ylook + lines(4 * ybeg, 4 * yn)
        assert (int(st[q, 0]), int(st[q, 1])) == (want_b, want_l), q
    assert checked > 20
