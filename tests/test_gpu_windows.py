"""GPU parity at the edges of the candidate kernel's windows and limits.

A query is one wavefront that draws, verifies and selects window after
window; lists it must not walk itself go to the long-list kernels and the
query to the finishing kernel.  Every output is compared with the CPU oracle,
element by element.
"""
import numpy as np
import pytest

import kgsynth
import paper_2110_14890_amd as sm
from gpu_common import assert_same, gpu_sample, graph_pair, progress, require_gpu
from test_gpu_parity import hub_graph_3p

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


# n_neg 551 is the longest row whose first draws (n_neg + n_neg / 32 + 8) are
# one window of 576, with the selection table over the staged lists; 552 the
# shortest with its own, and with a second window of one draw where the budget
# or the batch leaves its 577 as they are
@pytest.mark.parametrize("n_neg,neg_tries", [(1, 2), (56, 64), (57, 200), (549, 576), (550, 1000),
                                             (551, 1000), (552, 1000), (552, 577), (536, 2144), (537, 2148),
                                             (551, 2204), (560, 4096), (1100, 1200), (4096, 4096)])
def test_rows_around_the_window(n_neg, neg_tries):
    rng = np.random.default_rng(21)
    tr = kgsynth.random_tiny(rng, 6000, 4, 90000)
    g, og = graph_pair(tr, 6000, 4, False)
    for qt in ("1p", "3p", "ip", "pni"):
        progress(f"window {qt} n_neg {n_neg}")
        got = gpu_sample(g, qt, 65, n_neg, seed=2, neg_tries=neg_tries)
        ref = og.sample(qt, 65, n_neg, seed=2, neg_tries=neg_tries)
        assert_same(got, ref, what=f"{qt} n_neg {n_neg}")


@pytest.mark.parametrize("n_neg", [551, 552])
def test_rows_around_the_window_of_a_full_batch(n_neg):
    rng = np.random.default_rng(25)
    tr = kgsynth.random_tiny(rng, 6000, 4, 90000)
    g, og = graph_pair(tr, 6000, 4, False)
    for qt in ("1p", "ip"):
        progress(f"full batch {qt} n_neg {n_neg}")
        got = gpu_sample(g, qt, 4096, n_neg, seed=2)
        ref = og.sample(qt, 4096, n_neg, seed=2)
        assert_same(got, ref, what=f"{qt} n_neg {n_neg}")


# 30 entities for up to 600 draws: nearly every draw repeats an earlier one,
# within a step of 64, within a window and across windows
@pytest.mark.parametrize("batch", [33, 4096])
@pytest.mark.parametrize("qt", ["1p", "2p", "2u", "pin"])
def test_repeated_draws(qt, batch):
    rng = np.random.default_rng(22)
    tr = kgsynth.random_tiny(rng, 30, 3, 150)
    g, og = graph_pair(tr, 30, 3, False)
    for n_neg, nt in [(20, 80), (29, 600)]:
        got = gpu_sample(g, qt, batch, n_neg, seed=3, neg_tries=nt)
        ref = og.sample(qt, batch, n_neg, seed=3, neg_tries=nt)
        assert_same(got, ref, what=f"{qt} n_neg {n_neg}")


# every backward list and forward list longer than a wavefront may walk:
# queries deferred to the long-list kernels and finished after them
@pytest.mark.parametrize("qt", ["2p", "3p", "ip", "pi", "up", "inp", "pin", "pni"])
def test_long_lists_on_hub_graph(qt):
    tr, V, R = hub_graph_3p()
    # a second way into every y, so that two branches can meet there
    extra = np.stack([np.full(400, 5), np.zeros(400, int), np.arange(2500, 2900)], 1)
    tr = np.concatenate([tr, extra.astype(np.int32)])
    g, og = graph_pair(tr, V, R)
    for n_neg, nt in [(64, 300), (600, 2000)]:
        progress(f"hub {qt} n_neg {n_neg}")
        got = gpu_sample(g, qt, 150, n_neg, seed=4, neg_tries=nt)
        ref = og.sample(qt, 150, n_neg, seed=4, neg_tries=nt)
        assert_same(got, ref, what=f"hub {qt} n_neg {n_neg}")


# attempt lanes per query: 64 and 32 under a maximum expansion, 16, 8 and 4
# for plans with root siblings or a complemented operand; attempt budgets
# that are no multiple of the lanes
@pytest.mark.parametrize("qt,batch,max_fanout", [("2p", 7, 3), ("ip", 1025, 3), ("pni", 2049, 5), ("3i", 70, 0),
                                                 ("3in", 4097, 0), ("2u", 9000, 0), ("up", 300, 2)])
def test_attempt_lanes(qt, batch, max_fanout):
    rng = np.random.default_rng(23)
    tr = kgsynth.random_tiny(rng, 2000, 5, 12000)
    g, og = graph_pair(tr, 2000, 5, False)
    for pos_tries in (1, 5, 64, 67):
        got = gpu_sample(g, qt, batch, 4, seed=6, pos_tries=pos_tries, max_fanout=max_fanout)
        ref = og.sample(qt, batch, 4, seed=6, pos_tries=pos_tries, max_fanout=max_fanout)
        assert_same(got, ref, what=f"{qt} batch {batch} pos_tries {pos_tries}")


# the first test of a draw reads the signatures up to 2^22 entities, the
# in-edge mask up to 2^26, the coarse mask above
@pytest.mark.parametrize("V", [1 << 22, (1 << 22) + 1, 1 << 24, (1 << 24) + 1, 1 << 26, (1 << 26) + 1])
def test_first_test_by_graph_size(V):
    rng = np.random.default_rng(24)
    ents = rng.choice(V, 60_000, replace=False).astype(np.int32)
    ents[:2] = 0, V - 1
    tr = np.stack([ents[rng.integers(0, len(ents), 200_000)], rng.integers(0, 40, 200_000),
                   ents[rng.integers(0, len(ents), 200_000)]], axis=1).astype(np.int32)
    g, og = graph_pair(tr, V, 40, False)
    for qt in ("1p", "2p", "3p", "2u", "up", "pin"):
        progress(f"V {V} {qt}")
        got = gpu_sample(g, qt, 200, 300, seed=7)
        ref = og.sample(qt, 200, 300, seed=7)
        assert_same(got, ref, what=f"V {V} {qt}")
