"""Calls of few queries whose draws are mostly answers or meet long lists: the
rows (against the CPU oracle), and that such a call does not last as long as
one that fills the GPU with the same queries: its work has to be spread."""
import numpy as np
import pytest

import kgsynth
import paper_2110_14890_amd as sm
from gpu_common import assert_same, gpu_sample, graph_pair, progress, require_gpu, to_numpy
from test_gpu_parity import hub_graph_3p

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


LONG = ["2p", "3p", "ip", "pi", "up", "inp", "pin", "pni"]


# batches at the edges of the finishing kernel's workgroup sizes; budgets
# that end within a range, within a block of 64 draws and at a draw
@pytest.mark.parametrize("qt", LONG)
@pytest.mark.parametrize("batch", [1, 3, 256, 257, 512, 513])
def test_rows_of_small_calls(qt, batch):
    rng = np.random.default_rng(41)
    tr = kgsynth.random_tiny(rng, 500, 3, 20000)
    g, og = graph_pair(tr, 500, 3)
    for n_neg, tries in [(1, 7), (64, 256), (200, 801), (300, 2000)]:
        got = gpu_sample(g, qt, batch, n_neg, seed=5, neg_tries=tries)
        ref = og.sample(qt, batch, n_neg, seed=5, neg_tries=tries)
        assert_same(got, ref, what=f"{qt} batch {batch} n_neg {n_neg}")
        if batch >= 256 and tries > 7 and qt in ("2p", "3p", "up"):
            assert (got["neg_draws"] > n_neg + n_neg // 32 + 72).any()   # further draws were needed


def call_ms(g, qt, batch, n_neg):
    import torch
    dag, ws, out = sm.query_preset(qt), sm.Workspace(), sm.alloc_outputs(batch, n_neg)
    a, z = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = float("inf")
    for k in range(6):
        args = sm.make_args(batch, n_neg, seed=6, query_offset=k * batch, neg_tries=4 * n_neg)
        a.record()
        sm.sample_into(g, dag, args, out, workspace=ws)
        z.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(z)) if k else best
    return best


@pytest.mark.parametrize("qt", ["2p", "3p", "ip"])
def test_small_calls_are_spread_over_the_gpu(qt):
    rng = np.random.default_rng(42)
    g = sm.Graph(kgsynth.random_tiny(rng, 2000, 3, 300000), 2000, 3)
    few, many = call_ms(g, qt, 16, 1000), call_ms(g, qt, 1024, 1000)
    progress(f"{qt}: 16 queries {few:.2f} ms, 1,024 queries {many:.2f} ms")
    assert few < 0.5 * many


# the lists of hubs, and of 3p the units, where several workgroups share a query
@pytest.mark.parametrize("qt", LONG)
def test_few_queries_on_hub_graph(qt):
    tr, V, R = hub_graph_3p()
    extra = np.stack([np.full(400, 5), np.zeros(400, int), np.arange(2500, 2900)], 1)
    tr = np.concatenate([tr, extra.astype(np.int32)])
    g, og = graph_pair(tr, V, R)
    for batch, n_neg, tries in [(1, 40, 160), (12, 500, 2000), (130, 3900, 4096)]:
        progress(f"hub {qt} batch {batch}")
        got = gpu_sample(g, qt, batch, n_neg, seed=8, neg_tries=tries)
        ref = og.sample(qt, batch, n_neg, seed=8, neg_tries=tries)
        assert_same(got, ref, what=f"hub {qt} batch {batch}")


# one query cannot be dealt over workgroups but by its draws: its call stays
# near that of 256 of them
@pytest.mark.parametrize("qt", ["2p", "ip"])
def test_one_query_is_shared_by_workgroups(qt):
    rng = np.random.default_rng(42)
    g = sm.Graph(kgsynth.random_tiny(rng, 2000, 3, 300000), 2000, 3)
    one, many = call_ms(g, qt, 4, 1000), call_ms(g, qt, 256, 1000)
    progress(f"{qt}: 4 queries {one:.2f} ms, 256 queries {many:.2f} ms")
    assert one < 0.6 * many


# Beside a call that holds the GPU the workgroups that share a query start at
# different times, some after others have settled draws: they all have to come
# to the same shares of it.
@pytest.mark.parametrize("qt", LONG)
def test_shared_queries_beside_a_call_that_fills_the_gpu(qt):
    import torch
    rng = np.random.default_rng(43)
    g, og = graph_pair(kgsynth.random_tiny(rng, 2000, 3, 300000), 2000, 3)
    busy, here = torch.cuda.Stream(), torch.cuda.Stream()
    big = sm.alloc_outputs(16384, 512)
    big_ws, ws = sm.Workspace(), sm.Workspace()
    outs = [sm.alloc_outputs(16, 500) for _ in range(8)]
    torch.cuda.synchronize()
    for k, out in enumerate(outs):
        sm.sample_into(g, sm.query_preset("1p"), sm.make_args(16384, 512, seed=1), big, stream=busy, workspace=big_ws)
        sm.sample_into(g, sm.query_preset(qt), sm.make_args(16, 500, seed=9, query_offset=16 * k), out,
                       stream=here, workspace=ws)
    torch.cuda.synchronize()
    for k, out in enumerate(outs):
        ref = og.sample(qt, 16, 500, seed=9, query_offset=16 * k, neg_tries=2000)
        assert_same(to_numpy(out), ref, what=f"{qt} call {k}")


# 3p calls that fill the GPU have fewer wavefronts per query
def test_further_draws_of_a_full_3p_batch():
    rng = np.random.default_rng(44)
    g, og = graph_pair(kgsynth.random_tiny(rng, 500, 3, 20000), 500, 3)
    got = gpu_sample(g, "3p", 4097, 100, seed=5, neg_tries=500)
    assert_same(got, og.sample("3p", 4097, 100, seed=5, neg_tries=500), what="3p batch 4097")
