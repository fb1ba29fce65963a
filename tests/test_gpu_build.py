"""GPU parity of the graph build where its sort digits span fields: entity and
relation counts whose bit widths put one, two or three fields into a digit,
and record counts around the sort's tile, against the oracle's adjacency."""
import numpy as np
import pytest

import kgsynth
from gpu_common import graph_pair, require_gpu
from test_gpu_parity import check_graph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("V,R,n,inverse", [(2, 1, 9, False), (3, 2, 40, True), (7, 5, 300, False), (256, 1, 4096, False),
                                           (257, 255, 4097, False), (1000, 20, 8191, True), (65536, 3, 20000, False),
                                           (65537, 300, 20000, True), (1 << 20, 1 << 14, 30000, False)])
def test_build_over_field_widths(V, R, n, inverse):
    rng = np.random.default_rng(31)
    tr = kgsynth.random_tiny(rng, V, R, n)
    tr[-1] = (V - 1, R - 1, V - 1)      # the largest ids
    g, og = graph_pair(tr, V, R, inverse)
    check_graph(g, og)
