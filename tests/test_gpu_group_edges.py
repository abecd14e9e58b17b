"""Exact parity of haste_group_labels with the oracle at the edges of its kernels: one label, clusters of
exactly and just over 2048 members (the two greedy kernels), rows all equal (every choice a tie), widths
at and past the 256-, 512- and 768-dimension tiles, one label per group (many clusters), groups as large
as a cluster, label counts that leave part of a workgroup's labels and of a counting tile, and both sizes of its waves' share."""
import numpy as np
import pytest

import oracle
from gpu_helpers import say
from test_gpu_group import _run, planted, uneven

pytestmark = pytest.mark.gpu

# N, D, planted directions (0: all rows equal, -1: uneven norms), G, beta, iters
CASES = [(1, 16, 1, 4, 1, 2), (2048, 32, 3, 32, 64, 2), (2049, 32, 3, 32, 65, 2), (700, 48, 0, 16, 40, 1), (70, 16, 5, 1, 1, 2),
         (1500, 272, -1, 256, 3, 2), (1025, 528, 7, 8, 16, 2), (513, 1024, 4, 16, 8, 2), (3001, 784, 9, 5, 20, 3), (40, 64, 2, 64, 1, 1),
         # more labels than one workgroup of 256 per CU takes, at each width of the assignment's tiles
         (65600, 48, 40, 64, 64, 1), (66000, 272, 40, 256, 16, 1), (66001, 528, 40, 256, 16, 1), (65537, 784, 40, 256, 16, 1)]


@pytest.mark.parametrize("case", CASES)
def test_group_edges(case):
    import paper_2606_01117_amd as hs
    N, D, P, G, beta, iters = case
    say("[group]", case)
    rng = np.random.default_rng(N * 7 + D)
    E = np.tile(rng.integers(-127, 128, (1, D)).astype(np.int8), (N, 1)) if P == 0 else \
        uneven(N, D, rng) if P < 0 else planted(N, D, P, rng)
    order, gs, cl = _run(hs, E, G, beta, iters, 77 + N)
    order_o, gs_o, cl_o = oracle.get().group_labels(E, G, beta, iters, 77 + N)
    assert np.array_equal(cl, cl_o) and np.array_equal(gs, gs_o) and np.array_equal(order, order_o)
