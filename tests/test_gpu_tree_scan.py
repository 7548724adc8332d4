"""The node scan of draft trees at its edges: one node, a wave of nodes and one more, the most nodes a window may have (paths of
every length up to 1023), in the split form (from 28 nodes on, up to 1024 verify rows) and in the one launch."""
import numpy as np
import pytest

import oracle
import workloads as wl
from parity import make_inputs
from test_gpu_tree import check, random_trees, run_tree, tree_drafts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,K,shape,p_match", [
    (3, 1, "star", 0.5), (2, 16, "bushy", 0.8), (1, 17, "bushy", 0.8), (1, 31, "bushy", 0.8), (3, 27, "random", 0.8), (3, 28, "random", 0.8), (17, 64, "random", 0.8), (17, 65, "chain", 0.97), (40, 1, "star", 0.5), (1, 32, "bushy", 0.8), (2, 64, "random", 0.7), (2, 65, "chain", 0.97),
    (1, 1023, "chain", 0.999), (1, 1023, "bushy", 0.9), (2, 1023, "chain", 0.999), (2, 600, "random", 0.8), (16, 63, "bushy", 0.8),
    (17, 63, "bushy", 0.8),
])
@pytest.mark.parametrize("feat_offset", [1, 0])
def test_tree_scan_edges(B, K, shape, p_match, feat_offset):
    w = wl.scaled(wl.WORKLOADS["8b_b1_k16"], name="scan", B=B, K=K, d_t=64, d_d=8, V=400)
    x = make_inputs(w, 9)
    greedy = oracle.greedy_rows(x.ht, x.W)
    rng = np.random.default_rng(K + B)
    parent = random_trees(rng, B, K, shape)
    draft = tree_drafts(rng, greedy[0].reshape(B, K + 1), parent, w.V, p_match)
    for tau in (0.0, 0.5):
        check(x, draft, parent, tau, run_tree(x, draft, parent, tau, feat_offset), greedy, feat_offset)
