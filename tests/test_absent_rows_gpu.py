"""Rows of nodes that a tree does not have are not written to logits_out."""

from dataclasses import replace

import numpy as np
import pytest
import torch

from workloads import gen
from workloads.configs import SMALL_GQA

pytestmark = pytest.mark.gpu


# one row tile (whole and half), several sequences in one tile, several tiles; rows of whole 16-byte groups and not
@pytest.mark.parametrize("vocab", [1000, 1001])
@pytest.mark.parametrize("max_tree,nodes", [(64, (40,)), (64, (3,)), (20, (5, 20, 1)), (64, (9, 64, 1)), (40, (2, 33, 40))])
def test_logits_of_absent_nodes_are_left_alone(max_tree, nodes, vocab):
    import paper_2502_11018_amd as P
    m = replace(SMALL_GQA, name="absent", n_layers=1, vocab=vocab)
    mw, B = gen.make_weights(m, 5), len(nodes)
    trees = [gen.random_tree([w for w in (min(n - 1, 8), max(0, n - 9)) if w], vocab, 3 + b)[0]
             for b, n in enumerate(nodes)]
    assert tuple(t.n for t in trees) == nodes
    with P.TreeVerifier(m, mw.to("cuda"), max_batch=B, max_tree=max_tree, max_depth=8, kv_capacity=128) as v:
        print(f"[gpu-case] absent rows vocab {vocab} max_tree {max_tree} nodes {nodes}", flush=True)
        out = torch.full((B, max_tree, vocab), 7.0, device="cuda")
        v.step([0] * B, trees, out)
        pred = v.predictions()
        lg = out.cpu().numpy()
    for b, n in enumerate(nodes):
        assert (lg[b, n:] == 7.0).all(), b
        assert not (lg[b, :n] == 7.0).any() and np.array_equal(lg[b, :n].argmax(axis=1), pred[b, :n])
