"""Rows of nodes that a tree does not have are not written: logits_out of a verify
step, the top-k of a draft pass."""

from dataclasses import replace

import numpy as np
import pytest
import torch

from workloads import gen
from workloads.configs import DRAFTS, SMALL_GQA

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


def test_topk_of_absent_nodes_is_left_alone():
    import paper_2502_11018_amd as P
    from paper_2502_11018_amd import _native as N
    ds, T, k, B = DRAFTS["tiny"], 16, 4, 2
    mw, dw = gen.make_weights(ds.target, 0), gen.make_draft_weights(ds, 3)
    feat = gen.draft_root_features(ds.target.d_model, B, 11).cuda()
    trees = [gen.random_tree((4,), ds.target.vocab, 1)[0], gen.chain_tree(5, [])]
    p32 = lambda x: x.ctypes.data_as(N.POINTER(N.c_int32))  # noqa: E731
    with P.DraftModel(ds, dw.to("cuda"), mw.to("cuda"), max_batch=B, max_tree=T, max_depth=4, kv_capacity=64) as dm:
        n, tok, par = P.pack_trees(trees, T)
        prefix = np.zeros(B, np.int32)
        ktok, klp = np.full((B, T, k), -7, np.int32), np.full((B, T, k), 7.0, np.float32)
        print("[gpu-case] draft top-k of absent nodes", flush=True)
        rc = N.lib.griffin_draft_step(dm.h, B, p32(prefix), p32(n), p32(tok), p32(par), N.c_void_p(feat.data_ptr()), k,
                                      p32(ktok), klp.ctypes.data_as(N.POINTER(N.c_float)))
        assert rc == 0
    for b, t in enumerate(trees):
        assert (ktok[b, t.n:] == -7).all() and (klp[b, t.n:] == 7.0).all()
        assert (ktok[b, : t.n] >= 0).all() and (klp[b, : t.n] <= 0).all()
