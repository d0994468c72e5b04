"""The prefix attention against the fp64 oracle over the forms its launch takes:
row tiles per KV head (one head's 32 rows each, or a short chain's heads packed
into one tile), waves per workgroup, ragged and uniform key splits, and prefixes
at the edges of the 32-key blocks."""

from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from workloads import gen
from workloads.configs import SMALL_GQA
from tests import harness as H

pytestmark = pytest.mark.gpu

PREFIXES = (0, 1, 31, 32, 33, 64, 161, 423)


def _model(hq, hkv, dh):
    return replace(SMALL_GQA, name=f"attn-{hq}-{hkv}-{dh}", n_layers=1, d_model=256, n_q_heads=hq, n_kv_heads=hkv,
                   head_dim=dh, d_ff=256, vocab=520)


# (query heads, KV heads, head dim, max_tree, nodes): packed tiles full (8 x 4 = 32
# rows), partly filled and of one node; one row too many to pack (9 x 4); one, two, three
# and more row tiles per KV head, the last workgroup of three tiles half empty
@pytest.mark.parametrize("hq,hkv,dh,max_tree,nodes", [
    (8, 2, 128, 8, 8), (8, 2, 128, 3, 3), (8, 2, 64, 5, 1), (8, 2, 128, 9, 9), (3, 3, 128, 64, 50), (4, 4, 64, 32, 32),
    (6, 2, 64, 20, 17), (6, 2, 128, 64, 33), (4, 1, 64, 64, 64), (16, 2, 64, 64, 40)])
def test_launch_forms_match_oracle(hq, hkv, dh, max_tree, nodes):
    import paper_2502_11018_amd as P
    m = _model(hq, hkv, dh)
    mw = gen.make_weights(m, 5)
    ow = oracle.OracleWeights(mw)
    kvs = [H.prefix_kv_synthetic(m, b, p, 5) if p else None for b, p in enumerate(PREFIXES)]
    widths = [(nodes - 1 + k) // 4 for k in range(4)] if nodes > 4 else [1] * (nodes - 1)
    trees = [gen.random_tree([w for w in widths if w], m.vocab, 9 + b)[0] for b in range(len(PREFIXES))]
    mw_gpu = mw.to("cuda")
    ref = []
    for p, kv, t in zip(PREFIXES, kvs, trees):
        empty = np.zeros((m.n_kv_heads, 0, m.head_dim))
        fn = kv.fn() if kv is not None else (lambda l: (empty, empty))
        ref.append(oracle.verify_tree(ow, fn, t, p).logits)
    # all sequences at once (ragged splits), then each alone (uniform splits)
    for seqs in (tuple(range(len(PREFIXES))), (0,), (4,), (7,)):
        print(f"[gpu-case] attention heads {hq}/{hkv} dh {dh} max_tree {max_tree} nodes {nodes} seqs {seqs}", flush=True)
        with P.TreeVerifier(m, mw_gpu, max_batch=len(seqs), max_tree=max_tree, max_depth=max_tree - 1,
                            kv_capacity=512) as v:
            for row, b in enumerate(seqs):
                if kvs[b] is not None:
                    v.write_prefix(0, row, torch.from_numpy(kvs[b].K[0]).to(torch.bfloat16).cuda(),
                                   torch.from_numpy(kvs[b].V[0]).to(torch.bfloat16).cuda())
            out = torch.full((len(seqs) * max_tree, m.vocab), float("nan"), device="cuda")
            v.step([PREFIXES[b] for b in seqs], [trees[b] for b in seqs], out)
            v.accept()
            lg = out.view(len(seqs), max_tree, -1).cpu().numpy()
        for row, b in enumerate(seqs):
            n = trees[b].n
            rel = np.abs(lg[row, :n] - ref[b]).max(axis=1) / np.ptp(ref[b], axis=1)
            assert rel.max() <= H.REGRESS_REL_TOL, (seqs, b, rel.max())
