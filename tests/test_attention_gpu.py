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


def test_softmax_denominator_keeps_small_probabilities():
    """One node and one head over 65536 keys in 16 splits.  The first key of each
    split dominates (its value is 1, all others 0), every other key has a
    probability of just under half a unit of rounding beside it.  The output is 1 /
    denominator.  Added to the running sum key by key, the small ones of the
    dominant key's lane would all be lost (1.1e-4); a block's 16 as a tree, then the
    block, is off by at most 128 blocks x 2^-24, and the output's split into
    two bf16 parts by 2^-17: 1.6e-5 in all."""
    import paper_2502_11018_amd as P
    m = replace(SMALL_GQA, name="denominator", n_layers=1, d_model=64, n_q_heads=1, n_kv_heads=1, head_dim=64,
                d_ff=64, vocab=64, weight_std=0.2)
    keys, splits = 65536, 16
    mw = gen.make_weights(m, 5)
    lay = mw.layers[0]
    lay["w_qkv"][64:] = 0                       # the node's own key scores 0, its value is 0
    lay["w_o"].copy_(torch.eye(64))
    lay["w_down"].zero_()                       # feature = embedding + attention output
    ow = oracle.OracleWeights(mw)
    tree = gen.Tree(np.asarray([3], np.int32), np.asarray([-1], np.int32))
    x = ow.embed(tree.tokens)
    q = oracle.model.rmsnorm(x, ow.layer(0)["attn_norm"], m.rms_eps) @ ow.layer(0)["w_qkv"][:64].T
    q = oracle.model.rope(q[:, None, :], np.asarray([[keys]]), m.rope_base)[0, 0]
    scale = np.log2(np.e) / 8

    def key(score):                             # a bf16 key of about this score (log2 domain), and its exact one
        k = H.bf16_round(score / scale * q / (q @ q))
        return k, (q @ k) * scale

    top, s_top = key(60.0)
    low, s_low = next(kl for kl in (key(s_top - 24.15 + e) for e in np.linspace(-0.4, 0.4, 161))
                      if 0.85 < 2.0 ** (kl[1] - s_top + 24) < 0.95)
    K = np.broadcast_to(low, (1, keys, 64)).copy()
    V = np.zeros((1, keys, 64))
    K[0, :: keys // splits] = top
    V[0, :: keys // splits] = 1.0
    den = 1 + (keys // splits - 1) * 2.0 ** (s_low - s_top)
    ref = oracle.verify_tree(ow, lambda l: (K, V), tree, keys).hidden[0] - x[0]
    assert np.abs(ref * den - 1).max() < 1e-9
    print("[gpu-case] softmax denominator over 65536 keys", flush=True)
    with P.TreeVerifier(m, mw.to("cuda"), max_batch=1, max_tree=1, max_depth=0, kv_capacity=keys + 64) as v:
        v.write_prefix(0, 0, torch.from_numpy(K).to(torch.bfloat16).cuda(),
                       torch.from_numpy(V).to(torch.bfloat16).cuda())
        v.step([keys], [tree])
        out = v.features([[0]]).cpu().numpy()[0, 0].astype(np.float64) - x[0]
    rel = np.abs(out / ref - 1).max()
    print(f"[gpu-case] softmax denominator off by {rel:.2e}", flush=True)
    assert rel < 1.6e-5, rel
