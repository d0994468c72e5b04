"""Output rows that are no whole number of 16-byte groups: vocabularies and
fusion widths that are no multiple of 4 (or of 8, for a width that is also a K
extent).  A row's last group must not reach into the next row, nor past the
caller's buffer."""

from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from oracle import draft as od
from workloads import gen
from workloads.configs import DRAFTS, SMALL_GQA
from tests import harness as H

pytestmark = pytest.mark.gpu

PREFIX = 33


# one row tile, and three (gemm_rows.hip); node counts of a half tile and of a whole one
@pytest.mark.parametrize("batch", [1, 3])
@pytest.mark.parametrize("vocab", [1001, 1002, 1003, 1004])
def test_every_logit_of_odd_vocabularies(vocab, batch):
    import paper_2502_11018_amd as P
    m = replace(SMALL_GQA, name=f"v{vocab}", n_layers=1, vocab=vocab)
    mw = gen.make_weights(m, 5)
    ow, kv = oracle.OracleWeights(mw), H.prefix_kv_synthetic(m, 0, PREFIX, 5)
    with P.TreeVerifier(m, mw.to("cuda"), max_batch=batch, max_tree=64, max_depth=8, kv_capacity=128) as v:
        for b in range(batch):
            v.write_prefix(0, b, torch.from_numpy(kv.K[0]).to(torch.bfloat16).cuda(),
                           torch.from_numpy(kv.V[0]).to(torch.bfloat16).cuda())
        for widths in ((7, 14, 21, 21), (5, 6, 7)):
            print(f"[gpu-case] odd vocabulary {vocab} batch {batch} nodes {1 + sum(widths)}", flush=True)
            trees = [gen.random_tree(widths, vocab, 30 + b)[0] for b in range(batch)]
            buf = torch.full((batch * 64 * vocab + 64,), 7.0, device="cuda")
            v.step([PREFIX] * batch, trees, buf[: batch * 64 * vocab])
            v.accept()
            assert (buf[batch * 64 * vocab:] == 7.0).all()
            lg = buf[: batch * 64 * vocab].view(batch, 64, vocab).cpu().numpy()
            for b, t in enumerate(trees):
                ref = oracle.verify_tree(ow, kv.fn(), t, PREFIX).logits
                rel = np.abs(lg[b, : t.n] - ref) / np.ptp(ref, axis=1, keepdims=True)
                assert rel.max() <= H.REGRESS_REL_TOL, (b, np.unravel_index(rel.argmax(), rel.shape), rel.max())


@pytest.mark.parametrize("batch", [1, 2])
@pytest.mark.parametrize("width", [33, 62, 99, 100])
def test_draft_pass_of_odd_fusion_widths(width, batch):
    """The log-probabilities of every node's top-k under a fusion of `width`."""
    import paper_2502_11018_amd as P
    ds = replace(DRAFTS["tiny"], tgf_dim=width)
    m, k = ds.target, 16
    mw, dw = gen.make_weights(m, 0), gen.make_draft_weights(ds, 3)
    dow = od.DraftOracleWeights(dw, oracle.OracleWeights(mw))
    feat = gen.draft_root_features(m.d_model, batch, 11)
    with P.DraftModel(ds, dw.to("cuda"), mw.to("cuda"), max_batch=batch, max_tree=64, max_depth=8,
                      kv_capacity=128) as dm:
        kv = [gen.synthetic_kv(ds.layer, 0, b, PREFIX, 5) for b in range(batch)]
        for b in range(batch):
            dm.write_prefix(b, kv[b][0].cuda(), kv[b][1].cuda())
        prev = [None] * batch
        for widths in ((), (9,), (9, 20), (9, 20, 30)):  # a node's parent ran in the pass before
            print(f"[gpu-case] fusion width {width} batch {batch} nodes {1 + sum(widths)}", flush=True)
            trees = [gen.random_tree(widths, m.vocab, 50 + 7 * b)[0] for b in range(batch)]
            tok, lp = dm.step([PREFIX] * batch, trees, feat.cuda(), k)
            for b, t in enumerate(trees):
                feats = np.zeros((t.n, m.d_model))
                feats[0] = feat[b].double().numpy()
                for i in range(1, t.n):
                    feats[i] = prev[b][t.parents[i]]
                r = od.draft_forward(dow, t, feats, (kv[b][0].double().numpy(), kv[b][1].double().numpy()), PREFIX)
                prev[b] = r.regress
                for i in range(t.n):
                    x = r.logits[i]
                    full = x - (x.max() + np.log(np.exp(x - x.max()).sum()))
                    assert np.abs(lp[b, i] - full[tok[b, i]]).max() < 2e-3, (b, i)
