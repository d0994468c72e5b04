"""The GEMMs over several 64-row tiles (csrc/gemm_rows.hip) against the fp64
oracle.  The tile shape, the K splits and the last tile's padding depend on
the matrix and on the step's number of row tiles: a narrow model with a wide
head over every tile count of a context (its other matrices keep one shape), and
the widths of the models in use over the counts that give every shape to the
projections and to gate/up."""

from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from workloads import gen
from workloads.configs import SMALL_GQA
from tests import harness as H

pytestmark = pytest.mark.gpu

# vocab 100004: enough column tiles (782 groups, the last two past the vocabulary
# in part) that the LM head takes the widest tile shape; d_ff 1376 and K 1376
# end inside a column tile and a K step
MODEL = replace(SMALL_GQA, name="rows", n_layers=1, vocab=100004)
PREFIX = 37

# tests/test_host_sanitized.py checks that these batches take all four tile shapes
WIDE = replace(MODEL, name="rows-wide", d_model=4096, n_q_heads=32, n_kv_heads=8, d_ff=14336, vocab=1100)
WIDE_BATCHES = (1, 2, 3, 4, 5, 8, 9, 12)


@pytest.fixture(scope="module")
def model():
    mw = gen.make_weights(MODEL, 3)
    return mw, oracle.OracleWeights(mw), H.prefix_kv_synthetic(MODEL, 0, PREFIX, 3), mw.to("cuda")


# max_tree 64: whole tiles; 40: sequences straddle tiles and the last one is partial
@pytest.mark.parametrize("max_tree,batches", [(64, (1, 2, 3, 4, 5, 8)), (40, (1, 2, 5, 8))])
def test_every_tile_count_matches_oracle(model, max_tree, batches):
    import paper_2502_11018_amd as P
    mw, ow, kv, mw_gpu = model
    trees = [gen.random_tree((4, 8, 8, 8), MODEL.vocab, 50 + b)[0] for b in range(8)]
    refs = {b: oracle.verify_tree(ow, kv.fn(), trees[b], PREFIX).logits for b in (0, 1, 4, 7)}
    with P.TreeVerifier(MODEL, mw_gpu, max_batch=8, max_tree=max_tree, max_depth=8, kv_capacity=128) as v:
        for b in range(8):
            v.write_prefix(0, b, torch.from_numpy(kv.K[0]).to(torch.bfloat16).cuda(),
                           torch.from_numpy(kv.V[0]).to(torch.bfloat16).cuda())
        for B in batches:
            print(f"[gpu-case] rows max_tree {max_tree} batch {B}", flush=True)
            out = torch.full((B * max_tree, MODEL.vocab), float("nan"), device="cuda")
            v.step([PREFIX] * B, trees[:B], out)
            pred = v.predictions()
            lg = out.view(B, max_tree, -1).cpu().numpy()
            for b, ref in refs.items():
                if b >= B:
                    continue
                n = trees[b].n
                rel = np.abs(lg[b, :n] - ref).max(axis=1) / np.ptp(ref, axis=1)
                assert rel.max() <= H.REGRESS_REL_TOL, (B, b, rel.max())
                own = lg[b, :n].argmax(axis=1)   # the partial maxima against the step's own logits
                assert np.array_equal(pred[b, :n], own), (B, b)
        # rounded activations take the kernel's single-plane form; bound as for bf16 itself
        v.set_bf16_activations(True)
        out = torch.empty((8 * max_tree, MODEL.vocab), device="cuda")
        v.step([PREFIX] * 8, trees, out)
        v.accept()
        lg = out.view(8, max_tree, -1).cpu().numpy()
        for b, ref in refs.items():
            rel = np.abs(lg[b, : trees[b].n] - ref).max(axis=1) / np.ptp(ref, axis=1)
            assert rel.max() <= H.LOGIT_REL_TOL, (b, rel.max())


def test_every_tile_shape_at_wide_matrices():
    """One context, all batches, both activation precisions.  The K splits change
    with the batch, so a sequence's bits may; its logits stay within the bound."""
    import paper_2502_11018_amd as P
    m, T, top = WIDE, 64, max(WIDE_BATCHES)
    mw = gen.make_weights(m, 3, device="cuda")
    ow, kv = oracle.OracleWeights(mw.to("cpu"), cache=True), H.prefix_kv_synthetic(m, 0, PREFIX, 3)
    trees = [gen.random_tree((4, 8, 8, 8) if b % 2 else (10, 17, 18, 18), m.vocab, 50 + b)[0] for b in range(top)]
    refs = {}
    for b in (0, 1, 4, 8, 11):
        print(f"[gpu-case] rows wide: oracle of sequence {b}", flush=True)
        refs[b] = oracle.verify_tree(ow, kv.fn(), trees[b], PREFIX).logits
    with P.TreeVerifier(m, mw, max_batch=top, max_tree=T, max_depth=8, kv_capacity=128) as v:
        for b in range(top):
            v.write_prefix(0, b, torch.from_numpy(kv.K[0]).to(torch.bfloat16).cuda(),
                           torch.from_numpy(kv.V[0]).to(torch.bfloat16).cuda())
        for bf16, tol in ((False, H.REGRESS_REL_TOL), (True, H.LOGIT_REL_TOL)):
            v.set_bf16_activations(bf16)
            for B in WIDE_BATCHES:
                print(f"[gpu-case] rows wide batch {B} bf16 {bf16}", flush=True)
                out = torch.full((B * T, m.vocab), float("nan"), device="cuda")
                v.step([PREFIX] * B, trees[:B], out)
                pred = v.predictions()
                lg = out.view(B, T, -1).cpu().numpy()
                for b, ref in refs.items():
                    if b >= B:
                        continue
                    n = trees[b].n
                    rel = np.abs(lg[b, :n] - ref).max(axis=1) / np.ptp(ref, axis=1)
                    assert rel.max() <= tol, (B, b, bf16, rel.max())
                    assert np.array_equal(pred[b, :n], lg[b, :n].argmax(axis=1)), (B, b)
