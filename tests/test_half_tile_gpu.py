"""Half row tiles (csrc/gemm.hip): a step with at most 32 live rows, and an expert
routed at most 32, run the GEMMs over one 32-row half.  Each row sums the same
products in the same order either way, so the first nodes of a tree have the
same bits whichever of its later nodes come along."""

from dataclasses import replace
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from workloads import gen
from workloads.configs import SMALL_GQA
from tests import harness as H

pytestmark = pytest.mark.gpu

PREFIX = 45
DENSE = replace(SMALL_GQA, name="half-dense", n_layers=2, vocab=1100)
# both experts kept by every node: an expert's rows are the tree's nodes
MOE = replace(DENSE, name="half-moe", n_experts=2, top_k=2)
# one of four kept: counts on either side of the edge in one launch
MOE_MIXED = replace(DENSE, name="half-moe-mixed", n_experts=4, top_k=1)
# widths of the models in use: the deeper pipelines, and two K slices a workgroup in
# the down projection, that short K ranges do not take
WIDE = replace(DENSE, name="half-wide", n_layers=1, d_model=4096, n_q_heads=32, n_kv_heads=8, d_ff=14336)
WIDE_MOE = replace(WIDE, name="half-wide-moe", n_experts=2, top_k=2)
WIDE_MIXED = replace(WIDE, name="half-wide-moe-mixed", n_experts=4, top_k=1)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("m", [DENSE, MOE, MOE_MIXED, WIDE, WIDE_MOE, WIDE_MIXED], ids=lambda m: m.name)
def test_first_nodes_keep_their_bits(m, bf16):
    import paper_2502_11018_amd as P
    mw = gen.make_weights(m, 7, device="cuda")
    kv = H.prefix_kv_synthetic(m, 0, PREFIX, 7)
    full = gen.random_tree((7, 14, 21, 21), m.vocab, 4)[0]
    assert full.n == 64
    with P.TreeVerifier(m, mw.to("cuda"), max_batch=1, max_tree=64, max_depth=8, kv_capacity=128) as v:
        for l in range(m.n_layers):
            v.write_prefix(l, 0, torch.from_numpy(kv.K[l]).to(torch.bfloat16).cuda(),
                           torch.from_numpy(kv.V[l]).to(torch.bfloat16).cuda())
        v.set_bf16_activations(bf16)

        def step(n):
            print(f"[gpu-case] half tile {m.name} bf16 {bf16} nodes {n}", flush=True)
            t = SimpleNamespace(n=n, tokens=np.asarray(full.tokens[:n]), parents=np.asarray(full.parents[:n]))
            out = torch.full((64, m.vocab), float("nan"), device="cuda")
            v.step([PREFIX], [t], out)
            feat = v.features([list(range(n))]).cpu().numpy()[0]
            return out[:n].cpu().numpy(), feat, v.predictions()[0, :n], v.margins()[0, :n]

        ref = step(64)
        assert np.isfinite(ref[0]).all()
        for n in (1, 31, 32, 33, 63):
            for got, want in zip(step(n), ref):
                assert np.array_equal(got, want[:n]), n
