"""The token a stochastic acceptance emits, pinned where rounding decides it.

At 128256 tokens a token of the tail holds about 1e-7 of the mass, which is the
rounding of the fp32 sums a draw is compared with: another grouping of those
sums is as near to the exact distribution and still emits another token once
in some hundred draws.  So what is pinned here is not the exact
distribution (tests/test_sampling_gpu.py compares with the oracle) but that the
emitted tokens stay what they were: CRC-32 of the tokens of seeded draws, as
the library gave them before its normaliser was taken for the parents alone.
"""

import zlib

import numpy as np
import pytest
import torch

from workloads import gen

pytestmark = pytest.mark.gpu

LEAF_CALLS, LEAF_ROWS = 16, 256


def leaf_draws(P, V, with_q):
    """CRC per call of the tokens that single-node trees emit: 256 rows of
    logits, another u per call.  with_q: through the path of sampled drafts
    (whose walk ends at a leaf), else that of deterministic ones."""
    rng = np.random.default_rng(V)
    logits = torch.from_numpy(rng.standard_normal((LEAF_ROWS, V), dtype=np.float32) * 4).cuda()
    tree = gen.Tree(np.zeros(1, np.int32), np.full(1, -1, np.int32))
    out = []
    for _ in range(LEAF_CALLS):
        u = rng.random((LEAF_ROWS, 1), dtype=np.float32)
        r = P.accept_sampled_walk([tree] * LEAF_ROWS, logits, logits if with_q else None, u, u, 1.0, 1, 0, V)
        out.append(zlib.crc32(np.ascontiguousarray(r.tokens, dtype=np.int32).tobytes()))
    return out


def tree_draws(P, V):
    """CRC per call of lengths and tokens of three 61-node trees drawn from
    their draft distributions, other uniforms per call: 48 walks that test
    children, draw residuals and end at leaves."""
    max_tree, D, B = 64, 6, 3
    cases = [gen.sampled_case((10,) * 6, V, 500 + 17 * i) for i in range(B)]
    lg = np.zeros((B * max_tree, V), np.float32)
    q = np.zeros((B * max_tree, V), np.float32)
    for b, c in enumerate(cases):
        lg[b * max_tree: b * max_tree + c.tree.n] = c.logits
        q[b * max_tree: b * max_tree + c.tree.n] = c.q
    lg, q = torch.from_numpy(lg).cuda(), torch.from_numpy(q).cuda()
    rng = np.random.default_rng(7)
    out = []
    for _ in range(16):
        ua, uf = rng.random((2, B, max_tree), dtype=np.float32)
        r = P.accept_sampled_walk([c.tree for c in cases], lg, q, ua, uf, 1.0, max_tree, D, V)
        both = np.concatenate([r.length[:, None], r.tokens], axis=1)
        out.append(zlib.crc32(np.ascontiguousarray(both, dtype=np.int32).tobytes()))
    return out


# a deterministic draft's tree without children draws from the same distribution
LEAF = {
    128256: [
    0xae861a81, 0x25ee6899, 0xe3bdd39f, 0x8f75f42d, 0x27477861, 0xdf6d3abf, 0x966f09ca, 0x9f91389b,
    0x24df7cf2, 0x308cade9, 0x1ddb1d68, 0xc3e79b0e, 0xd1abe65d, 0x2a5a4975, 0x05c516ea, 0xb65727d5,
],
    20001: [
    0xa55c6940, 0x38bdff43, 0x5744819b, 0x9c1ccafb, 0x111ea103, 0xba85ea0f, 0x1c0978cb, 0x743da9f9,
    0x8b216e4b, 0xbfd56fef, 0x45dd759f, 0xe2b2acd6, 0xf18de62c, 0x3b9027aa, 0xed02ffd8, 0x7bee6ada,
],  # rows of this length are not 16-byte aligned
}
TREE = [
    0xd4b90eb4, 0x5a7e09f7, 0xc4e71f94, 0xc7edb70f, 0xd5c9c64d, 0x40fcbd62, 0x59388594, 0xa4c8d4e2,
    0x7e8fd834, 0x6deb5294, 0xda1a8343, 0x737ee053, 0xf4909e0a, 0x3afa6bd0, 0x9531958c, 0xa20e0e7a,
]


@pytest.mark.parametrize("with_q", [True, False])
@pytest.mark.parametrize("V", sorted(LEAF))
def test_leaf_draws_keep_their_tokens(V, with_q):
    import paper_2502_11018_amd as P
    print(f"[gpu-case] leaf draws V={V} q={with_q}", flush=True)
    assert leaf_draws(P, V, with_q) == LEAF[V]


def test_tree_draws_keep_their_tokens():
    import paper_2502_11018_amd as P
    print("[gpu-case] tree draws", flush=True)
    assert tree_draws(P, 128256) == TREE


# ---- thresholds on slice boundaries ------------------------------------------------

F = np.float32


def _slices(V):
    n = min(64, max(1, (V + 2047) // 2048))
    chunk = (-(-V // n) + 3) & ~3
    return [(min(V, s * chunk), min(V, s * chunk + chunk)) for s in range(n)]


def _block_sum(x):
    """A workgroup's sum of its 256 threads' values: butterflies over each wave, then the waves in order."""
    t = F(0)
    for w in x.reshape(4, 64):
        for o in (32, 16, 8, 4, 2, 1):
            w = w + w[np.arange(64) ^ o]
        t = F(t + w[0])
    return t


def _scan(x):
    """Inclusive doubling scan, as a wave and a workgroup do it."""
    x, o = x.copy(), 1
    while o < len(x):
        x[o:] = x[o:] + x[:-o]
        o *= 2
    return x


def _level_sums(live):
    """fp32 sums of a row whose live tokens all have p = 1 / n: per slice as the
    draw's first level adds them (a thread's groups of four), and per slice the
    scan of its second (a thread's contiguous range)."""
    p, top, inner = F(1) / F(live.sum()), [], []
    for lo, hi in _slices(len(live)):
        x = np.zeros((hi - lo + 1023) // 1024 * 1024, F)
        x[: hi - lo] = live[lo:hi] * p
        t = np.zeros(256, F)
        for grp in x.reshape(-1, 256, 4):
            for j in range(4):
                t = t + grp[:, j]
        top.append(_block_sum(t))
        per = -(-(hi - lo) // 256)
        y = np.zeros(256 * per, F)
        y[: hi - lo] = live[lo:hi] * p
        c = np.zeros(256, F)
        for col in y.reshape(256, per).T:
            c = c + col
        inner.append(_scan(c))
    return np.array(top, F), inner


@pytest.mark.parametrize("with_q", [True, False])
def test_a_draw_on_a_slice_boundary_has_mass(with_q):
    """Rows of equal live tokens, dead (-inf) at both ends of every slice, drawn
    at u within a few units of rounding of every slice boundary.  Their sums are
    known to the bit, and for some of these u the threshold lies outside the
    slice's own scan.  Every emitted token must be live, and the one that u asks
    for or its neighbour (fp32 sums over n tokens are off by far less than 1 / n)."""
    import paper_2502_11018_amd as P
    V = 128256
    rng = np.random.default_rng(5)
    live = rng.random(V) < 0.4
    for lo, hi in _slices(V):
        live[lo: lo + 5] = False
        live[hi - 9: hi] = False
    n = int(live.sum())
    top, inner = _level_sums(live)
    inc = np.zeros(64, F)
    inc[: len(top)] = top
    inc = _scan(inc)
    us, outside = [], 0
    for i in range(len(top) - 1):
        u = F(inc[i] / inc[63])
        for _ in range(4):
            u = np.nextafter(u, F(0), dtype=F)
        for _ in range(9):
            us.append(u)
            for thr in (float(F(u * inc[63])), float(u) * float(inc[63])):  # rounded, or kept in a fused subtraction
                s = int(np.argmax(inc > F(u * inc[63])))
                at = F(thr - float(F(inc[s] - top[s])))
                outside += not 0 <= at < inner[s][-1]
            u = np.nextafter(u, F(1), dtype=F)
    assert outside > 20, outside
    us = np.array(us, F)[:, None]
    row = torch.from_numpy(np.where(live, F(0), F(-np.inf)))
    logits = row.cuda().expand(len(us), V).contiguous()
    tree = gen.Tree(np.zeros(1, np.int32), np.full(1, -1, np.int32))
    print(f"[gpu-case] draws on slice boundaries q={with_q}: {len(us)} draws, {outside} thresholds outside", flush=True)
    r = P.accept_sampled_walk([tree] * len(us), logits, logits if with_q else None, us, us, 1.0, 1, 0, V)
    tok = r.tokens[:, 0]
    assert live[tok].all(), (us[~live[tok], 0], tok[~live[tok]])
    want = np.floor(us[:, 0].astype(np.float64) * n).astype(np.int64)
    assert np.abs(np.cumsum(live)[tok] - 1 - want).max() <= 1
