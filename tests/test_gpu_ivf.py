"""GPU parity of the IVF index (the indexed vector-DB search, Sec. 5.3 / Sec. 6)
against the oracle: centroids, lists, permutation and offsets of the build are
bit-identical (with and without Lloyd steps, bf16 and f32 rows, d up to 768),
the rows are stored in list order, and every search result (row, similarity,
K, the probed lists) equals the oracle's; probing every list gives the exact
lookup's results."""
import numpy as np
import pytest
import torch

import synth
from oracle import ivf

pytestmark = pytest.mark.gpu

T = [t for t, _ in synth.THRESHOLDS_PAPER]
K = [k for _, k in synth.THRESHOLDS_PAPER]


def _dev(X):
    return torch.from_numpy(X.view(np.int16) if X.dtype == np.uint16 else X).cuda()


def _queries(X, m, seed):
    rows = synth.from_bf16_bits(X) if X.dtype == np.uint16 else X
    rng = np.random.default_rng(seed)
    near = synth.make_queries_at_sims(rows[rng.integers(0, len(rows), m // 2)],
                                      rng.choice([0.97, 0.92, 0.87, 0.8, 0.7], m // 2), seed)
    fresh = synth.make_prompt_stream(m - m // 2, X.shape[1], seed, p_new=1.0)
    return np.concatenate([near, fresh]).astype(np.float32)


@pytest.mark.parametrize("n,d,dtype,L,iters", [(3000, 64, "bf16", 24, 0), (3000, 64, "bf16", 24, 2),
                                               (1200, 32, "f32", 8, 1), (2500, 768, "bf16", 32, 1),
                                               (700, 64, "bf16", 1, 1)])
def test_build_and_search_match_oracle(n, d, dtype, L, iters):
    import paper_2312_04429_amd as P
    print(f"ivf n={n} d={d} {dtype} L={L} iters={iters}", flush=True)
    X = synth.make_cache(n, d, 12, 0.15, n + d, dtype, dup_pairs=((3, 9),))
    init = np.random.default_rng(L).choice(n, L, replace=False)
    cache = _dev(X)
    index = P.NvIVF(cache, init, iters)
    c, lists, perm, off = ivf.build(X, init, iters)
    got_c = index.cents.cpu().numpy()
    if dtype == "bf16":
        got_c = got_c.view(np.uint16)
    assert np.array_equal(got_c, c)
    assert index.lists.cpu().numpy().tolist() == lists.tolist()
    assert index.perm.cpu().numpy().tolist() == perm.tolist()
    assert index.offsets.cpu().numpy().tolist() == off.tolist()
    assert index.max_list == int(np.diff(off).max())
    rows = index.rows.cpu().numpy()
    assert np.array_equal(rows.view(X.dtype) if dtype == "bf16" else rows, X[perm])
    q = torch.from_numpy(_queries(X, 24, 7)).cuda()
    qn = q.cpu().numpy()
    for nprobe in sorted({1, min(3, L), L}):
        print(f"  search nprobe={nprobe}", flush=True)
        gi, gs, gk, gp = index.search(q, nprobe, T, K, probed=True)
        oi, os_, ok, op = ivf.search(qn, X, c, perm, off, nprobe, T, K)
        assert gi.cpu().numpy().tolist() == oi.tolist()
        assert np.array_equal(gs.cpu().numpy(), os_)
        assert gk.cpu().numpy().tolist() == ok.tolist()
        assert gp.cpu().numpy().tolist() == op.tolist()
    ei, es, ek = P.nv_cache_lookup(q, cache, T, K)
    gi, gs, gk = index.search(q, L, T, K)
    assert torch.equal(gi, ei) and torch.equal(gs, es) and torch.equal(gk, ek)


# widths around the 64-value slices and the 48-chunk loads, list counts around the 64-centroid
# blocks, lists of several 256-row chunks, and equal rows (every one of them is summed canonically)
@pytest.mark.parametrize("n,d,dtype,L,same", [(600, 2048, "bf16", 65, 5), (900, 72, "f32", 300, 3),
                                              (1100, 520, "bf16", 2, 40), (513, 392, "f32", 1, 300)])
def test_search_forms(n, d, dtype, L, same):
    import paper_2312_04429_amd as P
    print(f"ivf forms n={n} d={d} {dtype} L={L} same={same}", flush=True)
    rng = np.random.default_rng(n + d)
    X = synth.make_cache(n, d, 12, 0.15, n + d, dtype)
    X[rng.choice(n, same, replace=False)] = X[n // 2]
    init = rng.choice(n, L, replace=False)
    index = P.NvIVF(_dev(X), init, 0)
    c, _, perm, off = ivf.build(X, init, 0)
    qn = _queries(X, 6, 7)
    qn[0] = (synth.from_bf16_bits(X) if dtype == "bf16" else X)[n // 2]
    for nprobe in sorted({1, min(17, L), min(256, L)}):
        print(f"  search nprobe={nprobe}", flush=True)
        got = index.search(torch.from_numpy(qn).cuda(), nprobe, T, K, probed=True)
        for g, r in zip(got, ivf.search(qn, X, c, perm, off, nprobe, T, K)):
            assert np.array_equal(g.cpu().numpy(), r)


def _tree(scores, ids):
    """(score, id) that the fixed comparison tree over 256 slots leaves in slot 0."""
    s, i = list(scores) + [-np.inf] * (256 - len(scores)), list(ids) + [-1] * (256 - len(ids))
    w = 128
    while w:
        for t in range(w):
            a, b = t + w, t
            if i[a] >= 0 and (i[b] < 0 or s[a] > s[b] or (s[a] == s[b] and i[a] < i[b])):
                s[b], i[b] = s[a], i[a]
        w //= 2
    return s[0], i[0]


# one list of one block: rows to sum on both sides of the line between a wave and a thread a row
@pytest.mark.parametrize("dtype,d", [("bf16", 136), ("f32", 72), ("bf16", 2048)])
@pytest.mark.parametrize("same", [8, 9, 64, 65, 256])
def test_equal_rows_of_one_block(dtype, d, same):
    import paper_2312_04429_amd as P
    n = 256
    print(f"ivf equal rows d={d} {dtype} same={same}", flush=True)
    X = synth.make_cache(n, d, 12, 0.15, d, dtype)
    at = np.sort(np.random.default_rng(same).choice(n, same, replace=False))
    X[at] = X[at[0]]
    init = np.array([0])
    index = P.NvIVF(_dev(X), init, 0)
    rows = synth.from_bf16_bits(X) if dtype == "bf16" else X
    q = np.stack([rows[at[0]] / np.linalg.norm(rows[at[0]]), -rows[at[0]]]).astype(np.float32)
    c, lists, perm, off = ivf.build(X, init, 0)
    gi, gs, gk = index.search(torch.from_numpy(q).cuda(), 1, T, K)
    oi, os_, ok, _ = ivf.search(q, X, c, perm, off, 1, T, K)
    assert gi.cpu().numpy().tolist() == oi.tolist() and gi[0].item() == at[0]
    assert np.array_equal(gs.cpu().numpy(), os_)
    assert gk.cpu().numpy().tolist() == ok.tolist()


@pytest.mark.parametrize("n,d,dtype,L", [(900, 64, "f32", 2), (700, 72, "bf16", 3)])
def test_rows_that_are_not_finite(n, d, dtype, L):
    """Scores that are not numbers are ordered by the comparison tree alone: with NaN and infinite
    rows in the lists every call gives the answer of the tree over list positions, then over the
    probes' chunks."""
    import paper_2312_04429_amd as P
    print(f"ivf not finite n={n} d={d} {dtype} L={L}", flush=True)
    X = synth.make_cache(n, d, 12, 0.15, n + d, dtype)
    index = P.NvIVF(_dev(X), np.arange(L) * (n // L), 0)
    rng = np.random.default_rng(d)
    at = torch.from_numpy(rng.choice(n, 60, replace=False)).cuda()
    flat = index.rows.view(torch.bfloat16) if dtype == "bf16" else index.rows
    for part, v in zip(at.chunk(4), (np.nan, np.inf, -np.inf, 3e38)):
        flat[part, int(rng.integers(d))] = float(v)
    rows = flat.double().cpu().numpy()
    perm, off = index.perm.cpu().numpy(), index.offsets.cpu().numpy()
    q = _queries(X, 8, 3)
    q[5] = np.nan
    got = [[a.cpu().numpy() for a in index.search(torch.from_numpy(q).cuda(), L, T, K, probed=True)]
           for _ in range(12)]
    with np.errstate(invalid="ignore", over="ignore"):
        for j in range(len(q)):
            s = np.zeros(n)
            for k in range(d):
                s = s + float(q[j, k]) * rows[:, k]
            parts = []
            for l in got[0][3][j]:
                for c in range(off[l], off[l] + 256 * max(1, -(-index.max_list // 256)), 256):
                    e = min(c + 256, off[l + 1])
                    parts.append(_tree(s[c:e], perm[c:e]) if c < e else (-np.inf, -1))
            assert len(parts) <= 256
            best, row = _tree(*zip(*parts))
            for r in got:
                assert r[0][j] == row
                assert np.array_equal(r[1][j], np.float32(best), equal_nan=True)
