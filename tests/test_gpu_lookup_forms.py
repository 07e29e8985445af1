"""Bit parity of the lookup's scan and finish forms at their edges: queries held in registers
(two or four blocks a wave, the last one partly filled, one pass and several, tiles over all
workgroups; the launch trace says which form ran), one or two queries converted by the scan, two
query blocks per f32 pass, ragged rows and widths, rows and queries that are not finite, and the
fused finish on both sides of its tile limits."""
import numpy as np
import pytest
import torch

from oracle import lookup as O

pytestmark = pytest.mark.gpu
THR, KV = [0.9, 0.6, 0.3], [20, 10, 5]


def _case(n, d, m, seed):
    rng = np.random.default_rng(seed)
    c = rng.standard_normal((n, d)).astype(np.float32)
    c /= np.linalg.norm(c, axis=1, keepdims=True)
    q = rng.standard_normal((m, d)).astype(np.float32)
    near = rng.integers(0, n, m)
    q = np.where((np.arange(m) % 2 == 0)[:, None], c[near] + 0.3 * q / np.sqrt(d), q)
    return c, np.ascontiguousarray(q / np.linalg.norm(q, axis=1, keepdims=True), dtype=np.float32)


@pytest.mark.parametrize("n,d,m,dtype", [
    (5000, 64, 65, "bf16"), (129, 96, 100, "bf16"), (40_001, 768, 129, "bf16"), (15, 768, 128, "bf16"),
    (1500, 328, 256, "bf16"), (2000, 128, 260, "bf16"), (2000, 136, 129, "bf16"),
    (2000, 384, 128, "bf16"), (2000, 392, 65, "bf16"), (777, 512, 300, "bf16"), (3000, 640, 1, "bf16"), (3001, 768, 2, "bf16"),
    (3001, 768, 3, "bf16"), (5000, 1000, 33, "f32"), (257, 40, 17, "f32"), (1023, 768, 16, "f32"),
    (600, 2048, 40, "f32"), (3000, 768, 300, "f32")])
def test_lookup_forms(n, d, m, dtype):
    import paper_2312_04429_amd as P
    print(f"lookup n={n} d={d} m={m} {dtype}", flush=True)
    c, q = _case(n, d, m, n + d + m)
    t = torch.from_numpy(c)
    if dtype == "bf16":
        t = t.bfloat16()
        c = t.view(torch.int16).numpy().view(np.uint16)
    got = [a.cpu().numpy() for a in P.nv_cache_lookup(torch.from_numpy(q).cuda(), t.cuda(), THR, KV)]
    ref = O.lookup(q, c, THR, KV)
    for g, r in zip(got, ref):
        assert np.array_equal(g, np.asarray(r, dtype=g.dtype))


@pytest.mark.parametrize("n,d,m,blocks", [
    (15, 768, 128, 2), (777, 512, 300, 2), (1500, 328, 256, 2), (2000, 392, 65, 2),
    (5000, 256, 1000, 4),
    (66003, 744, 120, 2), (66003, 768, 190, 4), (100003, 768, 500, 4), (66003, 640, 120, 2),
    (66003, 616, 240, 4), (100003, 512, 100, 2), (66003, 504, 500, 4), (140007, 384, 250, 4),
    (140007, 248, 500, 4), (40001, 768, 129, 0), (66003, 128, 300, 0)])
def test_scan_forms(n, d, m, blocks):
    """The form that ran is the one named; every query's row has the canonical score returned, and
    no row's float64 score in another order passes it by more than its rounding (d 2^-52 for unit
    rows)."""
    import paper_2312_04429_amd as P
    print(f"scan n={n} d={d} m={m} blocks={blocks}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + d + m)
    c = torch.randn(n, d, generator=g, device="cuda")
    c = (c / c.norm(dim=1, keepdim=True)).bfloat16()
    rows = torch.randint(0, n, (m,), generator=g, device="cuda")
    rows[0], rows[1], rows[-1] = n - 1, 0, (n - 1) // 128 * 128
    q = c[rows].float() + 0.3 * torch.randn(m, d, generator=g, device="cuda") / d ** 0.5
    q = (q / q.norm(dim=1, keepdim=True)).contiguous()
    P.nv_trace_enable(8, 4)
    try:
        idx, sim, _ = P.nv_cache_lookup(q, c, THR, KV)
        torch.cuda.synchronize()
    finally:
        P.nv_trace_disable()
    assert [r[1] for r in P.nv_trace_records()] == [(m, n, d, blocks)]
    qn, cn = q.double().cpu().numpy(), c[idx].double().cpu().numpy()
    canon = np.zeros(m)
    for k in range(d):
        canon = canon + qn[:, k] * cn[:, k]
    assert np.array_equal(sim.cpu().numpy(), canon.astype(np.float32))
    best = torch.stack([(q.double() @ c[a:a + 32768].double().T).max(1).values
                        for a in range(0, n, 32768)]).max(0).values
    assert float((best - torch.from_numpy(canon).cuda()).max()) <= d * 2.0 ** -52


@pytest.mark.parametrize("tiles,m", [(16384, 3), (16385, 3), (4096, 257), (4097, 257)])
def test_finish_limits(tiles, m):
    """The same rows looked up whole and with one row more or less around the tile limit of the
    fused finish: the planted best rows come out either way, with their canonical scores."""
    import paper_2312_04429_amd as P
    d, n = 64, tiles * 128 - 5
    print(f"finish tiles={tiles} m={m}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(tiles)
    c = torch.randn(n, d, generator=g, device="cuda")
    c = (c / c.norm(dim=1, keepdim=True)).bfloat16()
    rows = torch.randint(0, n, (m,), generator=g, device="cuda")
    rows[0], rows[1] = n - 1, 0
    q = c[rows].float().contiguous()
    idx, sim, kk = P.nv_cache_lookup(q, c, THR, KV)
    qn, cn = q.double().cpu().numpy(), c[idx].double().cpu().numpy()
    canon = np.zeros(m)
    for k in range(d):
        canon = canon + qn[:, k] * cn[:, k]
    assert np.array_equal(sim.cpu().numpy(), canon.astype(np.float32))
    full = torch.cat([(q.double() @ c[a:a + 262144].double().T).max(1).values[:, None]
                      for a in range(0, n, 262144)], 1).max(1).values
    assert float((full - torch.from_numpy(canon).cuda()).max()) <= 1e-12
    assert np.array_equal(kk.cpu().numpy(), np.where(canon.astype(np.float32) > np.float32(0.9), 20, 10))


@pytest.mark.parametrize("n,d,m,dtype", [
    (3000, 768, 1, "bf16"), (3000, 384, 5, "bf16"), (3000, 768, 130, "bf16"),
    (900, 1000, 20, "bf16"), (2000, 72, 20, "f32"), (16384 * 128 + 300, 64, 3, "bf16")])
def test_rows_that_are_not_finite(n, d, m, dtype):
    """Rows with NaN, infinities and values whose squares overflow float32, in the scan that holds
    rows, the one that holds queries, the wide one and the float32 one, with the fused finish and
    past its tile limit: a score that is not a number never wins, an infinite one does, the other
    rows keep their canonical order, and a query with NaN, or with an infinity over a bf16 cache
    (whose rounding error is then not a number), has no match."""
    import paper_2312_04429_amd as P
    print(f"lookup not finite n={n} d={d} m={m} {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + d)
    c = torch.randn(n, d, generator=g, device="cuda")
    c = c / c.norm(dim=1, keepdim=True)
    q = c[torch.randint(0, n, (m,), generator=g, device="cuda")]
    q = q + 0.3 * torch.randn(m, d, generator=g, device="cuda") / d ** 0.5
    q = (q / q.norm(dim=1, keepdim=True)).contiguous()
    rng = np.random.default_rng(n)
    for k, v in enumerate((np.nan, np.nan, np.inf, -np.inf, 3e38)):
        c[torch.from_numpy(rng.choice(n, 12, replace=False)).cuda(), 3 * k] = float(v)
    if dtype == "bf16":
        c = c.bfloat16()
    if m > 2:
        q[1, 7], q[2, 9] = np.nan, np.inf
    idx, sim, kk = [a.cpu().numpy() for a in P.nv_cache_lookup(q, c, THR, KV)]
    c64, q64 = c.double().cpu().numpy(), q.double().cpu().numpy()
    with np.errstate(invalid="ignore", over="ignore"):
        for j in sorted({0, 1, 2, 3, m // 2, m - 1} & set(range(m))):
            s = np.zeros(n)
            for k in range(d):
                s = s + q64[j, k] * c64[:, k]
            if np.isnan(q64[j]).any() or (dtype == "bf16" and np.isinf(q64[j]).any()):
                want = -1, -np.inf
            else:
                s[np.isnan(s)] = -np.inf
                want = int(s.argmax()), s.max()
            assert idx[j] == want[0] and sim[j] == np.float32(want[1]), (j, idx[j], sim[j], want)
