"""Bit parity of the lookup's scan and finish forms at their edges: queries held in registers
(more than 64; the last block partly filled, two passes past 256), one or two queries converted
by the scan, two query blocks per f32 pass, ragged rows and widths, and the fused finish on both
sides of its tile limits."""
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
