"""GPU parity of the wide GEMM forms (whole-chip tiles, k halves and k teams, the row-staged
epilogue) at the edges of their tiles: ragged rows and columns, one k tile (a team without
one), odd k tile counts, two sources, strided and upsampling convolutions; and, through small
networks of ragged row counts, the epilogues that have no call of their own (folded LayerNorm,
transposed columns, GEGLU, the time embedding's row vector).  The small-tile kernel's forms follow,
unsplit for column counts that the row-staged epilogue does not take, and split.  The tests that
name a form check in the launch trace that it ran."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _check(got, ref, mag, K):
    """float16 rounding of the result plus the worst case of K float32 additions, whose terms
    sum to `mag` in magnitude (any order)."""
    bound = 2.0 ** -11 * np.abs(ref) * (1 + 2.0 ** -10) + (K + 4) * 2.0 ** -24 * mag + 2.0 ** -24
    worst = float((np.abs(got - ref) / bound).max())
    assert worst <= 1.0, worst


# one ragged shape per form and k tile count (the form follows from the cost of its tiles)
@pytest.mark.parametrize("M,N,K1,K2", [
    (8199, 1432, 64, 0), (4100, 3848, 192, 0), (8200, 920, 576, 384), (8796, 904, 64, 0),
    (8561, 392, 1280, 0), (6740, 264, 64, 0), (6740, 264, 128, 192), (2476, 2080, 64, 0),
    (8839, 200, 128, 0), (8221, 80, 64, 128), (646, 5400, 64, 0), (646, 5400, 192, 128),
    (1000, 1288, 1280, 0), (1, 280, 64, 0), (515, 1288, 320, 64), (17, 8, 192, 0)])
def test_linear_forms(M, N, K1, K2):
    import paper_2312_04429_amd as P
    print(f"wide linear M={M} N={N} K={K1}+{K2}", flush=True)
    g = torch.Generator().manual_seed(M + N)
    x = torch.randn(M, K1 + K2, generator=g).half()
    w = (0.05 * torch.randn(N, K1 + K2, generator=g)).half()
    b = torch.randn(N, generator=g)
    r = torch.randn(M, N, generator=g).half()
    x1, x2 = x[:, :K1].contiguous(), x[:, K1:].contiguous() if K2 else None
    got = P.nv_op_linear(x1.cuda(), w.cuda(), b.cuda(), r.cuda(),
                         x2=x2.cuda() if K2 else None).cpu().double().numpy()
    ref = x.double() @ w.double().T + b.double() + r.double()
    mag = x.double().abs() @ w.double().abs().T + b.double().abs() + r.double().abs()
    _check(got, ref.numpy(), mag.numpy(), K1 + K2)


@pytest.mark.parametrize("B,H,W,C1,C2,Co,stride,up", [
    (2, 61, 63, 192, 0, 320, 1, 0), (2, 32, 32, 640, 0, 640, 1, 0), (3, 31, 33, 64, 128, 328, 1, 0),
    (2, 62, 34, 64, 64, 640, 2, 0), (2, 17, 19, 128, 0, 264, 1, 1), (1, 3, 5, 64, 0, 72, 1, 0),
    (4, 64, 64, 64, 64, 328, 1, 0)])
def test_conv_forms(B, H, W, C1, C2, Co, stride, up):
    import paper_2312_04429_amd as P
    print(f"wide conv {B}x{H}x{W} {C1}+{C2}->{Co} s{stride} u{up}", flush=True)
    g = torch.Generator().manual_seed(H * W + Co)
    C = C1 + C2
    x = torch.randn(B, H, W, C, generator=g).half()
    w = (torch.randn(Co, 3, 3, C, generator=g) / (9 * C) ** 0.5).half()
    b = torch.randn(Co, generator=g)
    x2 = x[..., C1:].contiguous().cuda() if C2 else None
    got = P.nv_op_conv3x3(x[..., :C1].contiguous().cuda(), w.cuda(), b.cuda(), stride=stride,
                          upsample=bool(up), x2=x2).cpu().double().numpy()

    def conv(a, k, bias):
        a = a.permute(0, 3, 1, 2)
        if up:
            a = a.repeat_interleave(2, 2).repeat_interleave(2, 3)
        return torch.nn.functional.conv2d(a, k.permute(0, 3, 1, 2), bias, stride=stride,
                                          padding=1).permute(0, 2, 3, 1).numpy()
    ref = conv(x.double(), w.double(), b.double())
    mag = conv(x.double().abs(), w.double().abs(), b.double().abs())
    _check(got, ref, mag, 9 * C)


# (tile rows, tile columns, wave groups that share out k) of the forms, in the rule's order
FORMS = [(256, 256, 1), (256, 160, 1), (128, 160, 1), (128, 160, 2), (128, 128, 1), (128, 80, 2),
         (64, 128, 2), (64, 80, 4), (64, 64, 2)]


def _code(form):
    bm, bn, shares = FORMS[form]
    return shares * 100_000_000 + bm * 10_000 + bn * 10 + 1


def _traced(P, call):
    P.nv_trace_enable(3, 8192)
    try:
        out = call()
        torch.cuda.synchronize()
    finally:
        P.nv_trace_disable()
    return out, [r[1] for r in P.nv_trace_records()]


def _linear(code, M, N, K):
    import paper_2312_04429_amd as P
    g = torch.Generator(device="cuda").manual_seed(M + N)
    x = torch.randn(M, K, generator=g, device="cuda").half()
    w = (0.05 * torch.randn(N, K, generator=g, device="cuda")).half()
    b = torch.randn(N, generator=g, device="cuda")
    r = torch.randn(M, N, generator=g, device="cuda").half()
    got, ran = _traced(P, lambda: P.nv_op_linear(x, w, b, r))
    assert [v for _, _, _, v in ran] == [code]
    ref = x.double() @ w.double().T + b.double() + r.double()
    mag = x.double().abs() @ w.double().abs().T + b.double().abs() + r.double().abs()
    _check(got.double().cpu().numpy(), ref.cpu().numpy(), mag.cpu().numpy(), K)


def _conv(code, B, H, W, C1, C2, Co, stride, up):
    import paper_2312_04429_amd as P
    g = torch.Generator(device="cuda").manual_seed(H * W + Co)
    C = C1 + C2
    x = torch.randn(B, H, W, C, generator=g, device="cuda").half()
    w = (torch.randn(Co, 3, 3, C, generator=g, device="cuda") / (9 * C) ** 0.5).half()
    b = torch.randn(Co, generator=g, device="cuda")
    x1, x2 = x[..., :C1].contiguous(), x[..., C1:].contiguous() if C2 else None
    got, ran = _traced(P, lambda: P.nv_op_conv3x3(x1, w, b, stride=stride, upsample=bool(up),
                                                  x2=x2))
    assert [v for _, _, _, v in ran] == [code]
    a = x.permute(0, 3, 1, 2)
    if up:
        a = a.repeat_interleave(2, 2).repeat_interleave(2, 3)
    a = torch.nn.functional.pad(a, (1, 1, 1, 1))
    ho, wo = got.shape[1:3]
    wf = w.reshape(Co, 9 * C).double()
    for i in range(B):  # one sample's taps at a time, in the weights' order
        cols = torch.stack([a[i, :, ky:ky + stride * (ho - 1) + 1:stride,
                              kx:kx + stride * (wo - 1) + 1:stride].reshape(C, ho * wo)
                            for ky in range(3) for kx in range(3)]).reshape(9 * C, ho * wo).double()
        ref = (wf @ cols).T + b.double()
        mag = (wf.abs() @ cols.abs()).T + b.double().abs()
        _check(got[i].reshape(ho * wo, Co).double().cpu().numpy(), ref.cpu().numpy(),
               mag.cpu().numpy(), 9 * C)


@pytest.mark.parametrize("form,M,N,K", [
    (0, 20552, 648, 192), (1, 21797, 264, 5120), (2, 16652, 264, 192), (3, 16548, 136, 320),
    (4, 16412, 88, 64), (5, 16396, 8, 64), (6, 8283, 72, 192), (7, 517, 4360, 192), (8, 1, 8, 64)])
def test_linear_each_form(form, M, N, K):
    print(f"wide linear form {form} M={M} N={N} K={K}", flush=True)
    _linear(_code(form), M, N, K)


@pytest.mark.parametrize("form,B,H,W,C1,C2,Co,stride,up", [
    (0, 4, 53, 58, 64, 0, 168, 1, 1), (0, 8, 43, 72, 64, 64, 416, 1, 0),
    (0, 8, 66, 68, 64, 0, 1640, 2, 0), (1, 3, 61, 70, 320, 128, 264, 1, 1),
    (1, 8, 62, 68, 320, 128, 1944, 2, 0), (2, 6, 45, 31, 64, 64, 144, 1, 1),
    (2, 8, 52, 58, 64, 0, 1288, 2, 0), (3, 8, 67, 31, 64, 64, 136, 1, 0),
    (3, 8, 56, 60, 64, 0, 536, 2, 0), (4, 4, 46, 34, 64, 64, 168, 1, 1),
    (4, 8, 60, 52, 64, 0, 904, 2, 0), (5, 4, 57, 72, 64, 64, 8, 1, 0),
    (5, 8, 70, 66, 64, 0, 136, 2, 0), (5, 3, 36, 38, 64, 0, 8, 1, 1),
    (6, 4, 35, 15, 64, 64, 88, 1, 1), (6, 8, 72, 70, 64, 0, 72, 2, 0),
    (7, 1, 50, 42, 64, 64, 72, 1, 1), (7, 8, 70, 60, 128, 0, 72, 2, 0),
    (8, 1, 4, 4, 64, 64, 8, 2, 0)])
def test_conv_each_form(form, B, H, W, C1, C2, Co, stride, up):
    print(f"wide conv form {form} {B}x{H}x{W} {C1}+{C2}->{Co} s{stride} u{up}", flush=True)
    _conv(_code(form), B, H, W, C1, C2, Co, stride, up)


# forms of the self-attention's q | k | v (folded LayerNorm, V transposed), of the cross-attention's
# q (folded LayerNorm) and of the GEGLU product (folded LayerNorm) over 1496 tokens a row
@pytest.mark.parametrize("C,heads,B,qkv,q,ff1", [(128, 4, 2, 5, 8, 4), (128, 4, 8, 6, 4, 4),
                                                 (320, 8, 4, 4, 3, 0), (320, 8, 8, 2, 2, 0)])
def test_network_epilogues(C, heads, B, qkv, q, ff1):
    import paper_2312_04429_amd as P
    import synth
    from oracle import schedule
    from oracle import unet as U
    cfg = synth.unet_config("tiny", H=88, W=68, ch=(64, C), n_heads=heads, mid_depth=0)
    w = dict(synth.make_weights(cfg, 0))
    rng = np.random.default_rng(C + B)
    for k in w:  # LayerNorms whose gains and shifts differ from channel to channel
        if ".ln" in k:
            w[k] = (w[k] + rng.uniform(-0.5, 0.5, w[k].shape)).astype(np.float32)
    print(f"wide network C={C} B={B}", flush=True)
    net = P.NvUNet(cfg, w)
    try:
        x = synth.make_latents(B, 4, 88, 68, 7)
        cond, unc = (synth.make_contexts(B, cfg["ctx_len"], cfg["ctx_dim"], s) for s in (11, 12))
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
        (eu, ec), ran = _traced(P, lambda: net.nv_unet_eps(t(x), [9] * B, t(cond), t(unc),
                                                           sched=(1000, 20, 0.00085, 0.012)))
        M = 2 * B * 44 * 34
        seen = {(n, k): v for m, n, k, v in ran if m == M}
        assert seen[3 * C, C] == _code(qkv)
        assert seen[8 * C, C] == _code(ff1)
        assert _code(q) in [v for m, n, k, v in ran if (m, n, k) == (M, C, C)]
        ora = U.UNet(cfg, w)
        ts = schedule.timesteps(20, 1000)[9]
        for b in (0, B - 1):
            for got, ctx in ((eu, unc), (ec, cond)):
                # the float16 bar of the network's other tests
                assert np.abs(got[b].cpu().numpy() - ora(x[b], ts, ctx[b])).max() <= 1e-2
    finally:
        net.close()


# tile rows, tile columns and splits of K; four and eight waves share a code (64 x 64 takes four
# beyond 512 workgroups, 128 x 128 for a long K over at least 128 tiles)
@pytest.mark.parametrize("bm,bn,splits,M,N,K", [
    (128, 128, 1, 8200, 964, 192), (128, 128, 1, 13200, 300, 128), (128, 128, 1, 8200, 965, 192),
    (64, 128, 1, 8200, 700, 192), (64, 128, 1, 1600, 1924, 128), (64, 64, 1, 2200, 1092, 192),
    (64, 64, 1, 1300, 668, 320), (64, 64, 1, 1300, 701, 320), (64, 64, 4, 300, 668, 2560),
    (64, 64, 2, 1200, 1004, 4096), (128, 128, 3, 1500, 1708, 8192)])
def test_linear_small_tiles(bm, bn, splits, M, N, K):
    print(f"small-tile linear {bm}x{bn}/{splits} M={M} N={N} K={K}", flush=True)
    _linear(bm * 10_000 + bn * 10 + splits, M, N, K)


@pytest.mark.parametrize("bm,bn,splits,B,H,W,C1,C2,Co,stride,up", [
    (128, 128, 1, 4, 128, 128, 64, 0, 36, 1, 0), (64, 128, 1, 3, 64, 60, 64, 0, 332, 1, 0),
    (64, 64, 1, 5, 60, 60, 64, 0, 68, 1, 0), (64, 64, 1, 3, 20, 20, 64, 64, 37, 1, 0),
    (64, 64, 1, 2, 20, 22, 64, 0, 260, 2, 0), (64, 64, 9, 2, 9, 10, 320, 320, 100, 1, 1),
    (128, 128, 9, 2, 30, 34, 640, 0, 260, 1, 0), (128, 128, 3, 2, 46, 45, 640, 384, 516, 1, 0)])
def test_conv_small_tiles(bm, bn, splits, B, H, W, C1, C2, Co, stride, up):
    print(f"small-tile conv {bm}x{bn}/{splits} {B}x{H}x{W} {C1}+{C2}->{Co} s{stride} u{up}",
          flush=True)
    _conv(bm * 10_000 + bn * 10 + splits, B, H, W, C1, C2, Co, stride, up)
