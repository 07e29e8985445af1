"""GPU parity of the wide GEMM forms (whole-chip tiles, k halves and k teams, the row-staged
epilogue) at the edges of their tiles: ragged rows and columns, one k tile (a team without
one), odd k tile counts, two sources, strided and upsampling convolutions."""
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
