"""GPU parity of the general kernels (the shapes without a kernel of their own)
against the oracle at the edges of their tiles: one element more and less than
a tile of positions, channels and reduction chunks, every stride class of a
backward pass, planes smaller than a tile, and operands that are not finite.

Bound: both sides form the same fp32 (or bf16-rounded) products; the GPU adds
them in fp32, so the error of a sum of L products is at most L 2^-24 of the
sum of their magnitudes and typically sqrt(L) 2^-24 of their root mean square:
2e-5 of the largest result covers every L here (at most 12,800; one sum of
1,048,600 is formed in parts of at most 1,088)."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TOL = 2e-5


@pytest.fixture(scope="module")
def P():
    from paper_1912_12675_amd import psw
    psw.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return psw


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).float().cuda()


def close(gpu, ref, what):
    torch.cuda.synchronize()
    g, r = gpu.double().cpu().numpy(), np.asarray(ref, dtype=np.float64)
    err = np.abs(g - r).max() / max(np.abs(r).max(), 1e-30)
    assert g.shape == r.shape and err <= TOL, f"{what}: max err {err:.3e}"


CONV = [
    # N, C, H, W, K, R, S, stride, pad
    (1, 1, 1, 1, 1, 1, 1, 1, 0),
    (2, 3, 17, 15, 6, 5, 5, 1, 2),       # one octet of channels, 16 output channels
    (1, 8, 32, 33, 33, 3, 3, 1, 1),      # one octet, a block of 64 output channels
    (3, 9, 31, 8, 64, 3, 3, 1, 1),       # 9 channels: two octets, the second nearly empty
    (2, 17, 15, 16, 65, 3, 3, 1, 1),     # one past a 16-channel chunk and a 64-channel block
    (2, 31, 16, 17, 63, 3, 3, 1, 1),
    (130, 33, 4, 4, 70, 3, 3, 1, 1),     # several images per tile, one past a 32-channel chunk
    (129, 64, 2, 2, 40, 3, 3, 1, 1),
    (130, 24, 14, 14, 33, 3, 3, 1, 1),   # planes a little smaller than a tile, and than a part of one
    (130, 40, 7, 7, 70, 3, 3, 1, 1),
    (40, 40, 1, 1, 48, 3, 3, 1, 1),
    (2, 24, 29, 23, 56, 3, 3, 2, 1),     # stride 2: four classes backward, odd plane
    (2, 20, 13, 14, 24, 5, 5, 3, 2),     # stride 3: nine classes
    (2, 20, 9, 9, 24, 1, 1, 2, 0),       # classes without a tap
    (2, 12, 6, 7, 20, 2, 3, 1, 2),       # a rectangular kernel, padding past it
    (2, 40, 12, 12, 17, 1, 1, 1, 0),
    (2, 64, 16, 16, 96, 5, 5, 1, 2),
    (1, 512, 4, 4, 512, 3, 3, 1, 1),
    (64, 16, 32, 32, 20, 3, 3, 1, 1),    # wide tiles of 32 output channels
    (64, 40, 32, 32, 64, 3, 3, 1, 0),    # ... of 64: two blocks, 512 in all
    (65, 40, 32, 32, 64, 3, 3, 1, 0),    # ... and more
    (65, 16, 30, 30, 16, 3, 3, 1, 1),    # wide tiles of 16
    (33, 16, 30, 30, 16, 3, 3, 1, 1),    # too few for those
    (9, 70, 13, 11, 130, 1, 1, 1, 0),    # 1x1 weight gradients of two blocks of 64 rows and of 64 channels, both ragged
    (9, 70, 13, 11, 130, 1, 1, 2, 0),
    (9, 16, 13, 11, 130, 1, 1, 1, 0),    # ... of one block of 16 channels
    (11, 3, 13, 11, 29, 1, 1, 2, 0),
    (4, 17, 14, 13, 15, 1, 1, 1, 0),     # ... of one channel past it
    (41, 20, 19, 21, 70, 5, 5, 1, 2),    # 5x5 weight gradients of 64 rows, whose steps take two sums in bf16
    (1, 24, 29, 23, 56, 3, 3, 2, 1),     # one image: weight gradients by the implicit GEMM
    (2, 64, 55, 57, 128, 3, 3, 2, 1),    # two: by it, and in bf16 not
    (3, 20, 21, 23, 40, 3, 3, 1, 0),
    (1, 4, 40, 40, 4, 9, 9, 4, 4),
    (21, 61, 10, 9, 50, 1, 1, 1, 0),     # 1x1 on planes that no power of two divides
    (19, 1, 8, 13, 152, 1, 1, 1, 0),
    (40, 24, 29, 23, 56, 3, 3, 2, 1),    # stride 2: 320 blocks of 32 x 64, the first that take it
    (39, 24, 29, 23, 56, 3, 3, 2, 1),    # one image fewer
    (3, 1, 28, 28, 6, 5, 5, 1, 2),       # one octet of channels: 16 output channels of 64 positions
    (37, 5, 28, 27, 16, 5, 5, 1, 2),     # ... of 128
    (257, 3, 32, 31, 13, 3, 3, 1, 1),    # ... of 256
    (130, 8, 21, 19, 15, 1, 1, 1, 0),    # ... with few taps
    (86, 6, 21, 19, 50, 3, 3, 2, 1),     # 32 output channels of 128
    (65, 3, 64, 62, 70, 3, 3, 1, 1),     # 64 of 256
    (17, 3, 64, 64, 40, 11, 11, 4, 2),   # a halo that leaves room for one workgroup a CU
    (86, 3, 64, 64, 40, 11, 11, 4, 2),   # ... and more tiles than those pay for
    (2, 5, 40, 40, 20, 13, 13, 3, 6),
]


def conv_data(case):
    N, C, H, W, K, R, S, st, pad = case
    rng = np.random.default_rng(sum(case) * 7 + K)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)  # noqa: E731
    Pq, Qq = (H + 2 * pad - R) // st + 1, (W + 2 * pad - S) // st + 1
    return f(N, C, H, W), f(K, C, R, S) * 0.3, f(K), f(N, K, Pq, Qq), f(N, C, H, W)


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("case", CONV, ids=lambda c: "x".join(map(str, c)))
def test_conv_edges(P, case, bf16):
    print("conv", case, bf16, flush=True)
    N, C, H, W, K, R, S, st, pad = case
    x, w, b, dy, base = conv_data(case)
    rd = lambda a: (torch.from_numpy(a).bfloat16() if bf16 else torch.from_numpy(a)).double()  # noqa: E731
    y = torch.empty(dy.shape, device="cuda")
    ref = torch.nn.functional.conv2d(rd(x), rd(w), None, st, pad).numpy()
    xg, wg, dyg = dev(x), dev(w), dev(dy)
    P.psw_conv_fwd(xg, wg, y, st, pad, bf16=bf16)
    close(y, ref, "fwd")
    P.psw_conv_fwd(xg, wg, y, st, pad, bias=dev(b), relu=True, bf16=bf16)
    close(y, np.maximum(ref + b[None, :, None, None], 0), "fwd + bias + relu")
    refdx = torch.nn.grad.conv2d_input(x.shape, rd(w), rd(dy), st, pad).numpy()
    dx = torch.full(x.shape, 7.0, device="cuda")
    P.psw_conv_bwd_data(x.shape, wg, dyg, dx, st, pad, bf16=bf16)
    close(dx, refdx, "bwd_data")
    dx = dev(base)
    P.psw_conv_bwd_data(x.shape, wg, dyg, dx, st, pad, accumulate=True, bf16=bf16)
    close(dx, refdx + base, "bwd_data accumulate")
    refdw = torch.nn.grad.conv2d_weight(rd(x), w.shape, rd(dy), st, pad).numpy()
    dw, db = torch.full(w.shape, 7.0, device="cuda"), torch.full((K,), 7.0, device="cuda")
    P.psw_conv_bwd_weight(xg, dyg, dw, st, pad, dbias=db, bf16=bf16)
    close(dw, refdw, "bwd_weight")
    close(db, dy.astype(np.float64).sum((0, 2, 3)), "bwd_bias")


def same_class(gpu, ref, what):
    """Finite values close (those beyond 1e30, one huge product, by themselves); infinities and NaNs alike."""
    torch.cuda.synchronize()
    g, r = gpu.double().cpu().numpy(), ref.float().double().numpy()
    assert np.array_equal(np.isnan(g), np.isnan(r)), what
    assert np.array_equal(g[np.isinf(r)], r[np.isinf(r)]) and np.array_equal(np.isinf(g), np.isinf(r)), what
    big = np.isfinite(r) & (np.abs(r) > 1e30)
    assert np.allclose(g[big], r[big], rtol=1e-5), what
    fin = np.isfinite(r) & ~big
    assert np.abs(g[fin] - r[fin]).max() <= TOL * np.abs(r[fin]).max(), what


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("case", [(2, 40, 12, 12, 70, 3, 3, 1, 0), (2, 12, 9, 9, 20, 3, 3, 2, 0),
                                  (3, 20, 8, 8, 12, 1, 1, 1, 0), (3, 24, 13, 11, 40, 3, 3, 1, 1),
                                  (2, 8, 14, 13, 20, 5, 5, 1, 0)], ids=lambda c: "x".join(map(str, c)))
def test_conv_not_finite(P, case, bf16):
    """An infinity, a NaN and the largest float among the operands (an infinity in bf16) reach exactly the
    sums they enter: also those in the last row and column of a plane, which a chunk of the weight gradient
    that reaches past the output plane meets with zeros, and those that a forward group's unused slots read."""
    print("conv not finite", case, bf16, flush=True)
    N, C, H, W, K, R, S, st, pad = case
    x, w, _, dy, _ = conv_data(case)
    w[np.abs(w) < 1e-3] = 0.01
    x[0, 3, 4, 4], x[1, 5, 2, 2], x[1, 0, 0, 0], x[N - 1, 2, H - 1, W - 1] = np.inf, np.nan, 3.4e38, np.inf
    dy[1, :, 0, 0] *= 0.1  # a product of the largest float that float32 holds
    dy[0, 1, 1, 1], dy[1, 2, 2, 2] = -np.inf, np.nan
    d = lambda a: (torch.from_numpy(a).bfloat16() if bf16 else torch.from_numpy(a)).double()  # noqa: E731
    y = torch.empty(dy.shape, device="cuda")
    P.psw_conv_fwd(dev(x), dev(w), y, st, pad, bf16=bf16)
    same_class(y, torch.nn.functional.conv2d(d(x), d(w), None, st, pad), "fwd")
    dx = torch.empty(x.shape, device="cuda")
    P.psw_conv_bwd_data(x.shape, dev(w), dev(dy), dx, st, pad, bf16=bf16)
    same_class(dx, torch.nn.grad.conv2d_input(x.shape, d(w), d(dy), st, pad), "bwd_data")
    dw = torch.empty(w.shape, device="cuda")
    P.psw_conv_bwd_weight(dev(x), dev(dy), dw, st, pad, bf16=bf16)
    same_class(dw, torch.nn.grad.conv2d_weight(d(x), w.shape, d(dy), st, pad), "bwd_weight")


def fp32_error(L):
    """Relative error (2-norm) of a sum of L products of zero mean with a rounding every four: each rounding errs
    2.5e-8 of the running sum (half an ulp, uniform), whose square grows with its length, so sqrt(L / 4 / 2) of
    those, and the result's own.  The fp32 matrix instructions round at each product: twice that."""
    return 2.5e-8 * (math.sqrt(L / 8) + 1)


@pytest.mark.parametrize("case", [(64, 256, 14, 14, 256, 3, 3, 1, 1), (16, 1, 28, 28, 6, 5, 5, 1, 2),
                                  (64, 128, 16, 16, 192, 1, 1, 1, 0)], ids=lambda c: "x".join(map(str, c)))
def test_conv_error_is_fp32s(P, case):
    """Products in three bfloat16 parts: nearer to 64 bits than the fp32 matrix instructions' sums."""
    print("conv error", case, flush=True)
    N, C, H, W, K, R, S, st, pad = case
    g = torch.Generator(device="cuda").manual_seed(5)
    x, w = torch.randn(N, C, H, W, generator=g, device="cuda"), torch.randn(K, C, R, S, generator=g, device="cuda")
    cols = torch.nn.functional.unfold(x.double(), (R, S), padding=pad, stride=st)
    want = w.double().view(K, -1) @ cols
    y = torch.empty(N, K, H, W, device="cuda")
    P.psw_conv_fwd(x, w, y, st, pad)
    assert float((y.view(N, K, -1) - want).norm() / want.norm()) <= fp32_error(C * R * S)
    dy = torch.randn(N, K, H, W, generator=g, device="cuda")
    dw = torch.empty_like(w)
    P.psw_conv_bwd_weight(x, dy, dw, st, pad)
    want = (dy.double().view(N, K, -1) @ cols.transpose(1, 2).contiguous()).sum(0).view(w.shape)
    assert float((dw - want).norm() / want.norm()) <= fp32_error(N * H * W)


@pytest.mark.parametrize("case", [(128, 4096, 4096), (200, 250, 2500), (16, 400, 120)], ids=lambda c: "x".join(map(str, c)))
def test_fc_error_is_fp32s(P, case):
    print("fc error", case, flush=True)
    n, fin, out = case
    g = torch.Generator(device="cuda").manual_seed(6)
    x, w, dy = (torch.randn(*s, generator=g, device="cuda") for s in ((n, fin), (out, fin), (n, out)))
    y, dx, dw = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(w)
    P.psw_fc_fwd(x, w, y)
    P.psw_fc_bwd(x, w, dy, dw, dx=dx)
    for got, want, L in ((y, x.double() @ w.double().t(), fin), (dx, dy.double() @ w.double(), out),
                         (dw, dy.double().t() @ x.double(), n)):
        assert float((got - want).norm() / want.norm()) <= fp32_error(L)


@pytest.mark.parametrize("scale", [1e-28, 1e-33, 1e-36])
def test_tiny_operands(P, scale):
    """Operands whose third bfloat16 part is at or past that format's smallest number: still fp32's error (twice
    that of a rounding every four products, since these sums are formed one product at a time)."""
    print("tiny", scale, flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    x, w, dy = rnd(9, 40, 12, 12), rnd(70, 40, 3, 3) * 0.1, rnd(9, 70, 10, 10)
    cols = lambda t: torch.nn.functional.unfold(t.double(), 3)  # noqa: E731
    err = lambda got, want: float((got - want).norm() / want.norm())  # noqa: E731
    y, dx, dw = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(w)
    P.psw_conv_fwd(x * scale, w, y, 1, 0)
    assert err(y.view(9, 70, -1), w.double().view(70, -1) @ cols(x * scale)) <= 2 * fp32_error(360)
    P.psw_conv_bwd_weight(x * scale, dy, dw, 1, 0)
    want = (dy.double().view(9, 70, -1) @ cols(x * scale).transpose(1, 2).contiguous()).sum(0).view(w.shape)
    assert err(dw, want) <= 2 * fp32_error(900)
    P.psw_conv_bwd_data(x.shape, w, dy * scale, dx, 1, 0)
    back = w.double().view(70, -1).t().contiguous() @ (dy * scale).double().view(9, 70, -1)
    assert err(dx, torch.nn.functional.fold(back, (12, 12), 3)) <= 2 * fp32_error(630)
    fx, fw, fdy = rnd(300, 700), rnd(200, 700) * 0.1, rnd(300, 200)
    y, dx, dw = torch.empty_like(fdy), torch.empty_like(fx), torch.empty_like(fw)
    P.psw_fc_fwd(fx * scale, fw, y)
    assert err(y, (fx * scale).double() @ fw.double().t()) <= 2 * fp32_error(700)
    P.psw_fc_bwd(fx, fw, fdy * scale, dw, dx=dx)
    assert err(dx, (fdy * scale).double() @ fw.double()) <= 2 * fp32_error(200)
    assert err(dw, (fdy * scale).double().t() @ fx.double()) <= 2 * fp32_error(300)


def test_products_near_the_largest_float(P):
    """3.3895e38 * 1.00391 is a float; the product of the two rounded to bfloat16 is not."""
    big, f = 3.3895e38, 1.00391
    x, w = torch.zeros(2, 12, 5, 5), torch.full((20, 12, 1, 1), f)
    x[1, 3, 2, 2] = big
    y = torch.empty(2, 20, 5, 5, device="cuda")
    P.psw_conv_fwd(x.cuda(), w.cuda(), y, 1, 0)
    want = torch.zeros(2, 20, 5, 5)
    want[1, :, 2, 2] = x[1, 3, 2, 2] * w[0, 0, 0, 0]
    assert want.isfinite().all() and torch.allclose(y.cpu(), want, rtol=1e-6, atol=0)
    dy, dw = torch.zeros(2, 20, 5, 5), torch.empty(20, 12, 1, 1, device="cuda")
    dy[1, 4, 2, 2] = f
    P.psw_conv_bwd_weight(x.cuda(), dy.cuda(), dw, 1, 0)
    assert torch.allclose(dw.cpu()[4, 3, 0, 0], want[1, 0, 2, 2], rtol=1e-6) and dw.isfinite().all()
    fx, fw, fy = torch.zeros(300, 40), torch.full((70, 40), f), torch.empty(300, 70, device="cuda")
    fx[7, 9] = big
    P.psw_fc_fwd(fx.cuda(), fw.cuda(), fy)
    assert torch.allclose(fy.cpu()[7], want[1, 0, 2, 2].expand(70), rtol=1e-6) and fy.isfinite().all()


FC = [
    # N, in, out
    (1, 1, 65),
    (3, 5, 65),
    (16, 400, 120),      # LeNet-5
    (16, 120, 84),
    (17, 33, 129),
    (33, 31, 4096),      # outputs by the row, a reduction shorter than a step
    (129, 70, 2049),     # 128, 64 and 32 rows a block, each with a part block, column and step
    (65, 99, 4100),
    (40, 97, 4098),
    (101, 10500, 2600),  # an x past 4 MB: in bf16 the tile of 128 rows
    (101, 10500, 1030),  # ... too few columns for it
    (1, 4097, 70),       # deep reductions, one k past a stage
    (20, 2047, 66),
    (130, 130, 66),
    (257, 16, 10),       # more rows than the small classifier takes
    (128, 5000, 300),
    (300, 200, 1100),    # rows past gemm_rows' 256
    (130, 2900, 3000),   # tiles of 128 x 128 in the weight gradient
    (129, 40, 33000),    # ... in the forward
    (129, 33000, 40),    # ... in the input gradient
    (128, 96, 16400),
    (33, 70, 16400),     # few k over many columns: 64 x 64 tiles in the forward
    (20, 70, 9000),      # the input's gradient over a deep k, in parts whose sums meet: few tiles
    (130, 1100, 2100),   # ... more of them
    (128, 4100, 530),    # ... 130 of 64 x 64, the last part short
    (5, 33001, 20),      # few rows, few k, many columns: one a thread
    (3, 262148, 17),     # ... four a thread, a second block of rows in dw
    (3, 5, 1048600),     # rows past the larger tiles' 31-bit offsets
]


def fc_data(case):
    n, fin, out = case
    rng = np.random.default_rng(n * 31 + fin * 7 + out)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)  # noqa: E731
    return f(n, fin), f(out, fin) * 0.3, f(out), f(n, out), f(n, fin)


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("case", FC, ids=lambda c: "x".join(map(str, c)))
def test_fc_edges(P, case, bf16):
    print("fc", case, bf16, flush=True)
    x, w, b, dy, base = fc_data(case)
    rd = lambda a: (torch.from_numpy(a).bfloat16() if bf16 else torch.from_numpy(a)).double()  # noqa: E731
    y = torch.empty(dy.shape, device="cuda")
    ref = (rd(x) @ rd(w).t()).numpy()
    P.psw_fc_fwd(dev(x), dev(w), y, bf16=bf16)
    close(y, ref, "fwd")
    P.psw_fc_fwd(dev(x), dev(w), y, b=dev(b), relu=True, bf16=bf16)
    close(y, np.maximum(ref + b, 0), "fwd + bias + relu")
    refdx, refdw = (rd(dy) @ rd(w)).numpy(), (rd(dy).t() @ rd(x)).numpy()
    dx, dw, db = (torch.full(s, 7.0, device="cuda") for s in (x.shape, w.shape, b.shape))
    P.psw_fc_bwd(dev(x), dev(w), dev(dy), dw, dx=dx, db=db, bf16=bf16)
    close(dx, refdx, "dx")
    close(dw, refdw, "dw")
    close(db, dy.astype(np.float64).sum(0), "db")
    dx = dev(base)
    P.psw_fc_bwd(dev(x), dev(w), dev(dy), dw, dx=dx, dx_accumulate=True, bf16=bf16)
    close(dx, refdx + base, "dx accumulate")


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("case", [(1, 33554500, 2), (2, 8388700, 3), (2, 3, 8388700)],
                         ids=lambda c: "x".join(map(str, c)))
def test_fc_rows_past_31_bits(P, case, bf16):
    """Rows whose byte offsets pass 31 bits within a tile.  x, w and dy hold 200 values each among zeros (the
    first and last elements among them), so every sum is short and the same bound holds."""
    print("fc far", case, bf16, flush=True)
    n, fin, out = case
    g = torch.Generator().manual_seed(fin + out)

    def sparse(rows, cols):
        t = torch.zeros(rows * cols, device="cuda")
        at = torch.randint(t.numel(), (200,), generator=g)
        at[0], at[1] = 0, t.numel() - 1
        at[2:100] = torch.randint(max(0, cols - 60), cols, (98,), generator=g) + cols * torch.randint(rows, (98,), generator=g)
        t[at.cuda()] = torch.randn(200, generator=g).cuda()
        return t.view(rows, cols)

    x, w, dy = sparse(n, fin), sparse(out, fin), sparse(n, out)
    rd = lambda a: (a.bfloat16() if bf16 else a).double()  # noqa: E731
    outer = lambda a, b: sum(a[:, k, None] * b[None, k] for k in range(a.shape[1]))  # noqa: E731
    y, dx, dw, db = (torch.full(s, 7.0, device="cuda") for s in (dy.shape, x.shape, w.shape, (out,)))
    P.psw_fc_fwd(x, w, y, bf16=bf16)
    P.psw_fc_bwd(x, w, dy, dw, dx=dx, db=db, bf16=bf16)

    def same(got, want):  # on the GPU: the tensors are large
        assert got.shape == want.shape and bool((got.double() - want).abs().max() <= TOL * want.abs().max())

    same(y, torch.stack([(rd(x[i]) * rd(w)).sum(1) for i in range(n)]))
    same(dx, torch.stack([(rd(dy[i])[:, None] * rd(w)).sum(0) for i in range(n)]))
    same(dw, outer(rd(dy).t(), rd(x)))
    same(db, dy.double().sum(0))


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("case", [(20, 300, 130), (5, 1500, 70)], ids=lambda c: "x".join(map(str, c)))
def test_fc_not_finite(P, case, bf16):
    print("fc not finite", case, bf16, flush=True)
    x, w, _, dy, _ = fc_data(case)
    w[np.abs(w) < 1e-3] = 0.01
    x[0, 3], x[1, 5], x[2, 7] = np.inf, np.nan, 3.4e38
    dy[2] *= 0.1  # a product of the largest float that float32 holds
    dy[3, 4], dy[4, 1] = -np.inf, np.nan
    d = lambda a: (torch.from_numpy(a).bfloat16() if bf16 else torch.from_numpy(a)).double()  # noqa: E731
    y, dx, dw = (torch.empty(s, device="cuda") for s in (dy.shape, x.shape, w.shape))
    P.psw_fc_fwd(dev(x), dev(w), y, bf16=bf16)
    same_class(y, d(x) @ d(w).t(), "fwd")
    P.psw_fc_bwd(dev(x), dev(w), dev(dy), dw, dx=dx, bf16=bf16)
    same_class(dx, d(dy) @ d(w), "dx")
    same_class(dw, d(dy).t() @ d(x), "dw")


BN = [
    # N, C, H, W, residual, relu: wide and flat planes, by fours and one by one, odd images and channels
    (3, 3, 1, 2, None, False),  # six values a channel (of two, dy is nothing but cancellation)
    (5, 7, 3, 5, "identity", True),
    (33, 300, 2, 2, "identity", True),
    (17, 64, 4, 4, None, True),
    (9, 40, 8, 8, "half", True),
    (6, 20, 15, 17, "identity", True),     # 255 elements: one by one, a plane just below a block
    (6, 20, 16, 16, "half", False),
    (3, 12, 14, 18, "third", True),        # 252 = 63 units: the largest flat plane
    (130, 5, 16, 16, None, True),
    (2, 4, 66, 66, "half", True),
    (1001, 5, 1, 1, None, True),           # planes of one: 51 images side by side, the last group short
    (2050, 3, 2, 2, "identity", True),     # ... 85 by fours
    (77, 130, 1, 1, None, False),          # one image at a time, a second block part full
    (1, 1, 2, 3, None, False),             # one image, one channel
]


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("case", BN, ids=lambda c: "x".join(map(str, c)))
def test_bn_edges(P, case, accumulate):
    """Sums are taken in double; what is left is the rounding of a few float operations per element."""
    print("bn", case, accumulate, flush=True)
    N, C, H, W, kind, relu = case
    rng = np.random.default_rng(N * 100 + C)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)  # noqa: E731
    y, gamma, beta, dz = f(N, C, H, W) * 2 + 0.5, f(C), f(C), f(N, C, H, W)
    z0 = np.maximum(f(N, C, H, W), 0)  # the output the backward pass masks by
    fac, rc = {"half": (2, C // 2), "third": (3, C // 3)}.get(kind, (1, C))
    res = None if kind is None else f(N, rc, H * fac, W * fac)
    lo = (C - rc) // 2
    t = lambda a: torch.from_numpy(a).double()  # noqa: E731
    mean, var = t(y).mean((0, 2, 3)), t(y).var((0, 2, 3), unbiased=False)
    inv = 1 / torch.sqrt(var + 1e-5)
    v = lambda a: a.view(1, -1, 1, 1)  # noqa: E731
    xh = (t(y) - v(mean)) * v(inv)
    ref = xh * v(t(gamma)) + v(t(beta))
    if res is not None:
        ref = ref + torch.nn.functional.pad(t(res)[:, :, ::fac, ::fac], (0, 0, 0, 0, lo, lo))
    ref = ref.clamp(min=0) if relu else ref
    out = torch.empty(y.shape, device="cuda")
    sm, si, dg, db = (torch.empty(C, device="cuda") for _ in range(4))
    rm, rv = torch.zeros(C, device="cuda"), torch.ones(C, device="cuda")
    P.psw_bn_relu_fwd(dev(y), dev(gamma), dev(beta), out, sm, si, res=None if res is None else dev(res), relu=relu,
                      run_mean=rm, run_var=rv)
    m = N * H * W
    for got, want, what in ((out, ref, "z"), (sm, mean, "mean"), (si, inv, "invstd"), (rm, 0.1 * mean, "run_mean"),
                            (rv, 0.9 + 0.1 * var * (m / (m - 1)), "run_var")):
        close(got, want.numpy(), what)
    g = t(dz) * (t(z0) > 0) if relu else t(dz)
    sb, sg = g.sum((0, 2, 3)), (g * xh).sum((0, 2, 3))
    refdy = v(t(gamma) * inv) * (g - v(sb) / m - xh * v(sg) / m)
    dy = torch.empty(y.shape, device="cuda")
    dres = base = None
    if res is not None:
        base = f(*res.shape)
        dres = dev(base)
        refres = torch.zeros(res.shape, dtype=torch.float64)
        refres[:, :, ::fac, ::fac] = g[:, lo:lo + rc]
        refres = refres + t(base) if accumulate else refres
    P.psw_bn_relu_bwd(dev(dz), dev(z0), dev(y), dev(gamma), sm, si, dy, dg, db, dres=dres, relu=relu,
                      res_accumulate=accumulate)
    close(dg, sg.numpy(), "dgamma")
    close(db, sb.numpy(), "dbeta")
    close(dy, refdy.numpy(), "dy")
    if res is not None:
        close(dres, refres.numpy(), "dres")


@pytest.mark.parametrize("case", [(1200001, 3, 1, 1), (1, 1, 8201, 8201)], ids=lambda c: "x".join(map(str, c)))
def test_bn_blocks_past_16_bits(P, case):
    """More blocks of images, or of a channel's units, than a grid's second dimension holds."""
    print("bn blocks", case, flush=True)
    g = torch.Generator(device="cuda").manual_seed(4)
    n, c, h, w = case
    y, dz = (torch.randn(*case, generator=g, device="cuda") for _ in range(2))
    gamma, beta = (torch.randn(c, generator=g, device="cuda") for _ in range(2))
    out, dy = torch.empty_like(y), torch.empty_like(y)
    sm, si, dg, db = (torch.empty(c, device="cuda") for _ in range(4))
    P.psw_bn_relu_fwd(y, gamma, beta, out, sm, si, relu=True)
    v = lambda a: a.double().view(1, -1, 1, 1)  # noqa: E731
    inv = 1 / torch.sqrt(y.double().var((0, 2, 3), unbiased=False) + 1e-5)
    xh = (y.double() - v(y.double().mean((0, 2, 3)))) * v(inv)
    want = (xh * v(gamma) + v(beta)).clamp(min=0)
    assert bool((out.double() - want).abs().max() <= TOL * want.abs().max())
    P.psw_bn_relu_bwd(dz, out, y, gamma, sm, si, dy, dg, db, relu=True)
    gz = dz.double() * (out > 0)
    sb, sg, m = gz.sum((0, 2, 3)), (gz * xh).sum((0, 2, 3)), n * h * w
    want = v(gamma) * v(inv) * (gz - v(sb) / m - xh * v(sg) / m)
    assert bool((dy.double() - want).abs().max() <= TOL * want.abs().max())
    assert torch.allclose(dg.double(), sg, rtol=1e-5, atol=1e-3) and torch.allclose(db.double(), sb, rtol=1e-5, atol=1e-3)


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("case", [(3, 5, 8, 8, 2), (2, 3, 9, 12, 2), (2, 3, 7, 10, 2), (2, 3, 8, 7, 2), (1, 1, 2, 2, 2),
                                  (2, 4, 11, 13, 3), (5, 67, 32, 32, 2)], ids=lambda c: "x".join(map(str, c)))
def test_maxpool_edges(P, case, accumulate):
    """Rows by fours, by twos and one by one, planes with a row or column no window covers; ties and NaNs: exact."""
    print("pool", case, accumulate, flush=True)
    N, C, H, W, k = case
    rng = np.random.default_rng(N + H * W)
    x = np.maximum(rng.integers(-3, 4, (N, C, H, W)), 0).astype(np.float32)
    x[0, 0, 0, 0], x[0, 0, 1, 1], x[-1, -1, 0, 1] = np.nan, np.inf, np.nan
    p, q = H // k, W // k
    win = x[:, :, :p * k, :q * k].reshape(N, C, p, k, q, k).transpose(0, 1, 2, 4, 3, 5).reshape(N, C, p, q, k * k)
    best, at = win[..., 0].copy(), np.zeros((N, C, p, q), dtype=np.int64)
    for e in range(1, k * k):
        better = win[..., e] > best
        best[better], at[better] = win[..., e][better], e
    flat = (np.arange(p)[:, None] * k + at // k) * W + np.arange(q) * k + at % k
    y, arg = torch.empty((N, C, p, q), device="cuda"), torch.empty((N, C, p, q), dtype=torch.int32, device="cuda")
    P.psw_pool_fwd(P.PSW_POOL_MAX, dev(x), y, k, k, argmax=arg)
    assert np.array_equal(y.cpu().numpy(), best, equal_nan=True) and np.array_equal(arg.cpu().numpy(), flat)
    dy, base = (rng.standard_normal(s).astype(np.float32) for s in (best.shape, x.shape))
    ref = np.zeros((N, C, H * W), dtype=np.float32)
    np.put_along_axis(ref, flat.reshape(N, C, -1), dy.reshape(N, C, -1), 2)
    dx = dev(base)
    P.psw_pool_bwd(P.PSW_POOL_MAX, x.shape, dev(dy), dx, k, k, argmax=arg, accumulate=accumulate)
    ref = ref.reshape(x.shape) + base if accumulate else ref.reshape(x.shape)
    assert np.array_equal(dx.cpu().numpy(), ref)


@pytest.mark.parametrize("n,classes", [(1, 1), (3, 2), (1024, 1), (1025, 3), (16, 64), (17, 65), (250, 100), (5, 1000),
                                       (2100, 33)])
def test_softmax_xent_lanes(P, n, classes):
    """Each number of lanes a row can get, a last pass of rows that is part full, classes that are not a
    multiple of the lanes; a row of which one logit is -inf, and one that has a NaN."""
    g = torch.Generator().manual_seed(n * classes)
    z = torch.randn(n, classes, generator=g) * 3
    if n > 2 and classes > 1:
        z[1, 0] = -math.inf
    lab = torch.randint(classes, (n,), generator=g, dtype=torch.int32)
    if n > 2 and classes > 1:
        lab[1] = classes - 1
    loss, dz = torch.empty(1, device="cuda"), torch.empty(n, classes, device="cuda")
    P.psw_softmax_xent(z.cuda(), lab.cuda(), loss, dz)
    p = torch.log_softmax(z.double(), 1)
    want = (p.exp() - torch.nn.functional.one_hot(lab.long(), classes)) / n
    # z - max and z - lse round at |z| + |lse| < 2 * 16 + 7, the sum of the classes at most `classes` times,
    # exp and log at a few ulp
    eps = 2.0 ** -24
    tol = (2 * (2 * 16 + 7) + classes + 16) * eps
    assert ((dz.cpu().double() - want).abs() <= tol / n).all()
    assert abs(float(loss) - float(-p[torch.arange(n), lab.long()].mean())) <= tol
    if n > 2 and classes > 1:
        z[2, classes - 1] = math.nan
        P.psw_softmax_xent(z.cuda(), lab.cuda(), loss, dz)
        assert dz[2].isnan().all() and not dz[torch.arange(n) != 2].isnan().any() and loss.isnan().all()
