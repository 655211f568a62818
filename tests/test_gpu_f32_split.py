"""fp32 products on the bf16 matrix instructions (csrc/gemm_f32_split.hip): three bf16 terms an operand element."""
import pytest

from tests.f32_form import split_tile, split_tiles

FP32 = 0


def test_split_tiles_keep_out_where_they_would_lose():
    """Short reductions, results small enough for 16x16 tiles, weight gradients whose eight-way sums are the more exact ones, and
    more tiles than a launch has threads for."""
    for wgrad in (False, True):
        assert split_tile(4096, 4096, 255, wgrad) == 0 and split_tile(4096, 4096, 256, wgrad) == 128
        assert split_tile(256, 256, 8192, wgrad) == 0
        assert split_tile(8, 1 << 26, 256, wgrad) == 0
    assert split_tile(1032, 520, 2000, True) == 0 and split_tile(1032, 520, 2000, False) == 64


@pytest.fixture(scope="module")
def env():
    from tests.gpu_util import require_gpu
    require_gpu()
    import torch

    import paper_2412_12636_amd as tm
    return torch, tm, int(torch.cuda.current_stream().cuda_stream)


def close(got, ref, size, n):
    """|got - ref| against the sums' roundings: six terms for every 16 of n products and the meeting of four waves, each half an
    ulp of at most the sum of the magnitudes `size`; the products left out are 2^-24 of each."""
    return bool(((got.double() - ref).abs() <= (0.375 * n + 8) * 2.0 ** -24 * size + 1e-44).all())


@pytest.mark.gpu
@pytest.mark.parametrize("T,N,K,tiles", [
    (1000, 1000, 1000, (64, 64, 64)),          # a reduction that ends inside a stage, edges inside a tile
    (3077, 776, 2056, (128, 128, 64)),         # odd token counts; 2056 = 64 stages of 32 and 8 elements
    (1100, 1928, 1992, (64, 64, 128)),
    (1601, 1640, 328, (128, 64, 0)),           # one row and one column of tiles nearly empty
    (1023, 1544, 520, (0, 64, 64)),            # weight gradient over 1023 tokens
    (2048, 2048, 256, (128, 0, 0)),            # the shortest reduction
])
def test_products_of_split_operands(env, T, N, K, tiles):
    """Forward with and without bias and residual, input gradient, weight gradient stored and added, against 64 bits and the bound
    of the sums; then with an infinite and a tiny row in x and a NaN in dy: only what reads those is not finite, and the
    tiny row's results keep their precision."""
    torch, tm, s = env
    assert split_tiles(T, N, K) == tiles
    print(f"split fp32 products T={T} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(T + N)
    rnd = lambda *shape: torch.randn(shape, device="cuda", generator=g)
    x, w, dy, bias, res, dw0 = rnd(T, K), rnd(N, K) * 0.05, rnd(T, N) * 0.1, rnd(N), rnd(T, N), rnd(N, K)
    X, W, D = x.double(), w.double(), dy.double()
    ax, aw, ad = X.abs(), W.abs(), D.abs()
    y, dx, dw = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(w)
    tm.tm_op_linear_fwd(FP32, T, N, K, x, w, None, None, y, s)
    assert close(y, X @ W.t(), ax @ aw.t(), K)
    tm.tm_op_linear_fwd(FP32, T, N, K, x, w, bias, res, y, s)
    assert close(y, X @ W.t() + bias.double() + res.double(), ax @ aw.t() + bias.double().abs() + res.double().abs(), K)
    tm.tm_op_linear_dgrad(FP32, T, N, K, dy, w, dx, s)
    assert close(dx, D @ W, ad @ aw, N)
    tm.tm_op_linear_wgrad(FP32, T, N, K, dy, x, dw, 0, s)
    assert close(dw, D.t() @ X, ad.t() @ ax, T)
    dw.copy_(dw0)
    tm.tm_op_linear_wgrad(FP32, T, N, K, dy, x, dw, 1, s)
    assert close(dw, D.t() @ X + dw0.double(), ad.t() @ ax + dw0.double().abs(), T)

    x[3] = float("inf")
    x[T - 1] *= 1e-35
    X = x.double()
    tm.tm_op_linear_fwd(FP32, T, N, K, x, w, None, None, y, s)
    assert not y[3].isfinite().any()
    ok = torch.arange(T, device="cuda") != 3
    assert close(y[ok], X[ok] @ W.t(), X[ok].abs() @ aw.t(), K)
    dy[5, 7] = float("nan")
    tm.tm_op_linear_dgrad(FP32, T, N, K, dy, w, dx, s)
    assert dx[5].isnan().all()
    ok = torch.arange(T, device="cuda") != 5
    assert close(dx[ok], D[ok] @ W, ad[ok] @ aw, N)


@pytest.mark.gpu
def test_elements_of_extreme_size(env):
    """Magnitudes whose leading bf16 is infinite or whose lower terms underflow, and results next to the largest number, beside
    their exact values."""
    torch, tm, s = env
    T, N, K = 1024, 1024, 1024
    assert split_tiles(T, N, K) == (64, 64, 64)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x, w = (torch.randn(1024, 1024, device="cuda", generator=g) for _ in range(2))
    y = torch.empty(T, N, device="cuda")
    for sx, sw in ((1e-37, 1e30), (1e30, 1e-37), (1e-39, 1e30), (1e36, 1e-3)):
        a, b = x * sx, w * sw
        tm.tm_op_linear_fwd(FP32, T, N, K, a, b, None, None, y, s)
        assert close(y, a.double() @ b.double().t(), a.double().abs() @ b.double().abs().t(), K), (sx, sw)
    a = x.clone()
    a[17, 31] = 3.4028e38                      # rounds to an infinite bf16
    b = w * 1e-3
    b[:, 31] = 1e-3
    tm.tm_op_linear_fwd(FP32, T, N, K, a, b, None, None, y, s)
    assert y.isfinite().all() and close(y, a.double() @ b.double().t(), a.double().abs() @ b.double().abs().t(), K)
