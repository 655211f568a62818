"""bf16 products of few 32x32 tiles over long reductions (csrc/gemm_mfma_small.hip): four waves split the reduction."""
import pytest

from tests.gpu_util import require_gpu, stream_ptr

pytestmark = pytest.mark.gpu
BF16 = 1


@pytest.fixture(scope="module")
def env():
    torch = require_gpu()
    import paper_2412_12636_amd as tm
    return torch, tm


@pytest.mark.parametrize("M,N,K", [
    (1, 8, 1024),            # one row, one chunk of columns; the shortest reduction
    (33, 40, 1032),          # a tile's second row and column of tiles nearly empty; 17 chunks, the last one of 8 elements
    (32, 64, 1088),          # whole tiles; the first wave has one chunk more than the others
    (500, 504, 2056),        # 256 tiles
    (500, 520, 2048),        # 272: forward still, the input gradient on the larger tiles
    (512, 1024, 1024),       # 512
    (513, 1024, 1024),       # 544: neither
    (7, 8200, 4104)])        # 257 columns of tiles
def test_products_of_few_tiles(env, M, N, K):
    """C[M,N] over K as a forward product, with and without bias and residual, and as an input gradient, between infinities and
    with one infinite row, against 64 bits: fp32 sums of K exact products (K 2^-24 of their magnitudes' sum) and one rounding to
    bf16 (2^-8); the same bits again; nothing written past the result."""
    torch, tm = env
    print(f"small products M={M} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K)
    s = stream_ptr(torch)

    def inside(*shape, std=1.0):
        n = 1
        for d in shape:
            n *= d
        buf = torch.full((n + 1024,), float("inf"), dtype=torch.bfloat16, device="cuda")
        view = buf[512:512 + n].view(shape)
        view.copy_(torch.randn(shape, device="cuda", generator=g) * std)
        return view

    a, w, wt, bias, res = inside(M, K), inside(N, K, std=0.05), inside(K, N, std=0.05), inside(N), inside(M, N)
    bad = M // 2
    keep = torch.arange(M, device="cuda") != bad
    A, mag = a.double(), a.double().abs()
    out = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device="cuda")

    def close(got, ref, size):
        return bool(((got.double() - ref).abs() <= K * 2.0 ** -24 * size + 2.0 ** -8 * ref.abs() + 1e-30).all())

    def check(run, ref, size):
        run(out)
        first = out.clone()
        run(out)
        assert torch.equal(first, out) and bool((out[M] == 7.0).all())
        assert close(out[:M], ref, size)

    fwd = lambda b, r: lambda o: tm.tm_op_linear_fwd(BF16, M, N, K, a, w, b, r, o, s)
    grad = lambda o: tm.tm_op_linear_dgrad(BF16, M, K, N, a, wt, o, s)
    W, WT = w.double(), wt.double()
    check(fwd(None, None), A @ W.t(), mag @ W.abs().t())
    check(fwd(bias, res), A @ W.t() + bias.double() + res.double(), mag @ W.abs().t() + bias.double().abs() + res.double().abs())
    check(grad, A @ WT, mag @ WT.abs())
    a[bad] = float("inf")
    for run, weight in ((fwd(None, None), W.t()), (grad, WT)):
        run(out)
        assert not out[bad].isfinite().any()
        assert close(out[:M][keep], (A @ weight)[keep], (mag @ weight.abs())[keep])
