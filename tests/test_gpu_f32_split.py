"""fp32 products on the bf16 matrix instructions (csrc/gemm_f32_split.hip): three bf16 terms an operand element."""
import pytest

from tests.f32_form import form, forms, split, splits

FP32 = 0


def test_where_the_terms_keep_out():
    """Short reductions, below 1024 elements those over more tiles than units, results of few tiles, a row of tiles that are nearly empty, and every form whose sums are split finer than
    these: the 16x16 tiles, the four-way 64x64 and the eight-way 32x32 ones."""
    for wgrad in (False, True):
        assert not split(2048, 2048, 255, wgrad) and split(2048, 2048, 256, wgrad)
        assert not split(256, 256, 8192, wgrad)
        assert not split(1024, 8192, 1016, wgrad) and split(1024, 8192, 1024, wgrad)
        assert not split(8, 1 << 26, 256, wgrad)
        kept = set()
        for M in range(96, 2400, 136):
            for N in range(96, 2400, 136):
                for K in (328, 1024, 4096):
                    if form(M, N, K, wgrad)[:2] in ((16, 4), (64, 4), (32, 8)):
                        kept.add(form(M, N, K, wgrad)[:2])
                        assert not split(M, N, K, wgrad)
        assert len(kept) == 2 + wgrad


@pytest.fixture(scope="module")
def env():
    from tests.gpu_util import require_gpu
    require_gpu()
    import torch

    import paper_2412_12636_amd as tm
    return torch, tm, int(torch.cuda.current_stream().cuda_stream)


def close(got, ref, size, n):
    """|got - ref| against the sums' roundings: one of half an ulp for every eight of n products, taken twice, and a few for the
    meeting of the accumulators and the epilogue, of at most the sum of the magnitudes `size`."""
    return bool(((got.double() - ref).abs() <= (0.125 * n + 8) * 2.0 ** -24 * size + 1e-44).all())


def off(got, ref):
    return ((got.double() - ref).norm() / ref.norm()).item()


@pytest.mark.gpu
@pytest.mark.parametrize("T,N,K,taken", [
    (3077, 776, 2056, (True, False, False)),   # odd token counts; 2056 = 64 stages of 32 and 8 elements
    (1100, 1928, 1992, (True, True, True)),    # edges inside a tile, a reduction that ends inside a stage
    (1536, 1544, 1544, (True, True, True)),    # one column of tiles nearly empty
    (1021, 3096, 1032, (True, False, True)),   # weight gradient over 1021 tokens
    (1601, 2312, 328, (True, False, False)),
    (2048, 2048, 256, (True, False, False)),   # the shortest reduction
])
def test_products_of_split_operands(env, T, N, K, taken):
    """Forward with and without bias and residual, input gradient, weight gradient stored and added, against 64 bits and the bound
    of the sums; then with an infinite and a tiny row in x and a NaN in dy: only what reads those is not finite, and the
    tiny row's results keep their precision."""
    torch, tm, s = env
    assert splits(T, N, K) == taken
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
    """Magnitudes whose leading bf16 is infinite at the terms' scale or would underflow without it, and results beyond the scaled
    sums or next to the largest number, beside their exact values."""
    torch, tm, s = env
    T, N, K = 2048, 2048, 2048
    assert splits(T, N, K)[0]
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x, w = (torch.randn(2048, 2048, device="cuda", generator=g) for _ in range(2))
    y = torch.empty(T, N, device="cuda")
    for sx, sw in ((1e-37, 1e30), (1e30, 1e-37), (1e-39, 1e30), (1e36, 1e-3), (1e13, 1e13)):
        a, b = x * sx, w * sw
        tm.tm_op_linear_fwd(FP32, T, N, K, a, b, None, None, y, s)
        assert close(y, a.double() @ b.double().t(), a.double().abs() @ b.double().abs().t(), K), (sx, sw)
    a = x.clone()
    a[17, 31] = 3.4028e38                      # rounds to an infinite bf16
    b = w * 1e-3
    b[:, 31] = 1e-3
    tm.tm_op_linear_fwd(FP32, T, N, K, a, b, None, None, y, s)
    assert y.isfinite().all() and close(y, a.double() @ b.double().t(), a.double().abs() @ b.double().abs().t(), K)


@pytest.mark.gpu
@pytest.mark.parametrize("T,N,K,taken", [(1100, 1928, 1992, (True, True, True)), (1601, 2312, 328, (True, False, False))])
def test_rows_keep_their_bits_beside_others(env, T, N, K, taken):
    """An infinity, a NaN and an element past the terms' scale in one row each, of either operand: every result that reads none of
    them has the bits that it had without; those that read the large element are the finite ones of the definition."""
    torch, tm, s = env
    assert splits(T, N, K) == taken
    print(f"rows beside others T={T} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    rnd = lambda *shape: torch.randn(shape, device="cuda", generator=g)

    def check(run, a, b):  # of a [M, K], b [N, K]
        for mine, other in ((a, b), (b, a)):
            first = run(a, b)
            rows = [1, mine.shape[0] // 2, mine.shape[0] - 1]
            was = mine[rows].clone()
            mine[rows[0], 5], mine[rows[1], 6], mine[rows[2], 7] = float("inf"), float("nan"), 1e33
            got = run(a, b)
            ref = a[rows[2]].double() @ b.double().t() if mine is a else a.double() @ b[rows[2]].double()
            size = other.double().abs() @ mine[rows[2]].double().abs()
            mine[rows] = was
            keep = torch.ones(mine.shape[0], dtype=torch.bool, device="cuda")
            keep[rows] = False
            if mine is b:
                first, got = first.t(), got.t()
            assert torch.equal(first[keep], got[keep])
            assert got[rows[1]].isnan().all() and not got[rows[0]].isfinite().any()
            assert close(got[rows[2]], ref, size, a.shape[1])

    def fwd(a, b):
        y = torch.empty(T, N, device="cuda")
        tm.tm_op_linear_fwd(FP32, T, N, K, a, b, None, None, y, s)
        return y

    def wgrad(a, b):
        dw = torch.empty(N, K, device="cuda")
        tm.tm_op_linear_wgrad(FP32, T, N, K, a.t().contiguous(), b.t().contiguous(), dw, 0, s)
        return dw

    def dgrad(a, b):
        dx = torch.empty(T, K, device="cuda")
        tm.tm_op_linear_dgrad(FP32, T, N, K, a, b.t().contiguous(), dx, s)
        return dx

    check(fwd, rnd(T, K), rnd(N, K))
    if taken[1]:
        check(dgrad, rnd(T, N), rnd(K, N))
    if taken[2]:
        check(wgrad, rnd(N, T), rnd(K, T))


@pytest.mark.gpu
@pytest.mark.parametrize("small", [1e-30, 1e-36, 1e-39])
def test_small_elements_beside_ordinary_ones(env, small):
    """Rows of one operand with an ordinary element that meets zeros: what the small ones, normal and subnormal numbers, sum up to
    has the precision that it has alone, in either operand and in the weight gradient."""
    torch, tm, s = env
    T, N, K = 2048, 2048, 2048
    assert splits(T, N, K) == (True, True, True)
    g = torch.Generator(device="cuda")
    g.manual_seed(9)
    rnd = lambda *shape: torch.randn(shape, device="cuda", generator=g)
    mixed, plain, out = rnd(2048, 2048) * small, rnd(2048, 2048), torch.empty(2048, 2048, device="cuda")
    mixed[:, 77], plain[:, 77] = rnd(2048), 0.0

    def right(a, b):  # (normal numbers: in the root mean square too, as test_no_less_precise_than_fused_multiply_adds)
        ref = a.double() @ b.double().t()
        return close(out, ref, a.double().abs() @ b.double().abs().t(), 2048) and (small < 1e-38 or off(out, ref) <= 3e-8 * 129 ** 0.5)

    for a, b in ((mixed, plain), (plain, mixed)):
        print(f"small elements of {small}, first operand {'mixed' if a is mixed else 'plain'}", flush=True)
        tm.tm_op_linear_fwd(FP32, T, N, K, a, b, None, None, out, s)
        assert right(a, b)
        a_t, b_t = a.t().contiguous(), b.t().contiguous()
        tm.tm_op_linear_dgrad(FP32, T, N, K, a, b_t, out, s)
        assert right(a, b)
        tm.tm_op_linear_wgrad(FP32, T, N, K, a_t, b_t, out, 0, s)
        assert right(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("T,N,K", [(2048, 2048, 256), (1100, 1928, 1992)])
def test_no_less_precise_than_fused_multiply_adds(env, T, N, K):
    """Rows with one element that is not zero: the product rounded once, 0.51 ulp (the second accumulator's roundings are 2^-8 of
    an ulp, the omitted product 2^-10); with a few: no further from 64 bits, in the root mean square, than a chain
    of fused multiply-adds, each of which rounds; full ones: an eighth of the products round, partial sums of n N(0,1) products
    grow like their root, an ulp's rounding is 2.4e-8 of a value, so 2.4e-8 sqrt(n / 16 + 1), here with a quarter to spare (one
    of the omitted 2^-16 products would be 1e-6)."""
    torch, tm, s = env
    assert split(T, N, K, False)
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    rnd = lambda *shape: torch.randn(shape, device="cuda", generator=g)
    w, y = rnd(N, K), torch.empty(T, N, device="cuda")
    for count in (1, 2, 4, 16, 64):
        at = torch.rand(T, K, device="cuda", generator=g).topk(count, 1).indices.sort(1).values
        values = rnd(T, count)
        x = torch.zeros(T, K, device="cuda").scatter_(1, at, values)
        tm.tm_op_linear_fwd(FP32, T, N, K, x, w, None, None, y, s)
        ref = x.double() @ w.double().t()
        if count == 1:
            ulp = torch.exp2(torch.floor(torch.log2(ref.abs())) - 23)
            assert bool(((y.double() - ref).abs() <= 0.51 * ulp).all())
            continue
        rows = slice(0, T, 16)
        chain = torch.zeros(len(range(0, T, 16)), N, device="cuda")
        for i in range(count):
            chain = (chain.double() + values[rows, i, None].double() * w[:, at[rows, i]].t().double()).float()
        print(f"{count} of {K}: {off(y, ref):.3e}, chain {off(chain, ref[rows]):.3e}", flush=True)
        assert off(y, ref) <= off(chain, ref[rows])
    x = rnd(T, K)
    tm.tm_op_linear_fwd(FP32, T, N, K, x, w, None, None, y, s)
    e = off(y, x.double() @ w.double().t())
    print(f"all of {K}: {e:.3e}", flush=True)
    assert e <= 3e-8 * (K / 16 + 1) ** 0.5


@pytest.mark.gpu
@pytest.mark.parametrize("T,N,K,which", [(2048, 2048, 256, "128/1"), (3077, 776, 2056, "64/1"), (870, 2376, 1000, "32/4p")])
def test_results_off_the_16_byte_grid(env, T, N, K, which):
    """Products that the terms would have, results, bias and residual one element off 16 bytes: the fp32 instructions form them, to
    n 2^-24 of the sum of the magnitudes, between guards that stay."""
    torch, tm, s = env
    assert split(T, N, K, False) and forms(T, N, K).split()[0] == which
    print(f"results off the grid T={T} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    rnd = lambda *shape: torch.randn(shape, device="cuda", generator=g)
    x, w = rnd(T, K), rnd(N, K)
    bias, res = rnd(N + 1)[1:], rnd(T * N + 1)[1:].view(T, N)
    buf = torch.full((T * N + 8,), 7.0, device="cuda")
    aligned = torch.empty(T, N, device="cuda")
    X, W = x.double(), w.double()
    for b, r, y in ((None, None, buf[1:1 + T * N].view(T, N)), (bias, None, aligned), (None, res, aligned)):
        tm.tm_op_linear_fwd(FP32, T, N, K, x, w, b, r, y, s)
        ref, size = X @ W.t(), X.abs() @ W.abs().t()
        for extra in (b, r):
            if extra is not None:
                ref, size = ref + extra.double(), size + extra.double().abs()
        assert bool(((y.double() - ref).abs() <= (K + 8) * 2.0 ** -24 * size).all())
    assert bool((buf[:1] == 7.0).all()) and bool((buf[1 + T * N:] == 7.0).all())
