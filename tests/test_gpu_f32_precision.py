"""What the fp32 products keep on rows that are not dense N(0,1) data: few elements that are not zero, small elements beside large
ones, values that are not finite, extreme magnitudes, and results off 16 bytes; on every tile form that large products take."""
import pytest

from tests.f32_form import forms
from tests.gpu_util import require_gpu, stream_ptr

pytestmark = pytest.mark.gpu
FP32 = 0


@pytest.fixture(scope="module")
def env():
    torch = require_gpu()
    import paper_2412_12636_amd as tm
    return torch, tm, stream_ptr(torch)


def normal(torch, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return lambda *shape: torch.randn(shape, device="cuda", generator=g)


def close(got, ref, size, n):
    """|got - ref| against an fp32 sum of n exact products: half an ulp of at most the sum of the magnitudes `size` for each, and
    a few more for split waves and the epilogue; 1e-44 for results that are subnormal numbers."""
    return bool(((got.double() - ref).abs() <= (n + 8) * 2.0 ** -24 * size + 1e-44).all())


def off(got, ref):
    return ((got.double() - ref).norm() / ref.norm()).item()


def product(torch, tm, s, kind, a, b):
    """a [M, K] b [N, K]^T as a forward product, an input gradient or a weight gradient."""
    (M, K), N = a.shape, b.shape[0]
    out = torch.full((M + 1, N), 7.0, device="cuda")
    if kind == "forward":
        tm.tm_op_linear_fwd(FP32, M, N, K, a, b, None, None, out, s)
    elif kind == "input gradient":
        tm.tm_op_linear_dgrad(FP32, M, K, N, a, b.t().contiguous(), out, s)
    else:
        tm.tm_op_linear_wgrad(FP32, K, M, N, a.t().contiguous(), b.t().contiguous(), out, 0, s)
    assert bool((out[M] == 7.0).all())
    return out[:M]


KINDS = {"forward": 0, "input gradient": 1, "weight gradient": 2}
SIZES = [(2048, 2048, 256, "128/1"), (3077, 776, 2056, "64/1"), (1000, 1000, 1000, "64/4"), (870, 2376, 1000, "32/4p")]


@pytest.mark.parametrize("M,N,K,which", SIZES)
def test_no_less_precise_than_fused_multiply_adds(env, M, N, K, which):
    """Rows with one element that is not zero: its product rounded once, half an ulp.  With a few: no further from 64 bits, in the
    root mean square, than a chain of fused multiply-adds, each of which rounds (5 % for the sample of rows).  Waves that split
    the reduction round their products before these meet: of two, four squares in place of three, 1.155, of four at most 13
    in place of 10, of more less.  Full ones: at most as many roundings, partial sums that grow like a root and roundings of
    2.4e-8 of them: 2.4e-8 sqrt(K / 2 + 1), with a quarter to spare."""
    torch, tm, s = env
    assert forms(M, N, K).split()[0] == which
    rnd = normal(torch, K)
    w = rnd(N, K)
    for count in (1, 2, 4, 16, 64):
        at = torch.rand(M, K, device="cuda").topk(count, 1).indices.sort(1).values
        values = rnd(M, count)
        x = torch.zeros(M, K, device="cuda").scatter_(1, at, values)
        y, ref = product(torch, tm, s, "forward", x, w), x.double() @ w.double().t()
        if count == 1:
            ulp = torch.exp2(torch.floor(torch.log2(ref.abs())) - 23)
            assert bool(((y.double() - ref).abs() <= 0.5 * ulp).all())
            continue
        rows = slice(0, M, 16)
        chain = torch.zeros(len(range(0, M, 16)), N, device="cuda")
        for i in range(count):
            chain = (chain.double() + values[rows, i, None].double() * w[:, at[rows, i]].t().double()).float()
        print(f"{count} of {K}: {off(y, ref):.3e}, chain {off(chain, ref[rows]):.3e}", flush=True)
        assert off(y, ref) <= 1.05 * (1.0 if which.split("/")[1] == "1" else 1.155) * off(chain, ref[rows])
    x = rnd(M, K)
    e = off(product(torch, tm, s, "forward", x, w), x.double() @ w.double().t())
    print(f"all of {K}: {e:.3e}", flush=True)
    assert e <= 3e-8 * (K / 2 + 1) ** 0.5


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("small", [1e-30, 1e-36, 1e-39])
def test_small_elements_beside_ordinary_ones(env, kind, small):
    """Rows of one operand with an ordinary element that meets zeros: what the small ones, normal and subnormal numbers, sum up to
    has the precision that it has alone."""
    torch, tm, s = env
    M = N = K = 2048
    rnd = normal(torch, 9)
    mixed, plain = rnd(M, K) * small, rnd(N, K)
    mixed[:, 77], plain[:, 77] = rnd(M), 0.0
    for a, b in ((mixed, plain), (plain, mixed)):
        print(f"{kind}: small elements of {small}, first operand {'mixed' if a is mixed else 'plain'}", flush=True)
        got, ref = product(torch, tm, s, kind, a, b), a.double() @ b.double().t()
        assert close(got, ref, a.double().abs() @ b.double().abs().t(), K)
        assert small < 1e-38 or off(got, ref) <= 3e-8 * (K / 2 + 1) ** 0.5


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("M,N,K", [s[:3] for s in SIZES])
def test_rows_keep_their_bits_beside_others(env, kind, M, N, K):
    """An infinity, a NaN and an element of 1e33 in one row each, of either operand: every result that reads none of them has the
    bits that it had without, and those that read the large element are the definition's."""
    torch, tm, s = env
    if kind != "forward":
        M, N, K = (M // 8 * 8, N, K // 8 * 8)
    print(f"{kind}: rows beside others M={M} N={N} K={K}", flush=True)
    rnd = normal(torch, M)
    a, b = rnd(M, K), rnd(N, K)
    first = product(torch, tm, s, kind, a, b)
    for mine, other in ((a, b), (b, a)):
        rows = [1, mine.shape[0] // 2, mine.shape[0] - 1]
        was = mine[rows].clone()
        mine[rows[0], 5], mine[rows[1], 6], mine[rows[2], 7] = float("inf"), float("nan"), 1e33
        got, large = product(torch, tm, s, kind, a, b), mine[rows[2]].double()
        mine[rows] = was
        want, got = (first, got) if mine is a else (first.t(), got.t())
        keep = torch.ones(mine.shape[0], dtype=torch.bool, device="cuda")
        keep[rows] = False
        assert torch.equal(want[keep], got[keep])
        assert got[rows[1]].isnan().all() and not got[rows[0]].isfinite().any()
        assert close(got[rows[2]], other.double() @ large, other.double().abs() @ large.abs(), K)


def test_elements_of_extreme_size(env):
    """Magnitudes at both ends of the range, subnormal ones too, beside their exact products' sums."""
    torch, tm, s = env
    rnd = normal(torch, 3)
    x, w = rnd(2048, 2048), rnd(2048, 2048)
    for sx, sw in ((1e-37, 1e30), (1e30, 1e-37), (1e-39, 1e30), (1e36, 1e-3), (1e13, 1e13)):
        a, b = x * sx, w * sw
        assert close(product(torch, tm, s, "forward", a, b), a.double() @ b.double().t(), a.double().abs() @ b.double().abs().t(), 2048), (sx, sw)
    a, b = x.clone(), w * 1e-3
    a[17, 31], b[:, 31] = 3.4028e38, 1e-3
    y = product(torch, tm, s, "forward", a, b)
    assert y.isfinite().all() and close(y, a.double() @ b.double().t(), a.double().abs() @ b.double().abs().t(), 2048)


@pytest.mark.parametrize("M,N,K,which", SIZES)
def test_results_off_the_16_byte_grid(env, M, N, K, which):
    """Results, bias and residual one element off 16 bytes, between guards that stay: the same bits as on the grid."""
    torch, tm, s = env
    assert forms(M, N, K).split()[0] == which
    print(f"results off the grid M={M} N={N} K={K}", flush=True)
    rnd = normal(torch, M)
    x, w, bias, res = rnd(M, K), rnd(N, K), rnd(N), rnd(M, N)
    want = torch.empty(M, N, device="cuda")
    tm.tm_op_linear_fwd(FP32, M, N, K, x, w, bias, res, want, s)
    buf = torch.full((M * N + 8,), 7.0, device="cuda")
    moved = lambda t: torch.cat([t.new_zeros(1), t.reshape(-1)])[1:].view(t.shape)
    got = buf[1:1 + M * N].view(M, N)
    tm.tm_op_linear_fwd(FP32, M, N, K, x, w, moved(bias), moved(res), got, s)
    assert torch.equal(got, want)
    assert bool((buf[:1] == 7.0).all()) and bool((buf[1 + M * N:] == 7.0).all())
