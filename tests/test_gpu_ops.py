"""GPU parity of every step of the hot path against the fp64 CPU checker, element by element,
through the C ABI.  Small shapes that still span several tiles and ragged tails, plus the
degenerate cases (one token, one position, one head)."""
import math

import numpy as np
import pytest

import synth_inputs as si
from oracle import stage_oracle as so
from tests.f32_form import forms, splits
from tests.gpu_util import (TOL_ADAM, TOL_BF16, TOL_FP32, f32_dev, rand, rel_err, require_gpu, stream_ptr, to_dev,
                            to_host, torch_dtype)

pytestmark = pytest.mark.gpu

BF16, FP32 = si.DTYPE_BF16, si.DTYPE_FP32


def tol_of(dtype):
    return TOL_BF16 if dtype == BF16 else TOL_FP32


@pytest.fixture(scope="module")
def env():
    torch = require_gpu()
    import paper_2412_12636_amd as tm
    return torch, tm


# ------------------------------------------------------------------ linear maps
LINEAR_SHAPES = [
    (BF16, 300, 264, 200),     # ragged in every dimension, several 128-tiles
    (BF16, 512, 512, 256),     # exact 256-tiles
    (BF16, 1, 8, 8),           # one token
    (BF16, 1000, 136, 72),     # tall, K tail of 8
    (FP32, 70, 72, 40),
    (FP32, 256, 256, 64),
]


@pytest.mark.parametrize("dtype,T,N,K", LINEAR_SHAPES)
def test_linear_fwd_dgrad_wgrad(env, dtype, T, N, K):
    torch, tm = env
    print(f"linear dtype={dtype} T={T} N={N} K={K}", flush=True)
    rng = np.random.default_rng(T * 7 + N)
    x, w = rand(rng, (T, K), 1.0, dtype), rand(rng, (N, K), 0.05, dtype)
    bias, res = rand(rng, (N,), 0.5, dtype), rand(rng, (T, N), 1.0, dtype)
    dy = rand(rng, (T, N), 0.1, dtype)
    td = torch_dtype(torch, dtype)
    xd, wd, bd, rd, dyd = (to_dev(torch, a, dtype) for a in (x, w, bias, res, dy))
    s = stream_ptr(torch)
    tol = tol_of(dtype)

    y = torch.empty((T, N), dtype=td, device="cuda")
    tm.tm_op_linear_fwd(dtype, T, N, K, xd, wd, bd, rd, y, s)
    ref = x.astype(np.float64) @ w.astype(np.float64).T + bias + res
    assert rel_err(to_host(y), ref) <= tol
    y2 = torch.empty((T, N), dtype=td, device="cuda")
    tm.tm_op_linear_fwd(dtype, T, N, K, xd, wd, None, None, y2, s)
    assert rel_err(to_host(y2), x.astype(np.float64) @ w.astype(np.float64).T) <= tol

    dx = torch.empty((T, K), dtype=td, device="cuda")
    tm.tm_op_linear_dgrad(dtype, T, N, K, dyd, wd, dx, s)
    assert rel_err(to_host(dx), dy.astype(np.float64) @ w.astype(np.float64)) <= tol

    g0 = rng.standard_normal((N, K)).astype(np.float32)
    dw = f32_dev(torch, g0)
    tm.tm_op_linear_wgrad(dtype, T, N, K, dyd, xd, dw, 1, s)
    ref = g0.astype(np.float64) + dy.astype(np.float64).T @ x.astype(np.float64)
    # fp32 accumulation of exact products: far tighter than the storage tolerance
    assert rel_err(to_host(dw), ref) <= 1e-5


def test_every_tile_configuration_gives_the_same_bits_and_matches_the_checker(env):
    """Each tile configuration in turn is forced on the three products of a linear map (ragged edges, several tiles of
    the largest shape, all dimensions multiples of 64 so that the pipelined kernel runs): results equal the checker's
    within tolerance and equal the first configuration's bit for bit."""
    torch, tm = env
    T, N, K = 712, 584, 448
    rng = np.random.default_rng(11)
    x, w = rand(rng, (T, K), 1.0, BF16), rand(rng, (N, K), 0.05, BF16)
    bias, res, dy = rand(rng, (N,), 0.5, BF16), rand(rng, (T, N), 1.0, BF16), rand(rng, (T, N), 0.1, BF16)
    xd, wd, bd, rd, dyd = (to_dev(torch, a, BF16) for a in (x, w, bias, res, dy))
    dy64 = dy.astype(np.float64)
    s = stream_ptr(torch)
    ref_y = x.astype(np.float64) @ w.astype(np.float64).T + bias + res
    first = None
    n = tm.tm_gemm_config_count()
    assert n >= 13
    try:
        for c in range(n):
            print(f"tile configuration {c}", flush=True)
            tm.tm_gemm_force_config(c)
            y = torch.empty((T, N), dtype=torch.bfloat16, device="cuda")
            dx = torch.empty((T, K), dtype=torch.bfloat16, device="cuda")
            dw = torch.empty((N, K), dtype=torch.float32, device="cuda")
            tm.tm_op_linear_fwd(BF16, T, N, K, xd, wd, bd, rd, y, s)
            tm.tm_op_linear_dgrad(BF16, T, N, K, dyd, wd, dx, s)
            tm.tm_op_linear_wgrad(BF16, T, N, K, dyd, xd, dw, 0, s)
            tm.tm_op_linear_wgrad(BF16, T, N, K, dyd, xd, dw, 1, s)      # adds the same product again
            torch.cuda.synchronize()
            assert rel_err(to_host(y), ref_y) <= TOL_BF16
            assert rel_err(to_host(dx), dy64 @ w.astype(np.float64)) <= TOL_BF16
            assert rel_err(to_host(dw), 2.0 * (dy64.T @ x.astype(np.float64))) <= 1e-5
            if first is None:
                first = (y, dx, dw)
            else:
                assert torch.equal(y, first[0]) and torch.equal(dx, first[1]) and torch.equal(dw, first[2]), c
    finally:
        tm.tm_gemm_force_config(-1)
    with pytest.raises(tm.TmError):
        tm.tm_gemm_force_config(n)


@pytest.mark.parametrize("T,N,K", [(8, 8, 8), (257, 264, 72), (130, 200, 56), (384, 136, 1016), (200, 392, 328)])
def test_reduction_lengths_off_the_step_in_every_configuration(env, T, N, K):
    """Reduction lengths that are no multiple of 64 (one short step; one step and 8; 56, 48, 8 left over) in every tile
    configuration.  The operands sit between stretches of infinities and one row of x is infinite: an element from
    past a row's end would show as NaN.  bf16 results are off by their rounding (2^-9) beside
    fp32 sums, fp32 results by the sums alone."""
    torch, tm = env
    print(f"linear ragged T={T} N={N} K={K}", flush=True)
    rng = np.random.default_rng(T + N + K)
    x, w, dy = rand(rng, (T, K), 1.0, BF16), rand(rng, (N, K), 0.05, BF16), rand(rng, (T, N), 0.1, BF16)

    def inside(a):                                       # the matrix between two stretches of infinities
        buf = torch.full((a.size + 1024,), float("inf"), dtype=torch.bfloat16, device="cuda")
        view = buf[512:512 + a.size].view(a.shape)
        view.copy_(to_dev(torch, a, BF16))
        return view

    xd, wd, dyd = inside(x), inside(w), inside(dy)
    bad = T // 2                                         # one row of infinities: its neighbours stay finite
    xbad = xd.clone()
    xbad[bad] = float("inf")
    x64, w64, dy64 = (a.astype(np.float64) for a in (x, w, dy))
    s = stream_ptr(torch)
    try:
        for c in range(tm.tm_gemm_config_count()):
            print(f"tile configuration {c}", flush=True)
            tm.tm_gemm_force_config(c)
            y, yb = (torch.empty((T, N), dtype=torch.bfloat16, device="cuda") for _ in range(2))
            dx = torch.empty((T, K), dtype=torch.bfloat16, device="cuda")
            dw = torch.zeros((N, K), dtype=torch.float32, device="cuda")
            tm.tm_op_linear_fwd(BF16, T, N, K, xd, wd, None, None, y, s)
            tm.tm_op_linear_fwd(BF16, T, N, K, xbad, wd, None, None, yb, s)
            tm.tm_op_linear_dgrad(BF16, T, N, K, dyd, wd, dx, s)
            tm.tm_op_linear_wgrad(BF16, T, N, K, dyd, xd, dw, 1, s)
            assert rel_err(to_host(y), x64 @ w64.T) <= 2.0 ** -8
            assert rel_err(to_host(dx), dy64 @ w64) <= 2.0 ** -8
            assert rel_err(to_host(dw), dy64.T @ x64) <= 1e-5
            rows = np.arange(T) != bad
            assert np.array_equal(to_host(yb)[rows], to_host(y)[rows])
    finally:
        tm.tm_gemm_force_config(-1)


@pytest.mark.parametrize("T,N,K", [(1, 8, 8), (33, 40, 72), (257, 136, 200), (300, 1096, 520), (2050, 2056, 40), (2048, 2040, 72), (2040, 136, 2040),
                                   (136, 2040, 2040)],
                         ids=["one_row", "tiles_of_16", "tiles_of_16_ragged", "tiles_of_32_and_64", "tiles_of_64_ragged", "tiles_of_128", "tiles_of_128_dgrad",
                              "tiles_of_128_wgrad"])
def test_linear_fp32_tiles(env, T, N, K):
    """The fp32 products in each of their tile forms, ragged in every dimension, against the definition (fp32 sums of
    at most 2056 terms: 1e-5), with one infinite row of x: its neighbours stay as they are."""
    torch, tm = env
    print(f"linear fp32 T={T} N={N} K={K}", flush=True)
    rng = np.random.default_rng(T + N + K)
    x, w, dy = rand(rng, (T, K), 1.0, FP32), rand(rng, (N, K), 0.05, FP32), rand(rng, (T, N), 0.1, FP32)
    bias, res, g0 = rand(rng, (N,), 0.5, FP32), rand(rng, (T, N), 1.0, FP32), rand(rng, (N, K), 1.0, FP32)
    xd, wd, dyd, bd, rd = (to_dev(torch, a, FP32) for a in (x, w, dy, bias, res))
    s = stream_ptr(torch)
    y, yb, dx = (torch.full((T + 1, n), 7.0, device="cuda") for n in (N, N, K))
    dw0, dw1 = torch.full((N + 1, K), 7.0, device="cuda"), torch.full((N + 1, K), 7.0, device="cuda")
    dw1[:N].copy_(to_dev(torch, g0, FP32))
    tm.tm_op_linear_fwd(FP32, T, N, K, xd, wd, bd, rd, y, s)
    tm.tm_op_linear_dgrad(FP32, T, N, K, dyd, wd, dx, s)
    tm.tm_op_linear_wgrad(FP32, T, N, K, dyd, xd, dw0, 0, s)
    tm.tm_op_linear_wgrad(FP32, T, N, K, dyd, xd, dw1, 1, s)
    x64, w64, dy64 = (a.astype(np.float64) for a in (x, w, dy))
    assert rel_err(to_host(y[:T]), x64 @ w64.T + bias + res) <= 1e-5
    assert rel_err(to_host(dx[:T]), dy64 @ w64) <= 1e-5
    assert rel_err(to_host(dw0[:N]), dy64.T @ x64) <= 1e-5
    assert rel_err(to_host(dw1[:N]), g0 + dy64.T @ x64) <= 1e-5
    for t, n in ((y, T), (dx, T), (dw0, N), (dw1, N)):
        assert bool((t[n:] == 7.0).all())
    xd[T // 2] = float("inf")
    tm.tm_op_linear_fwd(FP32, T, N, K, xd, wd, bd, rd, yb, s)
    rows = np.arange(T) != T // 2
    assert np.array_equal(yb[:T].cpu().numpy()[rows], y[:T].cpu().numpy()[rows])


@pytest.mark.parametrize("T,N,K,which", [
    (16, 16, 128, "16/4 16/4 16/4"), (17, 24, 136, "16/4 16/4 16/4"), (40, 136, 264, "16/4 16/4 16/4"), (64, 2048, 72, "16/4 16/4 32/4"),
    (250, 248, 1000, "16/4 32/4 32/4"), (330, 296, 1032, "16/4 32/4 32/8"), (90, 1048, 1080, "16/4p 16/4p 32/4"), (1090, 1032, 136, "32/4 32/4 32/8"),
    (577, 520, 1032, "32/4 32/4 32/8"), (1000, 1032, 328, "32/4 32/4 32/8"), (777, 776, 1032, "32/4p 64/4 64/4"), (1001, 776, 904, "64/4 64/4 32/8p"),
    (1001, 1000, 776, "64/4 64/4 64/4"), (1028, 840, 1032, "64/4 32/4p 64/4"),
    (520, 328, 1032, "32/4 64/1 32/8"), (1100, 1504, 1032, "64/1 32/4p 64/1")], ids=str)
def test_linear_fp32_split_waves(env, T, N, K, which):
    """The fp32 products whose waves split a stage's reduction elements (16x16, 32x32 and 64x64 tiles), at the ends of tiles
    and stages, in plain order and in patches; which: the forms of the three products (tile / split, p: patches), so that
    a change of the rule shows here.  An fp32 sum of n products is off by at most n 2^-24 of the sum of their
    magnitudes and by about sqrt(n) 2^-24 for these signs, 2e-6 at 1100 terms; stored and added to."""
    assert forms(T, N, K) == which and not any(splits(T, N, K))
    torch, tm = env
    print(f"linear fp32 split waves T={T} N={N} K={K}", flush=True)
    rng = np.random.default_rng(T + N + K)
    x, w, dy = rand(rng, (T, K), 1.0, FP32), rand(rng, (N, K), 0.05, FP32), rand(rng, (T, N), 0.1, FP32)
    bias, res, g0 = rand(rng, (N,), 0.5, FP32), rand(rng, (T, N), 1.0, FP32), rand(rng, (N, K), 1.0, FP32)
    xd, wd, dyd, bd, rd = (to_dev(torch, a, FP32) for a in (x, w, dy, bias, res))
    s = stream_ptr(torch)
    y, dx, dw0 = (torch.full((r + 1, c), 7.0, device="cuda") for r, c in ((T, N), (T, K), (N, K)))  # one row more: stays as it is
    dw1 = torch.full((N + 1, K), 7.0, device="cuda")
    dw1[:N].copy_(to_dev(torch, g0, FP32))
    tm.tm_op_linear_fwd(FP32, T, N, K, xd, wd, bd, rd, y, s)
    tm.tm_op_linear_dgrad(FP32, T, N, K, dyd, wd, dx, s)
    tm.tm_op_linear_wgrad(FP32, T, N, K, dyd, xd, dw0, 0, s)
    tm.tm_op_linear_wgrad(FP32, T, N, K, dyd, xd, dw1, 1, s)
    x64, w64, dy64 = (a.astype(np.float64) for a in (x, w, dy))
    for got, ref, n in ((y, x64 @ w64.T + bias + res, T), (dx, dy64 @ w64, T), (dw0, dy64.T @ x64, N), (dw1, g0 + dy64.T @ x64, N)):
        assert rel_err(to_host(got[:n]), ref) <= 2e-6
        assert bool((got[n:] == 7.0).all())


@pytest.mark.parametrize("T", [24, 32, 33, 136, 480, 488, 704, 712, 1024, 1032, 1400, 1416])
@pytest.mark.parametrize("N,K", [(1032, 2056), (2064, 1048), (2056, 4104), (4128, 2056), (2040, 4104)])
def test_weight_gradients_of_rows_off_the_lines(env, T, N, K):
    """Weight gradients whose rows start inside 128-byte lines, below and above the 2^23 results and around the token counts
    at which the choice of tiles changes, stored and added to, against exact products' sums (fp32, at most 1416 terms: 1e-5) and, behind the last
    row, nothing."""
    torch, tm = env
    print(f"weight gradient off the lines T={T} N={N} K={K}", flush=True)
    rng = np.random.default_rng(T + N)
    x, dy, g0 = rand(rng, (T, K), 1.0, BF16), rand(rng, (T, N), 0.1, BF16), rand(rng, (N, K), 1.0, FP32)
    xd, dyd = to_dev(torch, x, BF16), to_dev(torch, dy, BF16)
    dw0, dw1 = (torch.full((N + 1, K), 7.0, device="cuda") for _ in range(2))
    dw1[:N].copy_(to_dev(torch, g0, FP32))
    for dw, acc in ((dw0, 0), (dw1, 1)):
        tm.tm_op_linear_wgrad(BF16, T, N, K, dyd, xd, dw, acc, stream_ptr(torch))
    ref = (dyd.double().t().contiguous() @ xd.double()).cpu().numpy()
    assert rel_err(to_host(dw0[:N]), ref) <= 1e-5
    assert rel_err(to_host(dw1[:N]), g0 + ref) <= 1e-5
    assert bool((dw0[N:] == 7.0).all()) and bool((dw1[N:] == 7.0).all())


def split_gradient(env, T, N, K, seed, splits):
    """dx = dy W with scratch: whether the reduction was split shows in the scratch, which is filled before; the result meets
    the tolerance against the definition, is reproducible and independent of what the scratch held; without scratch the call
    is the plain product."""
    torch, tm = env
    print(f"input gradient T={T} N={N} K={K}", flush=True)
    rng = np.random.default_rng(seed)
    dy, w = rand(rng, (T, N), 0.1, BF16), rand(rng, (N, K), 0.05, BF16)
    dyd, wd = to_dev(torch, dy, BF16), to_dev(torch, w, BF16)
    s = stream_ptr(torch)
    need = tm.tm_op_linear_dgrad_scratch_bytes(BF16, T, N, K)
    assert need == 8 * T * K * 4                 # eight parts
    scratch = torch.full((need // 4,), -1.5e30, dtype=torch.float32, device="cuda")
    new = lambda: torch.full((T, K), float("nan"), dtype=torch.bfloat16, device="cuda")
    a, b, c, d = new(), new(), new(), new()
    tm.tm_op_linear_dgrad_ws(BF16, T, N, K, dyd, wd, a, scratch, need, s)
    untouched = int((scratch == -1.5e30).sum())
    assert untouched == (0 if splits else scratch.numel())
    scratch.fill_(float("nan"))                  # stale partial results must not matter
    tm.tm_op_linear_dgrad_ws(BF16, T, N, K, dyd, wd, b, scratch, need, s)
    tm.tm_op_linear_dgrad_ws(BF16, T, N, K, dyd, wd, c, None, 0, s)
    tm.tm_op_linear_dgrad(BF16, T, N, K, dyd, wd, d, s)
    torch.cuda.synchronize()
    ref = dy.astype(np.float64) @ w.astype(np.float64)
    assert rel_err(to_host(a), ref) <= TOL_BF16 and rel_err(to_host(d), ref) <= TOL_BF16
    assert torch.equal(a, b) and torch.equal(c, d)
    if not splits:
        assert torch.equal(a, d)


@pytest.mark.parametrize("T,N,K,splits", [(200, 16384, 264, True), (3, 8192, 248, True), (300, 4096, 264, False)])
def test_input_gradient_with_split_reduction(env, T, N, K, splits):
    """Few output tiles and a long reduction: eight parts on 128 x 192 tiles, ragged in both output dimensions; and an output
    that is small enough for it whose reduction is too short for the split to pay."""
    split_gradient(env, T, N, K, 21, splits)
    assert env[1].tm_op_linear_dgrad_scratch_bytes(BF16, 2048, 4608, 12288) == 0   # enough tiles: no split


@pytest.mark.parametrize("T,N,K,splits", [(1000, 16384, 1496, True), (1000, 4096, 1096, False)])
def test_input_gradient_with_split_reduction_on_large_tiles(env, T, N, K, splits):
    """Same, at shapes whose parts fill the chip with 256 x 192 tiles (the kernel with loader waves writes the fp32
    partial results): ragged in both output dimensions, eight parts."""
    split_gradient(env, T, N, K, 22, splits)


def test_gradient_overwrite_mode_ignores_old_contents(env):
    torch, tm = env
    rng = np.random.default_rng(4)
    T, N, K = 300, 264, 192
    x, dy = rand(rng, (T, K), 1.0, BF16), rand(rng, (T, N), 0.1, BF16)
    xd, dyd = to_dev(torch, x, BF16), to_dev(torch, dy, BF16)
    s = stream_ptr(torch)
    dw = torch.full((N, K), float("nan"), dtype=torch.float32, device="cuda")
    tm.tm_op_linear_wgrad(BF16, T, N, K, dyd, xd, dw, 0, s)
    assert rel_err(to_host(dw), dy.astype(np.float64).T @ x.astype(np.float64)) <= 1e-5
    db = torch.full((N,), float("nan"), dtype=torch.float32, device="cuda")
    scratch = torch.empty(tm.tm_op_reduce_scratch_bytes(T, 2 * N), dtype=torch.uint8, device="cuda")
    tm.tm_op_bias_grad(BF16, T, N, dyd, db, scratch, 0, s)
    assert rel_err(to_host(db), dy.astype(np.float64).sum(axis=0)) <= 1e-5
    # the fp32 stage dtype's own kernel
    dwf = torch.full((N, K), float("nan"), dtype=torch.float32, device="cuda")
    tm.tm_op_linear_wgrad(FP32, T, N, K, dyd.float(), xd.float(), dwf, 0, s)
    assert rel_err(to_host(dwf), dy.astype(np.float64).T @ x.astype(np.float64)) <= 1e-5


@pytest.mark.parametrize("dtype", [BF16, FP32])
def test_linear_off_the_alignment(env, dtype):
    """Operands that start one element past a 16-byte boundary go to the plain-ALU kernel, ragged in every dimension: the three
    products, with bias and residual and with both gradient modes, against the definition (fp32 sums of at most 200
    terms: 1e-6; bf16 results their rounding, 2^-8)."""
    torch, tm = env
    T, N, K = 130, 72, 200
    print(f"linear off the alignment dtype={dtype}", flush=True)
    rng = np.random.default_rng(17)
    x, w, dy = rand(rng, (T, K), 1.0, dtype), rand(rng, (N, K), 0.05, dtype), rand(rng, (T, N), 0.1, dtype)
    bias, res, g0 = rand(rng, (N,), 0.5, dtype), rand(rng, (T, N), 1.0, dtype), rng.standard_normal((N, K)).astype(np.float32)

    def off(a):
        t = to_dev(torch, a, dtype)
        view = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:].view(t.shape)
        view.copy_(t)
        return view

    xd, wd, dyd, bd, rd = off(x), off(w), off(dy), off(bias), off(res)
    y, dx = torch.empty_like(dyd), torch.empty_like(xd)
    dw0, dw1 = torch.full((N, K), float("nan"), device="cuda"), f32_dev(torch, g0)
    s = stream_ptr(torch)
    tm.tm_op_linear_fwd(dtype, T, N, K, xd, wd, bd, rd, y, s)
    tm.tm_op_linear_dgrad(dtype, T, N, K, dyd, wd, dx, s)
    tm.tm_op_linear_wgrad(dtype, T, N, K, dyd, xd, dw0, 0, s)
    tm.tm_op_linear_wgrad(dtype, T, N, K, dyd, xd, dw1, 1, s)
    x64, w64, dy64 = (a.astype(np.float64) for a in (x, w, dy))
    bound = 2.0 ** -8 if dtype == BF16 else 1e-6
    assert rel_err(to_host(y), x64 @ w64.T + bias + res) <= bound
    assert rel_err(to_host(dx), dy64 @ w64) <= bound
    assert rel_err(to_host(dw0), dy64.T @ x64) <= 1e-6
    assert rel_err(to_host(dw1), g0 + dy64.T @ x64) <= 1e-6


@pytest.mark.parametrize("config", [-1, 3], ids=["chosen_tiles", "large_tiles"])
def test_results_of_very_wide_rows(env, config):
    """Rows of 2^25 results: a tile's rows past the eighth and last lie 2^32 bytes further on from row 32 (fp32) or 64 (bf16)
    and must not be written to the front.  All three products, from the definition on columns at the front, in the
    middle and at the end (eight exact products each: bf16 rounding 2^-8, fp32 1e-6)."""
    torch, tm = env
    wide, n = 1 << 25, 8
    print(f"very wide rows config={config}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(8)
    small = torch.randn((n, n), generator=g, device="cuda").bfloat16()
    big = torch.randn((n, wide), generator=g, device="cuda").bfloat16()
    s = stream_ptr(torch)
    dw = torch.full((n, wide), float("nan"), device="cuda")
    dx, y = torch.empty_like(big), torch.empty_like(big)
    tall = big.t().contiguous()
    try:
        tm.tm_gemm_force_config(config)
        tm.tm_op_linear_wgrad(BF16, n, n, wide, small, big, dw, 0, s)
        tm.tm_op_linear_dgrad(BF16, n, n, wide, small, big, dx, s)
        tm.tm_op_linear_fwd(BF16, n, wide, n, small, tall, None, None, y, s)
    finally:
        tm.tm_gemm_force_config(-1)
    for first in (0, wide // 2 - 100, wide - 1000):
        cols = slice(first, first + 1000)
        a, b = to_host(small), to_host(big[:, cols])
        assert rel_err(to_host(dw[:, cols]), a.T @ b) <= 1e-6
        assert rel_err(to_host(dx[:, cols]), a @ b) <= 2.0 ** -8
        assert rel_err(to_host(y[:, cols]), a @ b) <= 2.0 ** -8


@pytest.mark.parametrize("T,N,K", [(48, 8192, 4096), (64, 8192, 4104), (1, 4096, 8200)])
def test_weight_gradient_of_one_step_and_many_parameters(env, T, N, K):
    """One reduction step, whole and ragged, 32 M parameters and more: a rule of its own picks the tiles.  The same bits as
    those of another configuration, and the definition on a stretch of rows (fp32 sums of exact products: 1e-5)."""
    torch, tm = env
    print(f"weight gradient T={T} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn((T, K), generator=g, device="cuda").bfloat16()
    dy = (torch.randn((T, N), generator=g, device="cuda") * 0.1).bfloat16()
    s = stream_ptr(torch)
    out = [torch.full((N, K), float("nan"), device="cuda") for _ in range(2)]
    tm.tm_op_linear_wgrad(BF16, T, N, K, dy, x, out[0], 0, s)
    try:
        tm.tm_gemm_force_config(1)
        tm.tm_op_linear_wgrad(BF16, T, N, K, dy, x, out[1], 0, s)
    finally:
        tm.tm_gemm_force_config(-1)
    assert torch.equal(out[0], out[1])
    rows = slice(N - 50, N)
    ref = to_host(dy[:, rows]).T @ to_host(x)
    assert rel_err(to_host(out[0][rows]), ref) <= 1e-5


def test_linear_results_are_bit_reproducible(env):
    torch, tm = env
    rng = np.random.default_rng(3)
    T, N, K = 384, 264, 320
    x, w, dy = rand(rng, (T, K), 1.0, BF16), rand(rng, (N, K), 0.05, BF16), rand(rng, (T, N), 0.1, BF16)
    xd, wd, dyd = (to_dev(torch, a, BF16) for a in (x, w, dy))
    outs = []
    for _ in range(2):
        y = torch.empty((T, N), dtype=torch.bfloat16, device="cuda")
        dw = torch.zeros((N, K), dtype=torch.float32, device="cuda")
        tm.tm_op_linear_fwd(BF16, T, N, K, xd, wd, None, None, y, stream_ptr(torch))
        tm.tm_op_linear_wgrad(BF16, T, N, K, dyd, xd, dw, 1, stream_ptr(torch))
        outs.append((y, dw))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])


# ------------------------------------------------------------------ bias gradient
@pytest.mark.parametrize("dtype,T,N", [(BF16, 300, 264), (BF16, 5, 8), (FP32, 131, 72), (BF16, 2048, 1536)])
def test_bias_grad(env, dtype, T, N):
    torch, tm = env
    rng = np.random.default_rng(11)
    dy = rand(rng, (T, N), 0.1, dtype)
    g0 = rng.standard_normal(N).astype(np.float32)
    db = f32_dev(torch, g0)
    scratch = torch.empty(tm.tm_op_reduce_scratch_bytes(T, N), dtype=torch.uint8, device="cuda")
    tm.tm_op_bias_grad(dtype, T, N, to_dev(torch, dy, dtype), db, scratch, 1, stream_ptr(torch))
    assert rel_err(to_host(db), g0 + dy.astype(np.float64).sum(axis=0)) <= 1e-5


# ------------------------------------------------------------------ norms
@pytest.mark.parametrize("dtype,kind,T,h", [
    (BF16, so.NORM_LAYERNORM, 37, 264), (BF16, so.NORM_RMSNORM, 37, 264), (BF16, so.NORM_LAYERNORM, 9, 12288),
    (BF16, so.NORM_RMSNORM, 300, 8192), (FP32, so.NORM_LAYERNORM, 37, 256), (FP32, so.NORM_RMSNORM, 1, 8),
    (BF16, so.NORM_LAYERNORM, 600, 16384)])
def test_norm_fwd_bwd(env, dtype, kind, T, h):
    torch, tm = env
    print(f"norm dtype={dtype} kind={kind} T={T} h={h}", flush=True)
    rng = np.random.default_rng(h + T)
    x = rand(rng, (T, h), 1.5, dtype, mean=0.3)
    gain, off = rand(rng, (h,), 0.1, dtype, mean=1.0), rand(rng, (h,), 0.1, dtype)
    dout, dres = rand(rng, (T, h), 0.1, dtype), rand(rng, (T, h), 0.1, dtype)
    eps = 1e-5
    td = torch_dtype(torch, dtype)
    s = stream_ptr(torch)
    xd, gd, od = to_dev(torch, x, dtype), to_dev(torch, gain, dtype), to_dev(torch, off, dtype)
    out = torch.empty((T, h), dtype=td, device="cuda")
    mean = torch.zeros(T, dtype=torch.float32, device="cuda")
    rstd = torch.zeros(T, dtype=torch.float32, device="cuda")
    ln = kind == so.NORM_LAYERNORM
    tm.tm_op_norm_fwd(dtype, kind, T, h, eps, xd, gd, od if ln else None, out, mean if ln else None, rstd, s)
    ref, xhat, r = so.norm_fwd(x, gain.astype(np.float64), off.astype(np.float64) if ln else None, kind, eps)
    assert rel_err(to_host(out), ref) <= tol_of(dtype)
    assert rel_err(to_host(rstd), r[:, 0]) <= 1e-5
    if ln:
        assert np.abs(to_host(mean) - x.astype(np.float64).mean(axis=1)).max() <= 1e-5

    dx = torch.empty((T, h), dtype=td, device="cuda")
    g0, o0 = rng.standard_normal(h).astype(np.float32), rng.standard_normal(h).astype(np.float32)
    dgain, doff = f32_dev(torch, g0), f32_dev(torch, o0)
    scratch = torch.empty(tm.tm_op_reduce_scratch_bytes(T, 3 * h), dtype=torch.uint8, device="cuda")
    tm.tm_op_norm_bwd(dtype, kind, T, h, to_dev(torch, dout, dtype), xd, mean if ln else None, rstd, gd,
                      to_dev(torch, dres, dtype), dx, dgain, doff if ln else None, scratch, 1, s)
    rdx, rdg, rdo = so.norm_bwd(dout, xhat, r, gain.astype(np.float64), kind)
    assert rel_err(to_host(dx), rdx + dres) <= tol_of(dtype)
    assert rel_err(to_host(dgain), g0 + rdg) <= 1e-4
    if ln:
        assert rel_err(to_host(doff), o0 + rdo) <= 1e-4
    # without a residual gradient, and storing instead of adding the gain / offset gradients
    tm.tm_op_norm_bwd(dtype, kind, T, h, to_dev(torch, dout, dtype), xd, mean if ln else None, rstd, gd, None, dx,
                      dgain, doff if ln else None, scratch, 0, s)
    assert rel_err(to_host(dx), rdx) <= tol_of(dtype)
    assert rel_err(to_host(dgain), rdg) <= 1e-4
    if ln:
        assert rel_err(to_host(doff), rdo) <= 1e-4
    # the variant that also returns the column sums of dx (a bias gradient without another pass): same dx, same
    # gain / offset gradients bit for bit, and the sums of the values as stored
    dx2 = torch.empty_like(dx)
    dg2, do2 = torch.empty_like(dgain), torch.empty_like(doff)
    c0 = rng.standard_normal(h).astype(np.float32)
    csum = f32_dev(torch, c0)
    tm.tm_op_norm_bwd(dtype, kind, T, h, to_dev(torch, dout, dtype), xd, mean if ln else None, rstd, gd,
                      to_dev(torch, dres, dtype), dx, dgain, doff if ln else None, scratch, 0, s)
    tm.tm_op_norm_bwd_colsum(dtype, kind, T, h, to_dev(torch, dout, dtype), xd, mean if ln else None, rstd, gd,
                             to_dev(torch, dres, dtype), dx2, dg2, do2 if ln else None, csum, scratch, 0, s)
    torch.cuda.synchronize()
    assert torch.equal(dx, dx2) and torch.equal(dgain, dg2) and (not ln or torch.equal(doff, do2))
    assert rel_err(to_host(csum), to_host(dx2).sum(axis=0)) <= 1e-5
    tm.tm_op_norm_bwd_colsum(dtype, kind, T, h, to_dev(torch, dout, dtype), xd, mean if ln else None, rstd, gd,
                             to_dev(torch, dres, dtype), dx2, dg2, do2 if ln else None, csum, scratch, 1, s)
    assert rel_err(to_host(csum), 2.0 * to_host(dx2).sum(axis=0)) <= 1e-5
    assert rel_err(to_host(csum), 2.0 * (rdx + dres).sum(axis=0)) <= tol_of(dtype)


@pytest.mark.parametrize("dtype,kind,T,h", [
    (BF16, so.NORM_LAYERNORM, 1, 8), (BF16, so.NORM_RMSNORM, 9, 512), (BF16, so.NORM_LAYERNORM, 300, 520), (BF16, so.NORM_RMSNORM, 2500, 1024),
    (BF16, so.NORM_LAYERNORM, 7, 1032), (BF16, so.NORM_LAYERNORM, 1500, 2048), (BF16, so.NORM_RMSNORM, 5, 2056),
    (FP32, so.NORM_LAYERNORM, 17, 264), (FP32, so.NORM_RMSNORM, 2100, 512), (FP32, so.NORM_LAYERNORM, 3, 1024), (FP32, so.NORM_LAYERNORM, 4, 1032),
    (BF16, so.NORM_LAYERNORM, 64, 512), (BF16, so.NORM_RMSNORM, 65, 512), (BF16, so.NORM_LAYERNORM, 192, 1024), (BF16, so.NORM_LAYERNORM, 193, 1024),
    (BF16, so.NORM_LAYERNORM, 193, 2048), (BF16, so.NORM_LAYERNORM, 257, 1536), (FP32, so.NORM_LAYERNORM, 193, 264), (FP32, so.NORM_LAYERNORM, 257, 1024),
    (FP32, so.NORM_LAYERNORM, 65, 256)])
def test_norm_rows_of_a_wave_or_two(env, dtype, kind, T, h):
    """The widths and row counts at which a row goes to one wave, two waves or a whole block, and row counts that leave part
    of a block's rows empty (one row; one more than a block holds; more rows than the blocks take at once): as
    test_norm_fwd_bwd."""
    test_norm_fwd_bwd(env, dtype, kind, T, h)


@pytest.mark.parametrize("dtype,kind,T,h", [
    (BF16, so.NORM_LAYERNORM, 256, 2056), (BF16, so.NORM_LAYERNORM, 257, 2056), (BF16, so.NORM_RMSNORM, 1024, 4096), (BF16, so.NORM_RMSNORM, 1025, 4096),
    (BF16, so.NORM_LAYERNORM, 1027, 4088), (BF16, so.NORM_LAYERNORM, 1026, 4104), (FP32, so.NORM_LAYERNORM, 1025, 1032), (FP32, so.NORM_RMSNORM, 1031, 2048),
    (FP32, so.NORM_LAYERNORM, 1280, 1032), (FP32, so.NORM_LAYERNORM, 1281, 1032), (FP32, so.NORM_RMSNORM, 1283, 1408), (BF16, so.NORM_LAYERNORM, 2304, 2056),
    (BF16, so.NORM_LAYERNORM, 2305, 2056), (BF16, so.NORM_RMSNORM, 2307, 2816), (BF16, so.NORM_LAYERNORM, 2307, 2824)])
def test_norm_rows_of_four_waves(env, dtype, kind, T, h):
    """The widths and row counts at which a row goes to four waves, forward (more than 256 rows of 4 to 8 KB) and backward (more
    than 1280 in fp32, 2304 in bf16, up to 5.5 KB), with a row too few for the last block: as test_norm_fwd_bwd."""
    test_norm_fwd_bwd(env, dtype, kind, T, h)


@pytest.mark.parametrize("dtype,T,N", [(BF16, 1, 8), (BF16, 513, 520), (FP32, 2049, 264), (BF16, 17000, 24)])
def test_bias_grad_row_groups(env, dtype, T, N):
    """One group of one row, and the row counts at which the number of row groups changes, as test_bias_grad."""
    test_bias_grad(env, dtype, T, N)


# ------------------------------------------------------------------ activations
@pytest.mark.parametrize("dtype", [BF16, FP32])
@pytest.mark.parametrize("act", [so.ACT_GELU_TANH, so.ACT_GELU_ERF, so.ACT_SWIGLU])
def test_activation_fwd_bwd(env, dtype, act):
    torch, tm = env
    rng = np.random.default_rng(act + 5)
    T, f = 77, 136
    width = 2 * f if act == so.ACT_SWIGLU else f
    u = rand(rng, (T, width), 2.0, dtype)
    dg = rand(rng, (T, f), 0.1, dtype)
    td = torch_dtype(torch, dtype)
    s = stream_ptr(torch)
    ud = to_dev(torch, u, dtype)
    g = torch.empty((T, f), dtype=td, device="cuda")
    du = torch.empty((T, width), dtype=td, device="cuda")
    tm.tm_op_act_fwd(dtype, act, T, f, ud, g, s)
    tm.tm_op_act_bwd(dtype, act, T, f, to_dev(torch, dg, dtype), ud, du, s)
    u64, dg64 = u.astype(np.float64), dg.astype(np.float64)
    if act == so.ACT_SWIGLU:
        ref = so.swiglu_fwd(u64[:, :f], u64[:, f:])
        rdu = np.concatenate(so.swiglu_bwd(dg64, u64[:, :f], u64[:, f:]), axis=1)
    else:
        ref, rdu = so.gelu_fwd(u64, act), so.gelu_bwd(dg64, u64, act)
    tol = TOL_BF16 if dtype == BF16 else 1e-5
    assert rel_err(to_host(g), ref) <= tol
    assert rel_err(to_host(du), rdu) <= tol


# ------------------------------------------------------------------ rotary
@pytest.mark.parametrize("dtype,seq,batch,heads,d", [(BF16, 33, 2, 3, 128), (FP32, 17, 1, 2, 8), (BF16, 4100, 1, 1, 64)])
def test_rotary_forward_and_inverse(env, dtype, seq, batch, heads, d):
    torch, tm = env
    rng = np.random.default_rng(seq)
    width = (heads + 2) * d        # two trailing heads (the V part) must stay untouched
    z = rand(rng, (seq, batch, width), 1.0, dtype)
    buf = to_dev(torch, z, dtype)
    tm.tm_op_rotary(dtype, seq, batch, heads, d, width, 10000.0, 0, buf, stream_ptr(torch))
    ang = so.rotary_angles(seq, d, 10000.0)
    z64 = z.astype(np.float64)
    ref = z64.copy()
    ref[..., :heads * d] = so.rotary_apply(z64[..., :heads * d].reshape(seq, batch, heads, d), ang).reshape(seq, batch, -1)
    got = to_host(buf)
    assert rel_err(got, ref) <= (TOL_BF16 if dtype == BF16 else 1e-5)
    assert (got[..., heads * d:] == z64[..., heads * d:]).all()
    tm.tm_op_rotary(dtype, seq, batch, heads, d, width, 10000.0, 1, buf, stream_ptr(torch))
    assert rel_err(to_host(buf), z64) <= (TOL_BF16 if dtype == BF16 else 1e-5)


@pytest.mark.parametrize("dtype,seq,batch,heads,d", [(BF16, 1, 1, 3, 16), (BF16, 37, 2, 5, 80), (FP32, 9, 3, 3, 8), (FP32, 130, 1, 33, 64),
                                                     (BF16, 5, 1, 4, 512), (BF16, 1024, 2, 5, 64), (FP32, 4096, 1, 13, 128), (BF16, 4095, 1, 2, 128)])
def test_rotary_rows_and_elements_agree(env, dtype, seq, batch, heads, d):
    """The form for whole 16-byte chunks (several rows a block, one row, a ragged last block, more heads than a pass of the
    block holds, the widest half, the fewest heads it takes at three numbers of angles) against the element-wise form, which a
    buffer off the 16-byte alignment takes (and calls of few heads: the last)."""
    torch, tm = env
    width = (heads + 1) * d
    z = to_dev(torch, rand(np.random.default_rng(d), (seq, batch, width), 1.0, dtype), dtype)
    buf = z.clone()
    store = torch.empty(z.numel() + 16, dtype=z.dtype, device="cuda")
    off = store[1:1 + z.numel()].view_as(z)
    off.copy_(z)
    for inverse in (0, 1, 1):
        tm.tm_op_rotary(dtype, seq, batch, heads, d, width, 10000.0, inverse, buf, stream_ptr(torch))
        tm.tm_op_rotary(dtype, seq, batch, heads, d, width, 10000.0, inverse, off, stream_ptr(torch))
        assert torch.equal(buf, off)


# ------------------------------------------------------------------ attention
ATTN_SHAPES = [
    # dtype, seq, batch, nq, nkv, d
    (BF16, 300, 2, 4, 2, 128),   # MFMA path, grouped heads, ragged: 2 query blocks + tail, 5 key tiles
    (BF16, 128, 1, 2, 2, 128),   # exactly one block
    (BF16, 1, 1, 1, 1, 128),     # a single position: ctx = v
    (BF16, 200, 1, 2, 1, 64),    # MFMA path with head size 64
    (BF16, 70, 2, 2, 1, 32),     # MFMA path, the narrowest padded width
    (FP32, 128, 2, 4, 4, 64),    # the tiny preset's attention
    (FP32, 45, 1, 4, 2, 16),
]


@pytest.mark.parametrize("which", ["qkv", "ctx", "dctx", "dqkv", "all"])
@pytest.mark.parametrize("dtype,seq,batch,nq,nkv,d", [(BF16, 70, 2, 4, 2, 64), (BF16, 40, 1, 2, 1, 256), (FP32, 45, 1, 4, 2, 16)])
def test_attention_off_the_alignment(env, dtype, seq, batch, nq, nkv, d, which):
    """Tensors that start one element past a 16-byte boundary: within the stated tolerance of the definition, as the
    aligned ones are (and no farther than twice that from each other, for the gradients)."""
    torch, tm = env
    print(f"attention off the alignment dtype={dtype} seq={seq} d={d} {which}", flush=True)
    rng = np.random.default_rng(seq + d)
    A, W = nq * d, (nq + 2 * nkv) * d
    td, s = torch_dtype(torch, dtype), stream_ptr(torch)
    qkv, dctx = rand(rng, (seq, batch, W), 1.0, dtype), rand(rng, (seq, batch, A), 0.1, dtype)
    scratch = torch.empty(tm.tm_op_attn_bwd_scratch_bytes(dtype, seq, batch, nq, nkv, d) // 4, device="cuda")

    def run(off):
        def place(name, shape, value=None):
            n = int(np.prod(shape))
            t = torch.empty(n + 1, dtype=td, device="cuda")[int(name in off):][:n].view(shape)
            if value is not None:
                t.copy_(to_dev(torch, value, dtype))
            return t
        q, dc = place("qkv", (seq, batch, W), qkv), place("dctx", (seq, batch, A), dctx)
        ctx, dq = place("ctx", (seq, batch, A)), place("dqkv", (seq, batch, W))
        lse = torch.empty((batch, nq, seq), device="cuda")
        tm.tm_op_attn_fwd(dtype, seq, batch, nq, nkv, d, q, ctx, lse, s)
        tm.tm_op_attn_bwd(dtype, seq, batch, nq, nkv, d, q, ctx, dc, lse, scratch, dq, s)
        return to_host(ctx), to_host(lse), to_host(dq)

    off = run(("qkv", "ctx", "dctx", "dqkv") if which == "all" else (which,))
    whole = run(())
    q64 = qkv.astype(np.float64)
    ref = so.attention_fwd(q64[..., :A].reshape(seq, batch, nq, d), q64[..., A:A + nkv * d].reshape(seq, batch, nkv, d),
                           q64[..., A + nkv * d:].reshape(seq, batch, nkv, d)).reshape(seq, batch, A)
    tol = tol_of(dtype)
    assert rel_err(off[0], ref) <= tol
    assert rel_err(off[1], whole[1]) <= 2 * tol
    assert rel_err(off[2], whole[2]) <= 2 * tol


@pytest.mark.parametrize("dtype,seq,batch,nq,nkv,d", ATTN_SHAPES)
def test_attention_fwd_bwd(env, dtype, seq, batch, nq, nkv, d):
    torch, tm = env
    print(f"attention dtype={dtype} seq={seq} batch={batch} nq={nq} nkv={nkv} d={d}", flush=True)
    rng = np.random.default_rng(seq * 3 + d)
    A, W = nq * d, (nq + 2 * nkv) * d
    qkv = rand(rng, (seq, batch, W), 1.0, dtype)
    dctx = rand(rng, (seq, batch, A), 0.1, dtype)
    td = torch_dtype(torch, dtype)
    s = stream_ptr(torch)
    qd = to_dev(torch, qkv, dtype)
    ctx = torch.empty((seq, batch, A), dtype=td, device="cuda")
    lse = torch.zeros((batch, nq, seq), dtype=torch.float32, device="cuda")
    tm.tm_op_attn_fwd(dtype, seq, batch, nq, nkv, d, qd, ctx, lse, s)
    q64 = qkv.astype(np.float64)
    q = q64[..., :A].reshape(seq, batch, nq, d)
    k = q64[..., A:A + nkv * d].reshape(seq, batch, nkv, d)
    v = q64[..., A + nkv * d:].reshape(seq, batch, nkv, d)
    ref = so.attention_fwd(q, k, v)
    tol = tol_of(dtype)
    assert rel_err(to_host(ctx), ref.reshape(seq, batch, A)) <= tol
    # log-sum-exp of the scaled scores, from the definition
    for n in range(batch):
        for g in (0, nq - 1):
            sc = q[:, n, g] @ k[:, n, g // (nq // nkv)].T / math.sqrt(d)
            sc = np.where(np.tril(np.ones((seq, seq), bool)), sc, -np.inf)
            mx = sc.max(axis=1)
            ref_lse = mx + np.log(np.exp(sc - mx[:, None]).sum(axis=1))
            assert np.abs(to_host(lse[n, g]) - ref_lse).max() <= (1e-3 if dtype == BF16 else 1e-4)

    dqkv = torch.zeros((seq, batch, W), dtype=td, device="cuda")
    dvec = torch.empty(tm.tm_op_attn_bwd_scratch_bytes(dtype, seq, batch, nq, nkv, d), dtype=torch.uint8, device="cuda")
    tm.tm_op_attn_bwd(dtype, seq, batch, nq, nkv, d, qd, ctx, to_dev(torch, dctx, dtype), lse, dvec, dqkv, s)
    dq, dk, dv = so.attention_bwd(dctx.astype(np.float64).reshape(seq, batch, nq, d), q, k, v)
    got = to_host(dqkv)
    assert rel_err(got[..., :A], dq.reshape(seq, batch, A)) <= tol
    assert rel_err(got[..., A:A + nkv * d], dk.reshape(seq, batch, -1)) <= tol
    assert rel_err(got[..., A + nkv * d:], dv.reshape(seq, batch, -1)) <= tol


@pytest.mark.parametrize("split", ["0", "1"], ids=["four_wave_blocks", "eight_wave_split_key_tiles"])
@pytest.mark.parametrize("seq,batch,nq,nkv", [(700, 1, 3, 3), (300, 2, 4, 2), (64, 1, 1, 1), (1, 1, 2, 1), (129, 1, 2, 2)],
                         ids=["ragged_11_key_tiles", "grouped_heads", "one_key_tile", "one_position", "one_row_past_a_block"])
def test_attention_block_forms(env, monkeypatch, split, seq, batch, nq, nkv):
    """The head-size-128 forward kernel comes in two block forms, chosen by the grid size (TM_ATTN_SPLIT forces one): four
    waves walking all key tiles of their query rows, and eight waves where two waves share the query rows and take the
    even and the odd key tiles (their softmax states merged at the end).  Both against the checker (and the backward
    pass from each one's log-sum-exp);
    with one key tile the odd side has nothing to do and must contribute nothing."""
    torch, tm = env
    monkeypatch.setenv("TM_ATTN_SPLIT", split)
    d, dtype = 128, BF16
    print(f"attention block form split={split} seq={seq} batch={batch} nq={nq} nkv={nkv}", flush=True)
    rng = np.random.default_rng(seq * 7 + nq)
    A, W = nq * d, (nq + 2 * nkv) * d
    qkv = rand(rng, (seq, batch, W), 1.0, dtype)
    dctx = rand(rng, (seq, batch, A), 0.1, dtype)
    s = stream_ptr(torch)
    qd = to_dev(torch, qkv, dtype)
    ctx = torch.empty((seq, batch, A), dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros((batch, nq, seq), dtype=torch.float32, device="cuda")
    tm.tm_op_attn_fwd(dtype, seq, batch, nq, nkv, d, qd, ctx, lse, s)
    q64 = qkv.astype(np.float64)
    q = q64[..., :A].reshape(seq, batch, nq, d)
    k = q64[..., A:A + nkv * d].reshape(seq, batch, nkv, d)
    v = q64[..., A + nkv * d:].reshape(seq, batch, nkv, d)
    tol = tol_of(dtype)
    assert rel_err(to_host(ctx), so.attention_fwd(q, k, v).reshape(seq, batch, A)) <= tol
    sc = q[:, 0, nq - 1] @ k[:, 0, (nq - 1) // (nq // nkv)].T / math.sqrt(d)
    sc = np.where(np.tril(np.ones((seq, seq), bool)), sc, -np.inf)
    mx = sc.max(axis=1)
    assert np.abs(to_host(lse[0, nq - 1]) - (mx + np.log(np.exp(sc - mx[:, None]).sum(axis=1)))).max() <= 1e-3
    dqkv = torch.zeros((seq, batch, W), dtype=torch.bfloat16, device="cuda")
    scratch = torch.empty(tm.tm_op_attn_bwd_scratch_bytes(dtype, seq, batch, nq, nkv, d), dtype=torch.uint8, device="cuda")
    tm.tm_op_attn_bwd(dtype, seq, batch, nq, nkv, d, qd, ctx, to_dev(torch, dctx, dtype), lse, scratch, dqkv, s)
    dq, dk, dv = so.attention_bwd(dctx.astype(np.float64).reshape(seq, batch, nq, d), q, k, v)
    got = to_host(dqkv)
    assert rel_err(got[..., :A], dq.reshape(seq, batch, A)) <= tol
    assert rel_err(got[..., A:A + nkv * d], dk.reshape(seq, batch, -1)) <= tol
    assert rel_err(got[..., A + nkv * d:], dv.reshape(seq, batch, -1)) <= tol


@pytest.mark.parametrize("form", ["0", "1", "2"], ids=["separate_blocks", "split_and_single_launch", "shared_walks"])
@pytest.mark.parametrize("seq,batch,nq,nkv,d", [(65, 1, 2, 2, 8), (300, 2, 4, 2, 32), (129, 1, 2, 1, 40), (1, 2, 2, 1, 64),
                                                 (193, 1, 2, 2, 64), (64, 1, 4, 1, 72), (200, 2, 2, 2, 80), (130, 1, 2, 1, 96),
                                                 (127, 1, 1, 1, 104), (257, 1, 2, 1, 120), (1, 1, 2, 1, 128), (65, 2, 2, 2, 128),
                                                 (300, 1, 2, 1, 128)])
def test_attention_head_sizes_below_128(env, monkeypatch, form, seq, batch, nq, nkv, d):
    """bf16 head sizes on the matrix cores: every padded width (32, 64, 96, 128), head sizes with and without padding
    columns, one position, ends of tiles, grouped heads, in every block form (0: a walk per block; 1: two sets of waves
    share a forward walk, one backward launch; 2: four share a forward walk, two a backward one).  Below 128
    probabilities keep 16 significand bits, so a result is off by its own rounding to bf16 (2^-9 of a value) and, behind ctx, by
    ctx's rounding in the row statistics of the backward pass: 2^-8 for ctx, 2^-7 for the gradients."""
    torch, tm = env
    for name in ("TM_ATTN_SPLIT", "TM_ATTN_BWD_BOTH"):
        monkeypatch.setenv(name, form)
    print(f"attention form={form} seq={seq} batch={batch} nq={nq} nkv={nkv} d={d}", flush=True)
    rng = np.random.default_rng(seq * 5 + d)
    A, B, W = nq * d, nkv * d, (nq + 2 * nkv) * d
    qkv, dctx = rand(rng, (seq, batch, W), 1.0, BF16), rand(rng, (seq, batch, A), 0.1, BF16)
    s = stream_ptr(torch)
    qd = to_dev(torch, qkv, BF16)
    ctx = torch.full((seq + 1, batch, A), 7.0, dtype=torch.bfloat16, device="cuda")        # one row more: stays as it is
    dqkv = torch.full((seq + 1, batch, W), 7.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros((batch, nq, seq), dtype=torch.float32, device="cuda")
    scratch = torch.empty(tm.tm_op_attn_bwd_scratch_bytes(BF16, seq, batch, nq, nkv, d), dtype=torch.uint8, device="cuda")
    tm.tm_op_attn_fwd(BF16, seq, batch, nq, nkv, d, qd, ctx, lse, s)
    tm.tm_op_attn_bwd(BF16, seq, batch, nq, nkv, d, qd, ctx, to_dev(torch, dctx, BF16), lse, scratch, dqkv, s)
    q64 = qkv.astype(np.float64)
    q, k, v = (a.reshape(seq, batch, -1, d) for a in (q64[..., :A], q64[..., A:A + B], q64[..., A + B:]))
    bounds = (tol_of(BF16), tol_of(BF16)) if d == 128 else (2.0 ** -8, 2.0 ** -7)
    assert rel_err(to_host(ctx[:seq]), so.attention_fwd(q, k, v).reshape(seq, batch, A)) <= bounds[0]
    refs = so.attention_bwd(dctx.astype(np.float64).reshape(seq, batch, nq, d), q, k, v)
    got = to_host(dqkv[:seq])
    for part, ref in zip((got[..., :A], got[..., A:A + B], got[..., A + B:]), refs):
        assert rel_err(part, ref.reshape(seq, batch, -1)) <= bounds[1]
    assert bool((ctx[seq:] == 7.0).all()) and bool((dqkv[seq:] == 7.0).all())


@pytest.mark.parametrize("form", ["0", "1", "2"], ids=["separate_blocks", "split_and_single_launch", "shared_walks"])
@pytest.mark.parametrize("d", [32, 64, 96, 120, 128])
def test_attention_maxima_that_rise_along_the_keys(env, monkeypatch, form, d):
    """Row maxima that rise by 3, 7.9, 8.1 and 30 powers of two from one tile of 64 keys to the next, in two thirds of the rows
    of a wave, half of these the other way round (falling): what a walk has summed up is rescaled, or kept beside probabilities
    of up to 2^8, in every block form.  Bounds as for random scores; an exponent of magnitude up to 72 is off by a few
    72 * 2^-24, which leaves 5e-5 for the log-sum-exp."""
    torch, tm = env
    for name in ("TM_ATTN_SPLIT", "TM_ATTN_BWD_BOTH"):
        monkeypatch.setenv(name, form)
    print(f"attention rising maxima form={form} d={d}", flush=True)
    seq, batch, nq, nkv = 596, 1, 2, 1
    rng = np.random.default_rng(d)
    A, B, W = nq * d, nkv * d, (nq + 2 * nkv) * d
    qkv, dctx = rand(rng, (seq, batch, W), 1.0, BF16), rand(rng, (seq, batch, A), 0.1, BF16)
    tile = np.arange(seq) // 64
    height = np.cumsum([0, 3, 7.9, 8.1, 30, 3, 7.9, 8.1, 3, 0])[tile] * math.log(2.0) * math.sqrt(d)
    coarse = si.snap_to_bf16_grid(height.astype(np.float32))
    k = qkv[:, 0, A:A + B]
    k[:] = si.snap_to_bf16_grid(0.25 * k)
    k[:, 0], k[:, 1] = coarse, si.snap_to_bf16_grid((height - coarse).astype(np.float32))
    for g in range(nq):                                       # rows that follow the rise, that fall with it, that ignore it
        qkv[:, 0, g * d:g * d + 2] = np.array([1.0, -1.0, 0.0], np.float32)[(np.arange(seq) + g) % 3][:, None]
    s = stream_ptr(torch)
    qd = to_dev(torch, qkv, BF16)
    ctx = torch.empty((seq, batch, A), dtype=torch.bfloat16, device="cuda")
    dqkv = torch.empty((seq, batch, W), dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros((batch, nq, seq), dtype=torch.float32, device="cuda")
    scratch = torch.empty(tm.tm_op_attn_bwd_scratch_bytes(BF16, seq, batch, nq, nkv, d), dtype=torch.uint8, device="cuda")
    tm.tm_op_attn_fwd(BF16, seq, batch, nq, nkv, d, qd, ctx, lse, s)
    tm.tm_op_attn_bwd(BF16, seq, batch, nq, nkv, d, qd, ctx, to_dev(torch, dctx, BF16), lse, scratch, dqkv, s)
    q64 = qkv.astype(np.float64)
    q, k, v = (a.reshape(seq, batch, -1, d) for a in (q64[..., :A], q64[..., A:A + B], q64[..., A + B:]))
    bounds = (tol_of(BF16), tol_of(BF16)) if d == 128 else (2.0 ** -8, 2.0 ** -7)
    assert rel_err(to_host(ctx), so.attention_fwd(q, k, v).reshape(seq, batch, A)) <= bounds[0]
    for g in range(nq):
        sc = np.where(np.tril(np.ones((seq, seq), bool)), q[:, 0, g] @ k[:, 0, 0].T / math.sqrt(d), -np.inf)
        mx = sc.max(axis=1)
        assert np.abs(to_host(lse[0, g]) - (mx + np.log(np.exp(sc - mx[:, None]).sum(axis=1)))).max() <= 5e-5
        rises = np.diff([sc[-20:, 64 * t:64 * t + 64].max(axis=1) for t in range(9)], axis=0) / math.log(2.0)
        assert rises.max() > 25 and ((rises > 2) & (rises < 7.9)).any() and ((rises > 8.1) & (rises < 12)).any()
    refs = so.attention_bwd(dctx.astype(np.float64).reshape(seq, batch, nq, d), q, k, v)
    got = to_host(dqkv)
    # (the two columns of dQ that the heights are in: their hundreds times ctx's rounding in the row statistics)
    assert rel_err(got[..., :A].reshape(seq, batch, nq, d)[..., 2:], refs[0][..., 2:]) <= bounds[1]
    for part, ref in zip((got[..., A:A + B], got[..., A + B:]), refs[1:]):
        assert rel_err(part, ref.reshape(seq, batch, -1)) <= bounds[1]


@pytest.mark.parametrize("seq,batch,nq,nkv,d", [(1, 2, 2, 1, 24), (5, 2, 2, 1, 8), (32, 1, 2, 2, 32), (33, 2, 4, 2, 40), (64, 1, 1, 1, 64), (65, 1, 4, 1, 64),
                                                 (200, 2, 2, 2, 80), (130, 1, 2, 1, 96), (127, 1, 2, 2, 104), (257, 1, 2, 1, 128)])
def test_attention_fp32_tiles(env, seq, batch, nq, nkv, d):
    """fp32 attention on the matrix cores: every padded width (32, 64, 96, 128), with and without padding columns, one
    position, ends of the 32-row tiles and 64-row blocks, grouped heads.  fp32 throughout: an exponent of magnitude up to
    30 is off by 30 * 2^-23 = 4e-6, which bounds a probability's relative error; 1e-5 with the sums."""
    torch, tm = env
    print(f"attention fp32 seq={seq} batch={batch} nq={nq} nkv={nkv} d={d}", flush=True)
    rng = np.random.default_rng(seq * 11 + d)
    A, B, W = nq * d, nkv * d, (nq + 2 * nkv) * d
    qkv, dctx = rand(rng, (seq, batch, W), 1.0, FP32), rand(rng, (seq, batch, A), 0.1, FP32)
    s = stream_ptr(torch)
    qd = to_dev(torch, qkv, FP32)
    ctx = torch.full((seq + 1, batch, A), 7.0, device="cuda")        # one row more: stays as it is
    dqkv = torch.full((seq + 1, batch, W), 7.0, device="cuda")
    lse = torch.zeros((batch, nq, seq), dtype=torch.float32, device="cuda")
    scratch = torch.empty(tm.tm_op_attn_bwd_scratch_bytes(FP32, seq, batch, nq, nkv, d), dtype=torch.uint8, device="cuda")
    tm.tm_op_attn_fwd(FP32, seq, batch, nq, nkv, d, qd, ctx, lse, s)
    tm.tm_op_attn_bwd(FP32, seq, batch, nq, nkv, d, qd, ctx, to_dev(torch, dctx, FP32), lse, scratch, dqkv, s)
    q64 = qkv.astype(np.float64)
    q, k, v = (a.reshape(seq, batch, -1, d) for a in (q64[..., :A], q64[..., A:A + B], q64[..., A + B:]))
    assert rel_err(to_host(ctx[:seq]), so.attention_fwd(q, k, v).reshape(seq, batch, A)) <= 1e-5
    refs = so.attention_bwd(dctx.astype(np.float64).reshape(seq, batch, nq, d), q, k, v)
    got = to_host(dqkv[:seq])
    for part, ref in zip((got[..., :A], got[..., A:A + B], got[..., A + B:]), refs):
        assert rel_err(part, ref.reshape(seq, batch, -1)) <= 1e-5
    assert bool((ctx[seq:] == 7.0).all()) and bool((dqkv[seq:] == 7.0).all())


@pytest.mark.parametrize("seq,batch,nq,nkv,d", [(65, 2, 2, 2, 64), (96, 1, 2, 1, 24), (97, 2, 2, 2, 96), (128, 1, 4, 2, 128), (129, 2, 4, 4, 64), (160, 1, 2, 2, 32),
                                                 (255, 1, 32, 8, 32), (256, 2, 32, 32, 32), (321, 2, 8, 2, 64), (512, 1, 16, 16, 40), (513, 1, 16, 16, 40)])
def test_attention_fp32_walk_shares(env, seq, batch, nq, nkv, d):
    """fp32 attention whose four waves share one walk, around the lengths and numbers of walks at which it takes over from
    the form with two sides, with last steps of one to four tiles: bounds as for the tiles (exponents to 30: 4e-6), 1e-5."""
    test_attention_fp32_tiles(env, seq, batch, nq, nkv, d)


@pytest.mark.parametrize("dtype,seq,batch,nq,nkv,d", [(BF16, 8, 40000, 16, 16, 64), (BF16, 1, 25000, 16, 16, 128), (FP32, 8, 40000, 16, 1, 64)])
def test_attention_rows_behind_a_short_sequence_read_as_zero(env, dtype, seq, batch, nq, nkv, d):
    """A few positions of a very large batch: the other rows of the staged query tiles lie behind the tensor, some of them
    a whole multiple of 2^32 bytes and a little more (bf16 heads of 64: row 53 of both tensors, 53 x 82 and 53 x 246 MB;
    heads of 128: row 42; fp32: row 27), and add nothing to dK and dV.  Entries are independent: the first, some in the
    middle and the last ones against the same entries in a batch of their own.  Both calls round alike up to the order of
    their sums: two bf16 roundings apart at most (2^-7 of the largest), 1e-5 in fp32."""
    torch, tm = env
    print(f"attention of {seq} positions dtype={dtype} batch={batch} heads={nq}/{nkv} d={d}", flush=True)
    A, W = nq * d, (nq + 2 * nkv) * d
    g = torch.Generator(device="cuda").manual_seed(batch + d)
    td = torch_dtype(torch, dtype)
    qkv = torch.randn((seq, batch, W), generator=g, device="cuda").to(td)
    dctx = (torch.randn((seq, batch, A), generator=g, device="cuda") * 0.1).to(td)
    s = stream_ptr(torch)

    def run(qd, dd):
        n = qd.shape[1]
        ctx, dqkv = torch.zeros_like(dd), torch.zeros_like(qd)
        lse = torch.zeros((n, nq, seq), dtype=torch.float32, device="cuda")
        scratch = torch.empty(tm.tm_op_attn_bwd_scratch_bytes(dtype, seq, n, nq, nkv, d), dtype=torch.uint8, device="cuda")
        tm.tm_op_attn_fwd(dtype, seq, n, nq, nkv, d, qd, ctx, lse, s)
        tm.tm_op_attn_bwd(dtype, seq, n, nq, nkv, d, qd, ctx, dd, lse, scratch, dqkv, s)
        return ctx.float(), dqkv.float()

    ctx, dqkv = run(qkv, dctx)
    for first in (0, batch // 2, batch - 20):
        part = slice(first, first + 20)
        for got, ref in zip((ctx[:, part], dqkv[:, part]), run(qkv[:, part].contiguous(), dctx[:, part].contiguous())):
            assert float((got - ref).abs().max()) <= (2.0 ** -7 if dtype == BF16 else 1e-5) * float(ref.abs().max())


SHORT_WALKS = [(BF16, 1, 256, 8, 2, 64), (BF16, 2, 256, 8, 8, 64), (BF16, 3, 256, 8, 4, 120), (BF16, 4, 64, 8, 8, 8), (BF16, 5, 256, 8, 8, 8),
               (BF16, 6, 256, 8, 8, 8), (FP32, 1, 64, 8, 8, 96), (FP32, 4, 64, 8, 2, 32), (FP32, 5, 64, 8, 8, 32), (FP32, 6, 64, 8, 4, 64),
               (FP32, 7, 64, 8, 8, 64), (FP32, 8, 64, 8, 8, 72), (FP32, 9, 64, 8, 8, 72), (FP32, 4, 40, 4, 4, 128), (FP32, 4, 2, 2, 2, 16)]


@pytest.mark.parametrize("dtype,seq,batch,nq,nkv,d", SHORT_WALKS + [(BF16, 20, 1, 4, 2, 160), (FP32, 70, 1, 2, 1, 256)])
def test_attention_one_row_per_wave(env, dtype, seq, batch, nq, nkv, d):
    """Short sequences of many heads and entries on both sides of the limits up to which they go to the kernels of one row
    per wave, and head sizes above 128, which always do.  bf16 results are off by their rounding and, behind ctx, by
    ctx's in the row statistics (2^-8, 2^-7); fp32 ones by an exponent's error (1e-5)."""
    torch, tm = env
    print(f"attention rows dtype={dtype} seq={seq} batch={batch} heads={nq}/{nkv} d={d}", flush=True)
    rng = np.random.default_rng(seq * 7 + d)
    A, B, W = nq * d, nkv * d, (nq + 2 * nkv) * d
    qkv, dctx = rand(rng, (seq, batch, W), 1.0, dtype), rand(rng, (seq, batch, A), 0.1, dtype)
    s = stream_ptr(torch)
    qd, dd = to_dev(torch, qkv, dtype), to_dev(torch, dctx, dtype)
    ctx, dqkv = torch.empty_like(dd), torch.empty_like(qd)
    lse = torch.zeros((batch, nq, seq), dtype=torch.float32, device="cuda")
    scratch = torch.empty(tm.tm_op_attn_bwd_scratch_bytes(dtype, seq, batch, nq, nkv, d), dtype=torch.uint8, device="cuda")
    tm.tm_op_attn_fwd(dtype, seq, batch, nq, nkv, d, qd, ctx, lse, s)
    tm.tm_op_attn_bwd(dtype, seq, batch, nq, nkv, d, qd, ctx, dd, lse, scratch, dqkv, s)
    q64 = qkv.astype(np.float64)
    q, k, v = (a.reshape(seq, batch, -1, d) for a in (q64[..., :A], q64[..., A:A + B], q64[..., A + B:]))
    bounds = (2.0 ** -8, 2.0 ** -7) if dtype == BF16 else (1e-5, 1e-5)
    assert rel_err(to_host(ctx), so.attention_fwd(q, k, v).reshape(seq, batch, A)) <= bounds[0]
    refs = so.attention_bwd(dctx.astype(np.float64).reshape(seq, batch, nq, d), q, k, v)
    got = to_host(dqkv)
    top = max(np.abs(r).max() for r in refs)     # with one position dQ and dK are zero
    for part, ref in zip((got[..., :A], got[..., A:A + B], got[..., A + B:]), refs):
        assert np.isfinite(part).all() and np.abs(part - ref.reshape(seq, batch, -1)).max() <= bounds[1] * top


NONFINITE_SHAPES = [(BF16, 70, 2, 2, 40), (BF16, 130, 4, 2, 64), (BF16, 200, 2, 1, 80), (BF16, 129, 2, 2, 120),
                    (FP32, 70, 4, 2, 24), (FP32, 130, 2, 2, 64), (FP32, 100, 2, 1, 96), (FP32, 65, 1, 1, 128)]


@pytest.mark.parametrize("form", ["0", "1", "2"], ids=["separate_blocks", "split_and_single_launch", "shared_walks"])
@pytest.mark.parametrize("dtype,seq,nq,nkv,d", NONFINITE_SHAPES)
def test_attention_keeps_infinities_and_nans_to_their_own_rows(env, monkeypatch, form, dtype, seq, nq, nkv, d):
    """A position that the causal mask excludes from a row leaves the row alone, whatever it holds: an infinite V and a
    NaN K leave the earlier rows of ctx and dQ what they are without them, an infinite dO and a NaN Q the later rows of dK
    and dV (position 5 and the one 5 before the end, so tiles hold both kinds of rows).  Rows whose first tile of scores is
    -Inf have the softmax of the rest.  Head size 128 in bf16 is not meant: it multiplies whole tiles.  Rows as without
    the value: bf16 results to their rounding, 2^-8 of the largest (2^-7 behind ctx), fp32 to 2e-5."""
    torch, tm = env
    for name in ("TM_ATTN_SPLIT", "TM_ATTN_BWD_BOTH"):
        monkeypatch.setenv(name, form)
    print(f"attention with infinities form={form} dtype={dtype} seq={seq} heads={nq}/{nkv} d={d}", flush=True)
    rng = np.random.default_rng(seq + d)
    A, B, W, batch = nq * d, nkv * d, (nq + 2 * nkv) * d, 2
    qkv, dctx = rand(rng, (seq, batch, W), 1.0, dtype), rand(rng, (seq, batch, A), 0.1, dtype)
    s = stream_ptr(torch)

    def run(qd, dd):
        ctx, dqkv = torch.empty_like(dd), torch.empty_like(qd)
        lse = torch.zeros((batch, nq, seq), dtype=torch.float32, device="cuda")
        scratch = torch.empty(tm.tm_op_attn_bwd_scratch_bytes(dtype, seq, batch, nq, nkv, d), dtype=torch.uint8, device="cuda")
        tm.tm_op_attn_fwd(dtype, seq, batch, nq, nkv, d, qd, ctx, lse, s)
        tm.tm_op_attn_bwd(dtype, seq, batch, nq, nkv, d, qd, ctx, dd, lse, scratch, dqkv, s)
        return to_host_raw(ctx), to_host_raw(dqkv)

    to_host_raw = lambda t: t.detach().float().cpu().numpy()
    clean_ctx, clean_d = run(to_dev(torch, qkv, dtype), to_dev(torch, dctx, dtype))
    tol = 2.0 ** -7 if dtype == BF16 else 2e-5

    def same(a, b):
        assert np.isfinite(a).all() and np.abs(a - b).max() <= tol * np.abs(b).max()

    late, early, inf = seq - 5, 5, float("inf")
    qd, dd = to_dev(torch, qkv, dtype), to_dev(torch, dctx, dtype)
    qd[late, 1, A + B] = inf                             # V of kv head 0, entry 1
    qd[late, 1, A] = float("nan")                        # its K
    ctx, dqkv = run(qd, dd)
    same(ctx[:late], clean_ctx[:late])
    same(dqkv[:late, :, :A], clean_d[:late, :, :A])
    same(ctx[:, 0], clean_ctx[:, 0])
    assert np.isnan(ctx[late:, 1, :d]).all()             # the rows that attend to it

    qd, dd = to_dev(torch, qkv, dtype), to_dev(torch, dctx, dtype)
    qd[early, 0, 0] = float("nan")
    dd[early, 0, 1] = inf
    ctx, dqkv = run(qd, dd)
    rows = np.arange(seq) != early
    same(ctx[rows], clean_ctx[rows])
    same(dqkv[rows][..., :A], clean_d[rows][..., :A])
    same(dqkv[early + 1:, :, A:], clean_d[early + 1:, :, A:])
    same(dqkv[:, 1], clean_d[:, 1])
    assert np.isnan(dqkv[:early + 1, 0, A:A + d]).all()

    qd = to_dev(torch, qkv, dtype)
    half = seq // 2
    qd[:, :, 0:A:d] = 1.0
    qd[:half, :, A:A + B:d] = -inf                       # the first half's scores are -Inf, and with them whole tiles
    ctx, _ = run(qd, to_dev(torch, dctx, dtype))
    q64 = qd.float().cpu().numpy().astype(np.float64)[half:]
    q, k, v = (a.reshape(seq - half, batch, -1, d) for a in (q64[..., :A], q64[..., A:A + B], q64[..., A + B:]))
    same(ctx[half:], so.attention_fwd(q, k, v).reshape(seq - half, batch, A))
    assert np.isnan(ctx[:half]).all()


@pytest.mark.parametrize("both", ["0", "1"], ids=["two_launches", "one_launch"])
@pytest.mark.parametrize("seq,batch,nq,nkv", [(700, 1, 3, 3), (300, 2, 4, 2), (64, 1, 1, 1), (1, 1, 2, 1), (129, 1, 2, 2),
                                               (193, 1, 2, 1)],
                         ids=["ragged_11_key_tiles", "grouped_heads", "one_key_tile", "one_position", "one_row_past_a_block",
                              "one_row_past_a_key_tile"])
def test_attention_backward_launch_forms(env, monkeypatch, both, seq, batch, nq, nkv):
    """The head-size-128 backward pass runs as two launches (dQ blocks, then dK/dV blocks) or, for grids that leave
    compute units idle, as one launch that holds both kinds of blocks (TM_ATTN_BWD_BOTH forces one).  Each form against
    the checker; nothing may be written past the tensor's last row."""
    torch, tm = env
    monkeypatch.setenv("TM_ATTN_BWD_BOTH", both)
    d, dtype = 128, BF16
    print(f"attention backward form both={both} seq={seq} batch={batch} nq={nq} nkv={nkv}", flush=True)
    rng = np.random.default_rng(seq * 11 + nq)
    A, W = nq * d, (nq + 2 * nkv) * d
    qkv = rand(rng, (seq, batch, W), 1.0, dtype)
    dctx = rand(rng, (seq, batch, A), 0.1, dtype)
    s = stream_ptr(torch)
    qd = to_dev(torch, qkv, dtype)
    ctx = torch.empty((seq, batch, A), dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros((batch, nq, seq), dtype=torch.float32, device="cuda")
    tm.tm_op_attn_fwd(dtype, seq, batch, nq, nkv, d, qd, ctx, lse, s)
    q64 = qkv.astype(np.float64)
    q = q64[..., :A].reshape(seq, batch, nq, d)
    k = q64[..., A:A + nkv * d].reshape(seq, batch, nkv, d)
    v = q64[..., A + nkv * d:].reshape(seq, batch, nkv, d)
    tol = tol_of(dtype)
    guard = 64                                      # rows after the tensor: nothing may be written there
    dqkv = torch.full((seq + guard, batch, W), float("nan"), dtype=torch.bfloat16, device="cuda")
    scratch = torch.empty(tm.tm_op_attn_bwd_scratch_bytes(dtype, seq, batch, nq, nkv, d), dtype=torch.uint8, device="cuda")
    tm.tm_op_attn_bwd(dtype, seq, batch, nq, nkv, d, qd, ctx, to_dev(torch, dctx, dtype), lse, scratch, dqkv[:seq], s)
    torch.cuda.synchronize()
    assert torch.isnan(dqkv[seq:]).all()
    dq, dk, dv = so.attention_bwd(dctx.astype(np.float64).reshape(seq, batch, nq, d), q, k, v)
    got = to_host(dqkv[:seq])
    assert np.isfinite(got).all()
    assert rel_err(got[..., :A], dq.reshape(seq, batch, A)) <= tol
    assert rel_err(got[..., A:A + nkv * d], dk.reshape(seq, batch, -1)) <= tol
    assert rel_err(got[..., A + nkv * d:], dv.reshape(seq, batch, -1)) <= tol


@pytest.mark.parametrize("seq,batch,nq,nkv", [(700, 1, 3, 3), (300, 2, 4, 2), (257, 1, 2, 1), (1, 1, 1, 1)],
                         ids=["ragged_3_blocks", "grouped_heads", "one_row_past_a_block", "one_position"])
def test_attention_blocks_of_256_query_rows(env, monkeypatch, seq, batch, nq, nkv):
    """Long sequences run the forward and the dQ walk in blocks of 256 query rows (eight waves sharing every staged key /
    value tile).  TM_ATTN_WIDE=1 forces that form on small shapes (with the other forms switched off): against the
    checker, and nothing written past the last row."""
    torch, tm = env
    monkeypatch.setenv("TM_ATTN_WIDE", "1")
    monkeypatch.setenv("TM_ATTN_SPLIT", "0")
    monkeypatch.setenv("TM_ATTN_BWD_BOTH", "0")
    d, dtype = 128, BF16
    print(f"attention 256-row blocks seq={seq} batch={batch} nq={nq} nkv={nkv}", flush=True)
    rng = np.random.default_rng(seq * 13 + nq)
    A, W = nq * d, (nq + 2 * nkv) * d
    qkv = rand(rng, (seq, batch, W), 1.0, dtype)
    dctx = rand(rng, (seq, batch, A), 0.1, dtype)
    s = stream_ptr(torch)
    qd = to_dev(torch, qkv, dtype)
    guard = 64
    ctx = torch.full((seq + guard, batch, A), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros((batch, nq, seq), dtype=torch.float32, device="cuda")
    tm.tm_op_attn_fwd(dtype, seq, batch, nq, nkv, d, qd, ctx[:seq], lse, s)
    q64 = qkv.astype(np.float64)
    q = q64[..., :A].reshape(seq, batch, nq, d)
    k = q64[..., A:A + nkv * d].reshape(seq, batch, nkv, d)
    v = q64[..., A + nkv * d:].reshape(seq, batch, nkv, d)
    tol = tol_of(dtype)
    torch.cuda.synchronize()
    assert torch.isnan(ctx[seq:]).all()
    assert rel_err(to_host(ctx[:seq]), so.attention_fwd(q, k, v).reshape(seq, batch, A)) <= tol
    dqkv = torch.full((seq + guard, batch, W), float("nan"), dtype=torch.bfloat16, device="cuda")
    scratch = torch.empty(tm.tm_op_attn_bwd_scratch_bytes(dtype, seq, batch, nq, nkv, d), dtype=torch.uint8, device="cuda")
    tm.tm_op_attn_bwd(dtype, seq, batch, nq, nkv, d, qd, ctx[:seq], to_dev(torch, dctx, dtype), lse, scratch, dqkv[:seq], s)
    torch.cuda.synchronize()
    assert torch.isnan(dqkv[seq:]).all()
    dq, dk, dv = so.attention_bwd(dctx.astype(np.float64).reshape(seq, batch, nq, d), q, k, v)
    got = to_host(dqkv[:seq])
    assert np.isfinite(got).all()
    assert rel_err(got[..., :A], dq.reshape(seq, batch, A)) <= tol
    assert rel_err(got[..., A:A + nkv * d], dk.reshape(seq, batch, -1)) <= tol
    assert rel_err(got[..., A + nkv * d:], dv.reshape(seq, batch, -1)) <= tol


def test_attention_is_bit_reproducible(env):
    torch, tm = env
    rng = np.random.default_rng(8)
    seq, batch, nq, nkv, d = 260, 1, 4, 1, 128
    A, W = nq * d, (nq + 2 * nkv) * d
    qd = to_dev(torch, rand(rng, (seq, batch, W), 1.0, BF16), BF16)
    dc = to_dev(torch, rand(rng, (seq, batch, A), 0.1, BF16), BF16)
    outs = []
    for _ in range(2):
        ctx = torch.empty((seq, batch, A), dtype=torch.bfloat16, device="cuda")
        lse = torch.empty((batch, nq, seq), dtype=torch.float32, device="cuda")
        dqkv = torch.empty((seq, batch, W), dtype=torch.bfloat16, device="cuda")
        dvec = torch.empty(tm.tm_op_attn_bwd_scratch_bytes(BF16, seq, batch, nq, nkv, d), dtype=torch.uint8, device="cuda")
        tm.tm_op_attn_fwd(BF16, seq, batch, nq, nkv, d, qd, ctx, lse, stream_ptr(torch))
        tm.tm_op_attn_bwd(BF16, seq, batch, nq, nkv, d, qd, ctx, dc, lse, dvec, dqkv, stream_ptr(torch))
        outs.append((ctx, lse, dqkv))
    for a, b in zip(*outs):
        assert torch.equal(a, b)


# ------------------------------------------------------------------ Adam
@pytest.mark.parametrize("n,lowp,zero,step,wd,gs", [(1000003, True, False, 1, 0.0, 1.0), (4096, False, True, 7, 0.01, 0.5),
                                                    (5, True, True, 2, 0.0, 1.0), (8, True, False, 1000, 0.1, 1.0)])
def test_adam_flat_matches_fp64_definition(env, n, lowp, zero, step, wd, gs):
    torch, tm = env
    p, g, m, v = si.make_adam_state(n, seed=step)
    pd, gd, md, vd = (f32_dev(torch, a) for a in (p, g, m, v))
    lo = torch.zeros(n, dtype=torch.bfloat16, device="cuda") if lowp else None
    hp = tm.make_hparams(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=wd, grad_scale=gs, zero_grads=zero)
    tm.tm_adam_step_flat(n, pd, gd, md, vd, lo, hp, step, stream_ptr(torch))
    rp, rm, rv = so.adam_step(p, g, m, v, step, 1e-3, 0.9, 0.999, 1e-8, wd, gs)
    assert rel_err(to_host(pd), rp) <= TOL_ADAM
    assert rel_err(to_host(md), rm) <= TOL_ADAM
    assert rel_err(to_host(vd), rv) <= TOL_ADAM
    if lowp:
        # the bf16 copy is the nearest-even rounding of the fp32 weight the kernel itself stored
        want = so.bf16_round_nearest_even(pd.cpu().numpy())
        got = lo.view(torch.int16).cpu().numpy().view(np.uint16)
        assert (got == want).all()
    if zero:
        assert float(gd.abs().max()) == 0.0
    else:
        assert torch.equal(gd.cpu(), torch.from_numpy(g))


def test_adam_first_step_closed_form(env):
    torch, tm = env
    n = 10000
    p, g, _, _ = si.make_adam_state(n)
    pd, gd = f32_dev(torch, p), f32_dev(torch, g)
    md, vd = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    tm.tm_adam_step_flat(n, pd, gd, md, vd, None, tm.make_hparams(), 1, stream_ptr(torch))
    ref = p.astype(np.float64) - 1e-3 * g.astype(np.float64) / (np.abs(g.astype(np.float64)) + 1e-8)
    assert rel_err(to_host(pd), ref) <= TOL_ADAM


# ------------------------------------------------------------------ argument errors
@pytest.mark.parametrize("n", [1, 7, 4096, 4097, 1_000_003])
def test_sum_of_squares(env, n):
    torch, tm = env
    rng = np.random.default_rng(n)
    g = (rng.standard_normal(n) * 1e-2).astype(np.float32)
    gd = f32_dev(torch, g)
    scratch = torch.empty(tm.tm_sq_sum_scratch_bytes(n), dtype=torch.uint8, device="cuda")
    out = torch.zeros(2, dtype=torch.float64, device="cuda")
    tm.tm_sq_sum(n, gd, scratch, out, stream_ptr(torch))
    tm.tm_sq_sum(n, gd, scratch, out[1:], stream_ptr(torch))
    torch.cuda.synchronize()
    ref = so.grad_sq_sum(g)
    assert abs(float(out[0]) - ref) <= 1e-6 * ref
    assert float(out[0]) == float(out[1])               # fixed summation order


def test_bad_arguments_are_reported_not_launched(env):
    torch, tm = env
    t = torch.zeros(64, dtype=torch.float32, device="cuda")
    with pytest.raises(tm.TmError) as e:
        tm.tm_op_linear_fwd(BF16, 4, 12, 8, t, t, None, None, t, 0)       # N not a multiple of 8
    assert e.value.code == tm.TM_ESIZE
    with pytest.raises(tm.TmError) as e:
        tm.tm_op_linear_fwd(BF16, 4, 8, 8, None, t, None, None, t, 0)
    assert e.value.code == tm.TM_EINVAL
    with pytest.raises(tm.TmError) as e:
        tm.tm_adam_step_flat(8, t, t, t, t, None, tm.make_hparams(), 0, 0)  # step < 1
    assert e.value.code == tm.TM_EINVAL
    with pytest.raises(tm.TmError) as e:
        tm.tm_op_attn_fwd(BF16, 16, 1, 3, 2, 64, t, t, t, 0)               # heads not divisible
    assert e.value.code == tm.TM_ESIZE
    with pytest.raises(tm.TmError) as e:
        tm.tm_op_norm_fwd(BF16, 0, 4, 32768, 1e-5, t, t, t, t, t, t, 0)    # row too wide
    assert e.value.code == tm.TM_ESIZE
