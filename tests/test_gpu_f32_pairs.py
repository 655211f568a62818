"""Small fp32 linear maps: both gradients in one launch, GeLU and its derivative in the products' epilogues (csrc/gemm_f32.hip)."""
import pytest

import synth_inputs as si
from tests.f32_form import form, split
from tests.gpu_util import require_gpu, stream_ptr, to_dev
from tests.stage_runner import GpuStage
from tests.test_gpu_stage import run_and_compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = require_gpu()
    import paper_2412_12636_amd as tm
    return torch, tm


def pairs(cfg):
    """Tiles of the two gradients of FC2, FC1, out-projection and QKV where they share a launch."""
    T, h, A, f = cfg.seq * cfg.micro_batch, cfg.hidden, cfg.n_q_heads * cfg.head_dim, cfg.ffn
    out = []
    for N, K in ((h, f), ((2 if cfg.act == si.ACT_SWIGLU else 1) * f, h), (h, A), (A + 2 * cfg.n_kv_heads * cfg.head_dim, h)):
        d, w = form(T, K, N, False), form(N, K, T, True)
        small = max(d[0], w[0]) <= 32 and not (d[2] or w[2] or split(T, K, N, False) or split(N, K, T, True))
        out.append((d[0],) + w[:2] if small else None)
    return out


def stage(*dims, **options):
    return si.StageConfig(*dims, dtype=si.DTYPE_FP32, **options)


@pytest.mark.parametrize("cfg,tiles", [
    (stage(1, 64, 2, 2, 32, 136, 33, 1), [(16, 16, 4)] * 4),
    (stage(2, 136, 2, 2, 64, 264, 130, 1, norm=si.NORM_RMSNORM, act=si.ACT_SWIGLU), [(16, 16, 4), (16, 32, 4), (16, 16, 4), (16, 16, 4)]),
    (stage(1, 256, 4, 4, 64, 1024, 65, 2, act=si.ACT_GELU_ERF), [(32, 32, 4), (16, 32, 4), (16, 16, 4), (16, 32, 4)]),
    (stage(1, 136, 2, 2, 64, 264, 520, 1), [(32, 16, 4), (16, 16, 4), (16, 16, 4), (16, 16, 4)]),
    (stage(1, 264, 3, 3, 88, 1096, 257, 1, act=si.ACT_GELU_ERF), [(32, 32, 8), (16, 32, 8), (16, 32, 8), (16, 32, 8)]),
    (stage(1, 520, 4, 4, 64, 520, 257, 1), [(32, 32, 8), (32, 32, 8), (16, 32, 8), (32, 32, 8)])],
    ids=["16", "odd_pairs_of_16", "32_split_4", "weight_16", "odd_32_split_8", "32_split_8"])
def test_gradients_that_share_a_launch(env, cfg, tiles):
    """Every pair of tile forms, with edges inside tiles and odd numbers of 16x16 tiles, against the checker; then a second
    micro-batch of the same inputs added in: twice the gradients, up to one rounding of the sum (2^-23)."""
    torch, tm = env
    assert pairs(cfg) == tiles
    print(f"shared launches {cfg}", flush=True)
    run_and_compare(torch, tm, cfg)
    st = GpuStage(torch, tm, cfg, si.make_flat_params(cfg))
    x, dy = to_dev(torch, si.make_x(cfg), cfg.dtype), to_dev(torch, si.make_dy(cfg), cfg.dtype)
    st.fwd(x)
    st.bwd(dy)
    once = st.grads.clone()
    tm.tm_stage_grad_mode(st.handle, tm.TM_GRAD_ADD)
    tm.tm_stage_bwd(st.handle, dy, st.dx, stream_ptr(torch))
    torch.cuda.synchronize()
    assert bool(((st.grads - 2 * once).abs() <= 2.0 ** -23 * (2 * once).abs()).all())
    st.close()
