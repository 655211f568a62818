"""A layer's second norm keeps its partial rows of gain and offset gradients until the first norm's are added up (csrc/stage.hip)."""
import pytest

import synth_inputs as si
from tests.gpu_util import require_gpu, stream_ptr, to_dev
from tests.stage_runner import GpuStage
from tests.test_gpu_stage import run_and_compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("norm,act,bias", [(si.NORM_LAYERNORM, si.ACT_GELU_ERF, 1), (si.NORM_RMSNORM, si.ACT_SWIGLU, 0)], ids=["gpt", "llama"])
@pytest.mark.parametrize("ffn,seq", [(96, 512), (8, 512), (96, 40)], ids=["behind_the_column_sums", "in_the_attention_gradient", "no_room"])
def test_partial_rows_of_the_second_norm(ffn, seq, norm, act, bias):
    """64 partial rows of 3 x 64 floats against 512 x 96 and 512 x 8 floats of FC width and 512 x 64 of attention width, and 40
    rows, which have room in neither: every gradient against the checker, over two layers; with the gradients added a second
    time exactly twice (the same sums)."""
    torch = require_gpu()
    import paper_2412_12636_amd as tm
    cfg = si.StageConfig(2, 64, 4, 4, 16, ffn, seq, 1, dtype=si.DTYPE_FP32, norm=norm, act=act, has_bias=bias)
    print(f"partial rows {cfg}", flush=True)
    run_and_compare(torch, tm, cfg)
    st = GpuStage(torch, tm, cfg, si.make_flat_params(cfg))
    st.fwd(to_dev(torch, si.make_x(cfg), cfg.dtype))
    dy = to_dev(torch, si.make_dy(cfg), cfg.dtype)
    st.bwd(dy)
    once = st.grads.clone()
    tm.tm_stage_grad_mode(st.handle, tm.TM_GRAD_ADD)
    tm.tm_stage_bwd(st.handle, dy, st.dx, stream_ptr(torch))
    torch.cuda.synchronize()
    gains = torch.cat([torch.arange(off, off + shape[0]) for name, off, shape in tm.tm_stage_param_layout(cfg) if "norm" in name])
    gains = gains.to("cuda")
    assert gains.numel() > 0 and torch.equal(st.grads[gains], 2 * once[gains])
    st.close()
