"""fp32 layers on bf16 matrix instructions (conv_gemm_split): each tile
configuration at ragged channel, pixel and K edges against the oracle, and
inputs the three-way split cannot represent against the fp32 kernels."""
import numpy as np
import pytest

import oracle
import workloads as W

from gpu_util import gpu_forward, rel_inf
from test_gpu_layers import LAYER_TOL, check, conv, make

pytestmark = pytest.mark.gpu

# (tile, C, Co, k, stride, pad, H, W, batch, residual)
CASES = [
    ("32x32", 256, 20, 1, 1, 0, 3, 11, 1, False),      # one pixel past a tile, ragged channels
    ("32x32", 260, 36, 1, 1, 0, 6, 6, 1, True),        # K tail of 4 in the last chunk
    ("32x32", 32, 64, 3, 1, 1, 13, 9, 3, True),        # 9 chunks over 4 K parts, padding
    ("32x32", 64, 100, 3, 2, 1, 15, 13, 2, False),     # stride, ragged channel tile
    ("32x64", 256, 512, 1, 1, 0, 31, 27, 1, True),     # ragged pixel tile
    ("32x64", 32, 516, 3, 1, 0, 20, 19, 3, False),     # odd chunk count over 2 K parts
    ("64x64", 288, 260, 1, 2, 0, 61, 59, 4, False),    # stride-2 1x1, ragged channels
    ("64x64", 32, 64, 3, 1, 1, 70, 71, 3, True),
    ("64x128", 32, 64, 3, 1, 1, 99, 101, 5, True),     # 50k pixels, ragged last tile
    ("64x128", 32, 132, 5, 2, 2, 121, 119, 6, False),  # 25 taps, ragged channel tile
]


@pytest.mark.parametrize("tile,ci,co,k,s,p,h,w,batch,res", CASES)
def test_split_tiles(tile, ci, co, k, s, p, h, w, batch, res):
    from paper_2507_18748_amd import Partition
    specs = [conv("c", -1, ci, co, k, s, p)]
    if res:   # residual: a 1x1 layer of the same input and output shape
        specs = [conv("r", -1, ci, co, 1, 1, 0), conv("c", -1, ci, co, k, s, p, res=0)]
    m = make((ci, h, w), specs)
    with Partition(m.layers, W.model_params(m, 0, "f32"), (ci, h, w), 0, len(specs), "f32",
                   max_batch=batch) as part:
        name = part.layer_info(len(specs) - 1, batch)["kernel"]
    assert name.startswith(f"conv_gemm_split<f32,{tile}> ")
    check(m, "f32", batch)


@pytest.mark.parametrize("h,w,batch", [(9, 9, 1), (40, 41, 8)])
def test_split_non_finite(h, w, batch):
    """Infinities, NaN and values that round to an infinite bf16 (3.4e38, whose
    products with the small weights stay finite) give what the fp32 matrix
    instruction gives, and leave the other pixels alone."""
    from paper_2507_18748_amd import Partition
    m = make((64, h, w), [conv("c", -1, 64, 64, 3, 1, 1, act="none")])
    P = W.model_params(m, 0, "f32")
    x = W.partition_input((64, h, w), batch, 0, "f32", "normal")
    x[0, 3, 1, 1] = np.inf
    x[0, 5, 1, 6] = -np.inf
    x[0, 7, 6, 1] = np.nan
    x[0, 9, 6, 6] = 3.4e38
    outs = []
    for tuning in (None, {"gemm_plan": (9, 0, 1)}):
        with Partition(m.layers, P, (64, h, w), 0, 1, "f32", max_batch=batch,
                       tuning=tuning) as part:
            name = part.layer_info(0, batch)["kernel"]
            assert name.startswith("conv_gemm<f32" if tuning else "conv_gemm_split<")
            outs.append(gpu_forward(part, x))
    got, want = outs
    assert not np.isfinite(want).all() and np.abs(want[np.isfinite(want)]).max() > 1e36
    np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
    inf = np.isinf(want)
    np.testing.assert_array_equal(got[inf], want[inf])
    fin = np.isfinite(want)
    assert np.isfinite(got[fin]).all()
    # element by element: the huge pixel's neighbours do not hide the others
    err = np.abs(got[fin].astype(np.float64) - want[fin])
    scale = np.maximum(np.abs(want[fin]), 1.0)
    assert (err / scale).max() <= LAYER_TOL["f32"]


def test_split_static_scratch_and_graph():
    """The split kernels take no scratch: static-scratch runs, graph replays and
    direct runs give the same bits."""
    import torch
    from paper_2507_18748_amd import Partition
    m = make((32, 33, 35), [conv("c", -1, 32, 64, 3, 1, 1)])
    x = W.partition_input((32, 33, 35), 4, 0, "f32", "normal")
    with Partition(m.layers, W.model_params(m, 0, "f32"), (32, 33, 35), 0, 1, "f32",
                   max_batch=4) as part:
        a = gpu_forward(part, x)
        xd = torch.from_numpy(np.ascontiguousarray(x.transpose(0, 2, 3, 1))).cuda()
        out = torch.empty((4, 33, 35, 64), device="cuda")
        part.run_static_scratch(4, xd.data_ptr(), out.data_ptr(),
                                torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy().transpose(0, 3, 1, 2), a)
        np.testing.assert_array_equal(gpu_forward(part, x, capture=True, reps=3), a)
    ref = oracle.forward(m.layers, W.model_params(m, 0, "f32"), 0, 1, x, "f32")
    assert rel_inf(a, ref) <= LAYER_TOL["f32"]
