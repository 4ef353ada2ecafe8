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


def product64(x, w):
    """1x1 convolution and the sum of its terms' magnitudes, in 64 bits."""
    w = w[:, :, 0, 0].astype(np.float64)
    x = x.astype(np.float64)
    n, c, h, wd = x.shape
    flat = x.transpose(1, 0, 2, 3).reshape(c, -1)
    y, mag = w @ flat, np.abs(w) @ np.abs(flat)
    shape = (w.shape[0], n, h, wd)
    return [a.reshape(shape).transpose(1, 0, 2, 3) for a in (y, mag)]


def run_1x1(x, w):
    from paper_2507_18748_amd import Partition
    c, h, wd = x.shape[1:]
    m = make((c, h, wd), [conv("c", -1, c, w.shape[0], act="none", bn=False)])
    with Partition(m.layers, {0: {"weight": w}}, (c, h, wd), 0, 1, "f32",
                   max_batch=x.shape[0]) as part:
        assert part.layer_info(0, x.shape[0])["kernel"].startswith("conv_gemm_split<f32")
        return gpu_forward(part, x)


def split_operands(c, co, h, batch, ex=0, ew=0, seed=0):
    rng = np.random.default_rng(seed)
    x = np.ldexp(np.maximum(rng.standard_normal((batch, c, h, h)), 0), ex).astype(np.float32)
    w = np.ldexp(rng.standard_normal((co, c, 1, 1)), ew).astype(np.float32)
    return x, w


# K roundings of 2^-24 each to the sum of the terms' magnitudes bound any order
# of fp32 sums; K = 256 and random signs leave a few of them
SUM_TOL = 8 * 2.0 ** -24


@pytest.mark.parametrize("ex,ew", [(-102, 100), (-110, 100), (-118, 100), (-126, 100), (-130, 110),
                                   (-140, 110), (100, -102), (100, -110), (100, -126), (100, -140)])
@pytest.mark.parametrize("c,co,h,batch", [(256, 68, 9, 1), (288, 132, 33, 9)])
def test_split_tiny_operands(c, co, h, batch, ex, ew):
    """Operands down to the subnormals keep every bit: as accurate as others."""
    x, w = split_operands(c, co, h, batch, ex, ew)
    ref, mag = product64(x, w)
    assert (np.abs(run_1x1(x, w) - ref) <= SUM_TOL * mag).all()


def test_split_tiny_pixel():
    """A tiny pixel among ordinary ones, an exactly zero one and a filter of
    zeros: the tiny one keeps its bits."""
    x, w = split_operands(256, 64, 12, 2)
    w[5] = 0
    x[1, :, 3, 4] = np.ldexp(x[1, :, 3, 4], -130)
    x[0, :, 7, 7] = 0
    w *= np.float32(2.0 ** 100)
    ref, mag = product64(x, w)
    got = run_1x1(x, w)
    assert (np.abs(got - ref) <= SUM_TOL * mag).all()
    assert (got[:, 5] == 0).all() and (got[0, :, 7, 7] == 0).all() and (got[1, :5, 3, 4] != 0).all()


# (tile, C, Co, H, batch) of 1x1 layers, K tail of 4 in three of them
TILES_1X1 = [("32x32", 260, 68, 12, 2), ("32x64", 260, 512, 29, 1), ("64x64", 256, 260, 30, 4),
             ("64x128", 260, 260, 64, 2)]


def tile_of(c, co, h, batch):
    from paper_2507_18748_amd import Partition
    m = make((c, h, h), [conv("c", -1, c, co, act="none", bn=False)])
    with Partition(m.layers, {0: {"weight": np.zeros((co, c, 1, 1), np.float32)}}, (c, h, h), 0, 1,
                   "f32", max_batch=batch) as part:
        return part.layer_info(0, batch)["kernel"]


@pytest.mark.parametrize("tile,c,co,h,batch", TILES_1X1)
def test_split_accuracy(tile, c, co, h, batch):
    """Every plane of both operands counts.  Random terms: an error of 2^-24 of
    each product and of a few partial sums averages below 1.5e-7 of the result
    (2-norm); a plane less gives 2e-6.  Mantissas whose lower planes all have
    one sign: below three roundings of 2^-24, a plane less gives 2^-17."""
    assert tile_of(c, co, h, batch).startswith(f"conv_gemm_split<f32,{tile}> ")
    x, w = split_operands(c, co, h, batch)
    ref, _ = product64(x, w)
    assert np.linalg.norm(run_1x1(x, w) - ref) <= 1.5e-7 * np.linalg.norm(ref)
    v = np.float32(1 + 2.0 ** -8 + 2.0 ** -15 + 2.0 ** -23)
    for a, b in ((v, v), (v, 1), (1, v)):
        ref, _ = product64(np.full_like(x, a), np.full_like(w, b))
        got = run_1x1(np.full_like(x, a), np.full_like(w, b))
        assert np.abs(got / ref - 1).max() <= 3 * 2.0 ** -24


def same_as_f32(m, P, x):
    """The split kernel against the fp32 matrix instruction, non-finite values
    and element by element: both are fp32 sums of the same terms, each within
    SUM_TOL of the sum of their magnitudes."""
    from paper_2507_18748_amd import Partition
    outs = []
    for tuning in (None, {"gemm_plan": (9, 0, 1)}):
        with Partition(m.layers, P, x.shape[1:], 0, 1, "f32", max_batch=x.shape[0],
                       tuning=tuning) as part:
            name = part.layer_info(0, x.shape[0])["kernel"]
            assert name.startswith("conv_gemm<f32" if tuning else "conv_gemm_split<")
            outs.append(gpu_forward(part, x))
    got, want = outs
    np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
    np.testing.assert_array_equal(np.isinf(got), np.isinf(want))
    np.testing.assert_array_equal(got[np.isinf(want)], want[np.isinf(want)])
    fin = np.isfinite(want)
    with np.errstate(invalid="ignore"):
        mag = product64(x, P[0]["weight"])[1][fin]
    err = np.abs(got[fin].astype(np.float64) - want[fin])
    assert (err <= 2 * SUM_TOL * mag).all(), (err / mag).max()
    return want


@pytest.mark.parametrize("tile,c,co,h,batch", TILES_1X1)
def test_split_non_finite_weights(tile, c, co, h, batch):
    """Infinite, NaN and huge weights (3.4e38 rounds to an infinite bf16, 1e33
    overflows when scaled) in the first, middle and last chunk."""
    x, w = split_operands(c, co, h, batch, ew=-4)
    x[:, :, 1, 2] = 0                     # 0 * inf there
    x *= np.float32(2.0 ** -6)
    w[3, 7], w[20, c // 2], w[41, c - 1], w[66, 9] = np.inf, np.nan, 3.4e38, 1e33
    m = make((c, h, h), [conv("c", -1, c, co, act="none", bn=False)])
    want = same_as_f32(m, {0: {"weight": w}}, x)
    # (the epilogue's clamp turns NaN into -inf)
    assert (want[:, 3, 1, 2] == -np.inf).all() and (want[:, 3] == np.inf).any()
    assert (want[:, 20] == -np.inf).all() and np.isfinite(want[:, 66]).all()


@pytest.mark.parametrize("tile,c,co,h,batch", [t for t in TILES_1X1 if t[1] % 32])
def test_split_non_finite_after_tail(tile, c, co, h, batch):
    """The last chunk of 260 channels reads on into the next pixel's first ones,
    under zero weights: what is there does not reach the pixel."""
    x, w = split_operands(c, co, h, batch)
    x[0, 5, 0, 1], x[0, 20, 3, 0], x[-1, 0, h - 1, h - 1] = np.inf, np.nan, 3.4e38
    m = make((c, h, h), [conv("c", -1, c, co, act="none", bn=False)])
    want = same_as_f32(m, {0: {"weight": w}}, x)
    assert np.isfinite(want[0, :, 0, 0]).all() and np.isfinite(want[0, :, 2, h - 1]).all()
    assert not np.isfinite(want[0, :, 0, 1]).any()
