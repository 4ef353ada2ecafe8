"""Index arithmetic by multiplication: maps whose sides are 1, primes, powers of
two and one off them, in every kernel that splits a flat index into image, row
and column."""
import pytest

from test_gpu_layers import check, conv, make

pytestmark = pytest.mark.gpu

SIDES = [(1, 1), (1, 67), (61, 1), (2, 3), (16, 16), (17, 31), (33, 64), (7, 127)]


@pytest.mark.parametrize("h,w", SIDES)
@pytest.mark.parametrize("batch", [1, 5])
@pytest.mark.parametrize("s", [1, 2])
def test_index_conv(h, w, batch, s):
    # 3x3 over whole stages per tap, per-vector taps (40 channels), K splits at
    # small maps
    check(make((64, h, w), [conv("c", -1, 64, 68, 3, s, 1)]), "f16", batch)
    check(make((40, h, w), [conv("c", -1, 40, 20, 3, s, 1)]), "bf16", batch)
    check(make((256, h, w), [conv("c", -1, 256, 64, 3, s, 1)]), "f16", batch)


@pytest.mark.parametrize("h,w", SIDES)
@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_index_depthwise_and_pool(h, w, dtype):
    for s in (1, 2):
        check(make((24, h, w), [conv("d", -1, 24, 24, 3, s, 1, g=24)]), dtype, 3)
    check(make((24, h, w), [dict(name="p", op="maxpool", src=-1, c_in=24, c_out=24, k=3,
                                 stride=2, pad=1)]), dtype, 3, exact=True)
    if h > 1 and w > 1:
        check(make((24, h, w), [dict(name="p", op="maxpool", src=-1, c_in=24, c_out=24, k=2,
                                     stride=2, pad=0)]), dtype, 3, exact=True)


@pytest.mark.parametrize("cfg", [9, 11, 15, 32])
@pytest.mark.parametrize("splits", [1, 3])
def test_index_split_ranges(cfg, splits):
    """K ranges that start inside a tap row of a 3x3 window."""
    check(make((64, 13, 11), [conv("c", -1, 64, 132, 3, 1, 1)]), "f16", 7,
          tuning={"gemm_plan": (cfg, 0, splits)})
