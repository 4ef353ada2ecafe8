"""The three-way bf16 split of fp32 operands, emulated on the CPU: exact for
every finite value once scaled into the bf16 range, and the partial products
that the kernels leave out stay below one fp32 rounding of the product."""
import numpy as np
import torch


def bf16(x):
    return torch.from_numpy(np.ascontiguousarray(x)).bfloat16().float().numpy()


def planes(x):
    x0 = bf16(x)
    r = x - x0
    x1 = bf16(r)
    return x0, x1, r - x1


def left_out(x, w):
    """x1 w2 + x2 w1 + x2 w2 over x w."""
    a, b = ([p.astype(np.float64) for p in planes(v)] for v in (x, w))
    return np.abs(a[1] * b[2] + a[2] * b[1] + a[2] * b[2]) / np.abs(x.astype(np.float64) * w)


def mantissas(n, seed):
    rng = np.random.default_rng(seed)
    return (1 + rng.integers(0, 2 ** 23, n) * 2.0 ** -23).astype(np.float32)


def test_split_is_exact():
    # weights: any bits below 2^103, subnormals among them, times 2^24
    bits = np.random.default_rng(0).integers(0, (127 + 103) << 23, 1 << 20, dtype=np.uint32)
    w = bits.view(np.float32) * np.float32(2.0 ** 24)
    tiny = (bits & 0x7fffff).view(np.float32) * np.float32(2.0 ** 24)   # subnormals only
    # activations as they are, from 2^-102 on
    x = bits[bits >= (127 - 102) << 23].view(np.float32)
    for v in (w, tiny, x, -x):
        p = planes(v)
        np.testing.assert_array_equal(sum(q.astype(np.float64) for q in p), v)
        for q in p:
            np.testing.assert_array_equal(bf16(q), q)              # fits a bf16
            assert (np.abs(q[q != 0]) >= 2.0 ** -126).all()        # and is a normal one


def test_left_out_terms_stay_below_one_rounding():
    worst = np.float32([1 + 2.0 ** -8 - 2.0 ** -17])
    assert 2.0 ** -25 < left_out(worst, worst)[0] < 2.0 ** -24
    d = left_out(mantissas(1 << 20, 1), mantissas(1 << 20, 2))
    assert d.max() < 2.0 ** -24 and d.mean() < 2.0 ** -28


def test_products_that_fit_fp32_are_whole():
    # up to 24 significant bits between the two operands
    rng = np.random.default_rng(3)
    for nx in range(1, 24):
        x = rng.integers(2 ** (nx - 1), 2 ** nx, 4096).astype(np.float32)
        w = rng.integers(2 ** (23 - nx), 2 ** (24 - nx), 4096).astype(np.float32)
        assert left_out(x, w).max() == 0
