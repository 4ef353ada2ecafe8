"""Weights read ahead by the previous launch: which launches do it, and a chain
of small layers run as one partition gives the bits of its layers run one by one
(which read nothing ahead), whatever the sizes of the weights that follow."""
import re

import numpy as np
import pytest

import workloads as W

from gpu_util import gpu_forward
from test_gpu_layers import conv, make

pytestmark = pytest.mark.gpu

# (input channels, side, layers as (C_out, k)); weight sizes with tails of less
# than a 1 KB load, over a K split and a skinny plan
CHAINS = [
    (24, 14, [(28, 1), (36, 3), (72, 1), (260, 1), (516, 1), (16, 1)]),
    (256, 14, [(256, 3), (1024, 1), (256, 1), (512, 3)]),
    # 16-bit weights of 2048, 4096 and 6144 bytes around the 4 KB limit, of 16
    # 16-bit weights of 2, 4 and 6 KB (the lower limit is 4), 8 KB below and 64 KB
    # above the upper limit of 5 MB
    (64, 7, [(64, 1), (16, 1), (64, 1), (32, 1), (48, 1), (1024, 1), (284, 3), (1024, 1), (288, 3)]),
    # two of exactly 5 MB
    (64, 7, [(1024, 1), (2560, 1), (1024, 1), (8, 1)]),
    # fp32 layers of at most 32 pixels (skinny kernel), then larger K
    (256, 3, [(256, 3), (64, 1), (516, 1), (32, 1), (260, 1)]),
    # more blocks than CUs, then fewer
    (32, 112, [(64, 1), (128, 3), (64, 1)]),
]
CUS = 256


def reads_ahead(info, nxt, w_bytes):
    """The rule: LDS-direct and skinny launches that leave CUs idle, for weights
    of 4 KB to 5 MB that a kernel reads as they are."""
    m = re.match(r"(\S+) tiles=(\d+) splits=(\d+)", info["kernel"])
    family = m[1]
    able = family.startswith("conv_gemm_skinny<") or re.match(r"conv_gemm<.*dma\d", family)
    return bool(able and int(m[2]) * int(m[3]) <= CUS and 4096 <= w_bytes <= 5 << 20 and
                not nxt["kernel"].startswith("conv_gemm_split"))


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("ci,side,layers", CHAINS)
@pytest.mark.parametrize("batch", [1, 3])
def test_prefetch_chain(dtype, ci, side, layers, batch):
    from paper_2507_18748_amd import Partition
    specs, c, sizes = [], ci, []
    esz = 4 if dtype == "f32" else 2
    for i, (co, k) in enumerate(layers):
        specs.append(conv(f"c{i}", i - 1, c, co, k, 1, k // 2))
        cpad = -(-c // (16 // esz)) * (16 // esz)
        sizes.append(co * (-(-k * k * cpad // 64) * 64) * esz)
        c = co
    m = make((ci, side, side), specs)
    P = W.model_params(m, 0, dtype)
    x = W.partition_input((ci, side, side), batch, 0, dtype, "normal")
    n = len(specs)
    with Partition(m.layers, P, (ci, side, side), 0, n, dtype, max_batch=batch) as part:
        info = [part.layer_info(i, batch) for i in range(n)]
        for i in range(n):
            want = i + 1 < n and reads_ahead(info[i], info[i + 1], sizes[i + 1])
            assert (f" ahead={i + 1}" in info[i]["kernel"]) == want, (i, info[i]["kernel"])
            assert want or "ahead" not in info[i]["kernel"]
        assert any("ahead" in k["kernel"] for k in info) or side == 112 or dtype == "f32"
        got = gpu_forward(part, x)
        np.testing.assert_array_equal(gpu_forward(part, x, capture=True, reps=2), got)
    for i in range(n):
        with Partition(m.layers, P, (ci, side, side), i, i + 1, dtype, max_batch=batch) as part:
            assert "ahead" not in part.layer_info(i, batch)["kernel"]
            x = gpu_forward(part, x)
    np.testing.assert_array_equal(got, x)


def test_prefetch_limits():
    """What the chains above are there for, in plain words."""
    from paper_2507_18748_amd import Partition

    def ahead(ci, side, layers, dtype, batch):
        specs, c = [], ci
        for i, (co, k) in enumerate(layers):
            specs.append(conv(f"c{i}", i - 1, c, co, k, 1, k // 2))
            c = co
        m = make((ci, side, side), specs)
        with Partition(m.layers, W.model_params(m, 0, dtype), (ci, side, side), 0, len(specs), dtype,
                       max_batch=batch) as part:
            return ["ahead" in part.layer_info(i, batch)["kernel"] for i in range(len(specs))]

    assert ahead(*CHAINS[2], "f16", 1) == [False, True, True, True, True, True, True, False, False]
    assert ahead(*CHAINS[4], "f32", 1) == [True, True, True, True, False]      # M = 9: no split kernel
    assert ahead(*CHAINS[5], "f16", 3) == [False, False, False]                # every CU is busy
    assert ahead(64, 14, [(64, 1), (64, 1)], "bf16", 1) == [True, False]
