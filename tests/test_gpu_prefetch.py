"""Weights read ahead by the previous launch: a chain of small layers run as one
partition gives the bits of its layers run one by one (which read nothing
ahead), whatever the sizes of the weights that follow."""
import numpy as np
import pytest

import workloads as W

from gpu_util import gpu_forward
from test_gpu_layers import conv, make

pytestmark = pytest.mark.gpu

# (input channels, layers as (C_out, k)); weight sizes below, at and above the
# 4 KB limit, with tails of less than a 1 KB load, over a K split and a skinny
# plan, and a classifier at the end
CHAINS = [
    (24, [(28, 1), (36, 3), (72, 1), (260, 1), (516, 1), (16, 1)]),
    (256, [(256, 3), (1024, 1), (256, 1), (512, 3)]),
]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("ci,layers", CHAINS)
@pytest.mark.parametrize("batch", [1, 3])
def test_prefetch_chain(dtype, ci, layers, batch):
    from paper_2507_18748_amd import Partition
    specs, c = [], ci
    for i, (co, k) in enumerate(layers):
        specs.append(conv(f"c{i}", i - 1, c, co, k, 1, k // 2))
        c = co
    m = make((ci, 14, 14), specs)
    P = W.model_params(m, 0, dtype)
    x = W.partition_input((ci, 14, 14), batch, 0, dtype, "normal")
    n = len(specs)
    with Partition(m.layers, P, (ci, 14, 14), 0, n, dtype, max_batch=batch) as part:
        got = gpu_forward(part, x)
        np.testing.assert_array_equal(gpu_forward(part, x, capture=True, reps=2), got)
    for i in range(n):
        with Partition(m.layers, P, (ci, 14, 14), i, i + 1, dtype, max_batch=batch) as part:
            x = gpu_forward(part, x)
    np.testing.assert_array_equal(got, x)
