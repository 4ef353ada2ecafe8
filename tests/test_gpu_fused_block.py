"""Inverted-residual blocks in one launch: the bits of the separate launches at
tile, channel-chunk and image edges, and the oracle's values."""
import numpy as np
import pytest

import workloads as W

from gpu_util import gpu_forward, rel_inf
from test_gpu_layers import conv, make

pytestmark = pytest.mark.gpu

# (C, Ce, Co, stride, pad, H, W, batch, residual, activations)
CASES = [
    (16, 96, 24, 2, 1, 33, 31, 2, False, ("relu6", "relu6", "none")),
    (24, 144, 24, 1, 1, 23, 17, 3, True, ("relu6", "relu6", "none")),   # half a last chunk
    (32, 192, 32, 1, 1, 28, 28, 4, True, ("relu6", "relu6", "none")),
    (32, 192, 64, 2, 1, 28, 27, 13, False, ("relu", "none", "relu6")),
    (8, 8, 4, 1, 1, 1, 1, 1, False, ("relu", "relu", "relu")),          # smallest
    (8, 40, 20, 1, 0, 9, 65, 2, False, ("none", "none", "none")),       # no padding, a row past a tile
    (24, 72, 36, 2, 0, 19, 18, 2, False, ("relu6", "relu", "none")),
    (8, 24, 8, 1, 2, 5, 6, 2, False, ("relu6", "relu6", "none")),       # output larger than the input
]


def block(c, ce, co, s, p, res, acts):
    return [conv("in", -1, c, c, act="none"),
            conv("e", 0, c, ce, act=acts[0]),
            conv("d", 1, ce, ce, 3, s, p, g=ce, act=acts[1]),
            conv("p", 2, ce, co, act=acts[2], res=0 if res else -1),
            conv("out", 3, co, 16, act="none")]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("c,ce,co,s,p,h,w,batch,res,acts", CASES)
def test_fused_block(dtype, c, ce, co, s, p, h, w, batch, res, acts):
    import oracle
    from paper_2507_18748_amd import Partition
    m = make((c, h, w), block(c, ce, co, s, p, res, acts))
    P = W.model_params(m, 0, dtype)
    x = W.partition_input((c, h, w), batch, 0, dtype, "normal")
    outs = {}
    # the block in the middle of a partition, and as the whole of one
    for begin, end in ((0, 5), (1, 4)) if not res else ((0, 5), (0, 4)):
        for tuning in (None, {"no_pair": 1}):
            with Partition(m.layers, P, (c, h, w), begin, end, dtype, max_batch=batch,
                           tuning=tuning) as part:
                names = [part.layer_info(i, batch)["kernel"] for i in (1, 2, 3)]
                assert all(("fused=1-3" in n) == (tuning is None) for n in names), names
                a = gpu_forward(part, x)
                if tuning is None:
                    np.testing.assert_array_equal(gpu_forward(part, x, capture=True, reps=3), a)
            outs[begin, end, tuning is None] = a
        np.testing.assert_array_equal(outs[begin, end, True], outs[begin, end, False])
    # three roundings to the storage type between input and output
    begin, end = (1, 4) if not res else (0, 4)
    ref = oracle.forward(m.layers, P, begin, end, x, dtype)
    assert rel_inf(outs[begin, end, True].reshape(ref.shape), ref) <= \
        4 * {"f16": 2.0 ** -9, "bf16": 2.0 ** -7}[dtype]


def test_not_fused():
    """Blocks outside the kernel's limits, or whose inner maps have another
    reader, keep their launches."""
    from paper_2507_18748_amd import Partition
    for specs, h in (
            (block(40, 96, 24, 1, 1, False, ("relu",) * 3), 9),       # C > 32
            (block(32, 200, 24, 1, 1, False, ("relu",) * 3), 9),      # Ce > 192
            (block(32, 96, 68, 1, 1, False, ("relu",) * 3), 9),       # Co > 64
            (block(32, 32, 32, 1, 1, False, ("relu",) * 3)[:4] +
             [conv("out", 3, 32, 32, act="none", res=1)], 9)):        # the expanded map read again
        c = specs[0]["c_in"]
        m = make((c, h, h), specs)
        with Partition(m.layers, W.model_params(m, 0, "f16"), (c, h, h), 0, 5, "f16",
                       max_batch=2) as part:
            assert not any("fused" in part.layer_info(i, 2)["kernel"] for i in range(5))


@pytest.mark.parametrize("offset", ["before", "after", "inside"])
@pytest.mark.parametrize("capture", [False, True])
def test_overlapping_buffers(offset, capture):
    """A partition that is one block, its output written over part of its input:
    the input is read whole first.  The same pointer twice stays refused."""
    import torch
    from paper_2507_18748_amd import Partition, PpipeError
    n, c, h, w = 2, 24, 40, 36
    m = make((c, h, w), block(c, 72, c, 1, 1, False, ("relu6", "relu6", "none"))[1:4])
    for i, L in enumerate(m.layers):
        L.src = i - 1
    P = W.model_params(m, 0, "f16")
    x = W.partition_input((c, h, w), n, 0, "f16", "normal")
    nb = n * c * h * w
    with Partition(m.layers, P, (c, h, w), 0, 3, "f16", max_batch=n) as part:
        assert "fused=0-2" in part.layer_info(0, n)["kernel"]
        want = gpu_forward(part, x)
        buf = torch.zeros(3 * nb, dtype=torch.float16, device="cuda")
        xin, k = buf[nb:2 * nb], {"before": nb - 48 * w, "after": nb + 48 * w, "inside": nb + 8}[offset]
        out = buf[k:k + nb]
        xin.copy_(torch.from_numpy(x.transpose(0, 2, 3, 1).reshape(-1)).half())
        if capture:
            part.capture(n, xin.data_ptr(), out.data_ptr())
        part.run(n, xin.data_ptr(), out.data_ptr(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        got = out.reshape(n, h, w, c).float().cpu().numpy().transpose(0, 3, 1, 2)
        np.testing.assert_array_equal(got, want)
        with pytest.raises(PpipeError):
            part.run(n, xin.data_ptr(), xin.data_ptr(), 0)


def test_timed_runs_issue_the_served_launches():
    """One record for a block, at its first layer, with the work of the three;
    the layer table's shares add up to its launch.  With buffers that share
    bytes a lone block is timed as its three launches."""
    import torch
    from paper_2507_18748_amd import Partition
    n, c, h, w = 4, 24, 56, 56
    m = make((c, h, w), block(c, 144, c, 1, 1, True, ("relu6", "relu6", "none")))
    P = W.model_params(m, 0, "bf16")
    x = W.partition_input((c, h, w), n, 0, "bf16", "normal")
    with Partition(m.layers, P, (c, h, w), 0, 5, "bf16", max_batch=n) as part:
        info = [part.layer_info(i, n) for i in range(5)]
        assert [i["kernel_count"] for i in info] == [1, 1, 0, 0, 1]
        want = gpu_forward(part, x)
        xd = torch.from_numpy(x.transpose(0, 2, 3, 1).copy()).bfloat16().cuda()
        out = torch.zeros((n, h, w, 16), dtype=torch.bfloat16, device="cuda")
        part.timing_setup(n, xd.data_ptr(), out.data_ptr())
        part.run_timed(torch.cuda.current_stream().cuda_stream)
        recs = part.timing_read()
        np.testing.assert_array_equal(out.float().cpu().numpy().transpose(0, 3, 1, 2), want)
        for r in (recs, part.profile_kernels(n, 1, 2),
                  part.profile_kernels_cold(n, reps=1, sweep_bytes=64 << 20)):
            assert [(k["layer"], k["launch"]) for k in r] == [(0, 0), (1, 0), (4, 0)]
            assert r[1]["kernel"] == "fused_block<bf16,s1>" and r[1]["mean_us"] > 0
            assert r[1]["flops"] == n * sum(i["flops_b1"] for i in info[1:4])
            maps = n * 3 * c * h * w * 2                        # input, residual, output
            assert r[1]["bytes"] == maps + sum(i["param_bytes"] for i in info[1:4])
        table, whole = part.profile_layers([1, n], warmup=2, reps=5)
        assert (table > 0).all()
        share = [i["flops_b1"] / sum(k["flops_b1"] for k in info[1:4]) for i in info[1:4]]
        np.testing.assert_allclose(table[1:4, 1] / table[1:4, 1].sum(), share, rtol=1e-5)
    lone = make((c, h, w), block(c, 72, c, 1, 1, False, ("relu6", "relu6", "none"))[1:4])
    for i, L in enumerate(lone.layers):
        L.src = i - 1
    with Partition(lone.layers, W.model_params(lone, 0, "bf16"), (c, h, w), 0, 3, "bf16",
                   max_batch=n) as part:
        buf = torch.zeros(2 * n * c * h * w, dtype=torch.bfloat16, device="cuda")
        part.timing_setup(n, buf.data_ptr(), buf[8:].data_ptr())
        part.run_timed(torch.cuda.current_stream().cuda_stream)
        recs = part.timing_read()
        assert [r["layer"] for r in recs] == [0, 1, 2] and all(r["mean_us"] > 0 for r in recs)
        assert not any("fused" in r["kernel"] for r in recs)


# (C, Ce, Co, stride, side, batch, one launch): both sides of every line of the
# dispatch rule
RULE = [
    (24, 192, 24, 1, 14, 1, True),        # stride 1: any length
    (24, 160, 24, 2, 14, 1, True),        # stride 2: five chunks, few outputs
    (24, 128, 64, 2, 14, 1, True),
    (24, 136, 64, 2, 14, 1, False),       # five chunks and more than 32 outputs: from 4000 pixels
    (24, 136, 64, 2, 64, 1, True),
    (24, 168, 24, 2, 40, 4, False),       # six chunks: from 8000
    (24, 168, 24, 2, 40, 5, True),
    (8, 16, 16, 1, 112, 31, True),        # few expanded channels: below 24 tiles per CU
    (8, 16, 16, 1, 112, 32, False),
    (8, 24, 16, 1, 112, 32, True),
    (8, 24, 20, 1, 112, 32, False),
    (8, 32, 20, 1, 112, 32, True),
    (8, 72, 48, 1, 112, 32, True),
    (8, 72, 52, 1, 112, 32, False),       # many outputs of few channels, maps within 350 MB
    (8, 80, 52, 1, 112, 32, True),
    (8, 72, 52, 1, 112, 64, False),
    (16, 72, 52, 1, 128, 64, True),
]


@pytest.mark.parametrize("c,ce,co,s,side,batch,on", RULE)
def test_dispatch_rule(c, ce, co, s, side, batch, on):
    from paper_2507_18748_amd import Partition
    m = make((c, side, side), block(c, ce, co, s, 1, False, ("relu6", "relu6", "none"))[1:4])
    for i, L in enumerate(m.layers):
        L.src = i - 1
    with Partition(m.layers, W.model_params(m, 0, "bf16"), (c, side, side), 0, 3, "bf16",
                   max_batch=batch) as part:
        assert ("fused=0-2" in part.layer_info(0, batch)["kernel"]) == on


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("acts", [("relu6", "relu6", "none"), ("none", "none", "none")])
@pytest.mark.parametrize("ce,s", [(72, 1), (40, 2)])      # part-filled last chunks
def test_non_finite_inputs(dtype, acts, ce, s):
    """Infinities, NaN and the type's largest values in the input and the residual:
    the bits of the separate launches, and pixels out of their reach stay finite."""
    from paper_2507_18748_amd import Partition
    n, c, h, w = 2, 24, 13, 19
    m = make((c, h, w), block(c, ce, c, s, 1, s == 1, acts))
    P = W.model_params(m, 0, dtype)
    x = W.partition_input((c, h, w), n, 0, dtype, "normal")
    big = 65504.0 if dtype == "f16" else 3.38e38
    x[0, 0, 0, 0], x[0, 5, 6, 7], x[0, 23, 12, 18] = np.inf, -np.inf, np.nan
    x[1, 3, 4, 4], x[1, 4, 4, 5], x[1, 9, 12, 0] = big, -big, np.inf
    outs = []
    for tuning in (None, {"no_pair": 1}):
        with Partition(m.layers, P, (c, h, w), 0, 5, dtype, max_batch=n, tuning=tuning) as part:
            assert ("fused=1-3" in part.layer_info(1, n)["kernel"]) == (tuning is None)
            outs.append(gpu_forward(part, x))
    assert np.isfinite(outs[1][:, :, 2 // s, 12 // s]).all()
    assert acts[0] == "relu6" or not np.isfinite(outs[1]).all()   # (relu6 bounds every value)
    np.testing.assert_array_equal(outs[0], outs[1])
