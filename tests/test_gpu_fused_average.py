"""cocod_average_apply_fused and the fused schedule keep up to 64 workers' rows in registers (column quads up to 32
workers, pairs above) and order their blocks and stores by where the rows start: same bits as the mean and line 6 in two
kernels, for every class of worker count, on and off the 128-byte lines, open round and blocking average."""
import numpy as np
import pytest
import torch

import paper_1906_12043_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [1, 7, 8, 9, 16, 17, 31, 32, 33, 50, 64, 65])
@pytest.mark.parametrize("extra,weighted,d", [(0, False, 5000), (4, True, 5001), (28, False, 262), (12, False, 3)])
def test_one_kernel_gives_the_bits_of_two(W, extra, weighted, d):
    dev = torch.device("cuda:0")
    stride = (d + 31) // 32 * 32 + extra
    rng = np.random.default_rng(W * 100 + d)
    data = [torch.from_numpy(rng.standard_normal((W, stride)).astype(np.float32)).to(dev) for _ in range(2)]
    data[0][0, 0], data[0][W - 1, 2] = float("inf"), float("nan")
    weights = None
    if weighted:
        p = rng.uniform(0.1, 1.0, W).astype(np.float32)
        weights = [float(v) for v in p / p.sum()]
    out = []
    for fused in (False, True):
        xA, g = data[0].clone(), data[1]
        xB, mean = torch.zeros_like(xA), torch.zeros(stride, device=dev)
        s = torch.cuda.Stream(device=dev)
        torch.cuda.synchronize()
        ctx = P.Context(W=W, d=d, stride=stride, xA=xA, xB=xB, mean=mean, lr=0.1, grad=P.GRAD_EXTERNAL, weights=weights,
                        compute_stream=s, avg_stream=s)
        ctx.average_begin()
        ctx.external_step(g)
        ctx.average_apply_fused() if fused else ctx.average_end_apply()      # x is not the stored model
        ctx.external_step(g)
        if fused:
            ctx.average_apply_fused()                                        # blocking average: it is
        else:
            ctx.average_begin()
            ctx.average_end_apply()
        ctx.sync()
        live = xA if ctx.live_model() == xA.data_ptr() else xB
        out.append([live[:, :d].cpu().view(torch.int32), mean[:d].cpu().view(torch.int32)])
        ctx.close()
    nan = [torch.isnan(t.view(torch.float32)) for t in out[0]]               # a NaN's payload is not part of the result
    for a, b, n in zip(out[0], out[1], nan):
        assert torch.equal(torch.isnan(b.view(torch.float32)), n) and torch.equal(a[~n], b[~n])


@pytest.mark.parametrize("W", [1, 8, 9, 16, 17, 32, 33, 64, 65])
@pytest.mark.parametrize("sizes,weighted", [([1], False), ([2050], True), ([3, 1023, 1026, 5, 700_001], False)])
def test_consensus_distance_of_every_worker_class(W, sizes, weighted):
    """Against 64 bits: a column's sum of W squares is formed in fp32 (each a few roundings), the rest in fp64."""
    from tests.gpu_harness import packed_positions
    d = sum(sizes)
    packed = sizes if len(sizes) > 1 else None
    stride = (P.plan_layout(d, packed)[0] + 3) // 4 * 4 + 4
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(W)
    x = rng.standard_normal((W, d)).astype(np.float32)
    pos = torch.from_numpy(packed_positions(packed, d)).to(dev)
    xA = torch.full((W, stride), 1e3, device=dev)                       # pads must not count
    xA[:, pos] = torch.from_numpy(x).to(dev)
    xB, mean, out = torch.zeros_like(xA), torch.zeros(stride, device=dev), torch.zeros(1, dtype=torch.float64, device=dev)
    p = np.full(W, 1.0 / W)
    if weighted:
        p = rng.uniform(0.1, 1.0, W).astype(np.float32)
        p = (p / p.sum()).astype(np.float32).astype(np.float64)
    s = torch.cuda.Stream(device=dev)
    torch.cuda.synchronize()
    ctx = P.Context(W=W, d=d, stride=stride, xA=xA, xB=xB, mean=mean, lr=0.1, grad=P.GRAD_EXTERNAL, tensor_numel=packed,
                    weights=[float(v) for v in p] if weighted else None, compute_stream=s, avg_stream=s)
    got = ctx.consensus_distance()
    ctx.consensus_distance_noalloc(out)
    ctx.sync()
    x64 = x.astype(np.float64)
    want = float((p[:, None] * (x64 - p @ x64) ** 2).sum())
    ctx.close()
    # W squares of a column in one fp32 chain, each with a difference that the rounded mean moves by 2^-23 of |x|
    assert abs(got - want) <= (W + 8) * 2.0**-24 * want + 2.0**-22 * float((p[:, None] * np.abs(x64) * np.abs(x64 - p @ x64)).sum()) + 1e-30
    assert got == float(out.item())
