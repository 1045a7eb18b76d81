"""The step kernel moves a worker's tiles to the 128-byte lines of its row: for every distance of the rows from a line,
every kind of step and every gradient the bits are those of rows that lie on lines, and pads stay untouched."""
import numpy as np
import pytest
import torch

import paper_1906_12043_amd as P
from tests.gpu_harness import one_round, packed_positions

pytestmark = pytest.mark.gpu
W = 3
HYPER = dict(lr=0.05, weight_decay=5e-4, noise_sigma=0.01, seed=77)


def rounds(sizes, extra, momentum, kind, on_device=False):
    """(x, v, mean) of the real parameters after rounds of every kind; models, h, c drawn by parameter index (large ones
    on the device)."""
    d = sum(sizes)
    packed = sizes if len(sizes) > 1 else None
    padded, _, _ = P.plan_layout(d, packed)
    stride = (padded + 31) // 32 * 32 + extra
    dev = torch.device("cuda:0")
    pos = torch.from_numpy(packed_positions(packed, d)).to(dev)
    rng = np.random.default_rng(d)
    gen = torch.Generator(device=dev).manual_seed(d)

    def buf(scale, fill=7.0):
        t = torch.full((W, stride), fill, device=dev)
        if on_device:
            t[:, pos] = scale * torch.randn((W, d), device=dev, generator=gen)
        else:
            t[:, pos] = torch.from_numpy((scale * rng.standard_normal((W, d))).astype(np.float32)).to(dev)
        return t
    xA, v, h, c = buf(0.5), buf(0.1), buf(1.0), buf(1.0)
    xB, mean = torch.full_like(xA, 7.0), torch.zeros(stride, device=dev)
    g16 = h.to(torch.bfloat16)
    s = torch.cuda.Stream(device=dev)
    torch.cuda.synchronize()
    ctx = P.Context(W=W, d=d, stride=stride, xA=xA, xB=xB, v=v if momentum else None, mean=mean, h=h, c=c, momentum=momentum,
                    tensor_numel=packed, compute_stream=s, avg_stream=s, **HYPER)
    if kind == "round":
        ctx.round(2)                                 # plain steps in one launch, line 6 alone
        one_round(ctx, 2, False, True)               # plain steps, out of place and in place
        ctx.round_fused_tail(2)                      # line 6 inside the only launch
        one_round(ctx, 2, True, True)                # line 6 inside the last step
        ctx.round_fused_tail(1)                      # line 6 inside the only step
    else:
        step, g = (ctx.external_step, h) if kind == "fp32" else (ctx.external_step_bf16, g16)
        for k in (2, 1):
            ctx.average_begin()
            for i in range(k):
                step(g, close_round=(i == k - 1))
    ctx.sync()
    live = xA if ctx.live_model() == xA.data_ptr() else xB
    real = torch.zeros(stride, dtype=torch.bool, device=dev)
    real[pos] = True
    tail_quad = torch.zeros(stride, dtype=torch.bool, device=dev)       # pads that share a tensor's last quad travel along
    tail_quad[pos // 4 * 4 + 3] = tail_quad[pos // 4 * 4 + 2] = tail_quad[pos // 4 * 4 + 1] = True
    for t in (xA, xB, v):
        assert bool((t[:, ~real & ~tail_quad] == 7.0).all())
    out = [live[:, pos].cpu(), v[:, pos].cpu(), mean[pos].cpu()]
    ctx.close()
    return out


@pytest.mark.parametrize("sizes", [[1], [27], [30], [255], [257], [283], [1024], [1025], [1051], [2077], [5000],
                                   [3, 29, 1024, 1055, 33, 2048], [1, 1, 6, 5000, 1020]])
@pytest.mark.parametrize("kind,momentum", [("round", 0.9), ("round", 0.0), ("fp32", 0.9), ("bf16", 0.9)])
def test_rows_off_the_lines_give_the_same_bits(sizes, kind, momentum):
    want = rounds(sizes, 0, momentum, kind)
    for extra in (4, 8, 16, 28):                     # three workers: leads of 0, -extra and -2 extra modulo 32
        got = rounds(sizes, extra, momentum, kind)
        assert all(torch.equal(a, b) for a, b in zip(got, want)), extra


CACHED_STATE = 224 << 20         # up to here (five arrays) the steps run without the streaming hint
PANEL_MEAN = 128 << 20           # above, the blocks of a line-6 step run in panels


@pytest.mark.parametrize("kind,momentum", [("round", 0.9), ("round", 0.0), ("fp32", 0.9), ("bf16", 0.9)])
def test_large_states_off_the_lines_give_the_same_bits(kind, momentum):
    """The same above the size up to which the steps do without the streaming hint: the other instantiations."""
    sizes = [3, 29, 1_300_001, 1055, 33, 2_750_002]
    assert 20 * W * sum(sizes) > CACHED_STATE
    want = rounds(sizes, 0, momentum, kind, on_device=True)
    got = rounds(sizes, 12, momentum, kind, on_device=True)
    assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("kind", ["round", "fp32"])
def test_panels_off_the_lines_give_the_same_bits(kind):
    """A mean above the size from which line 6, alone or in a step, takes its tiles panel by panel (a short last panel)."""
    sizes = [34_000_003]
    assert 4 * sum(sizes) > PANEL_MEAN and sum(sizes) // 256 % 16384 != 0
    want = rounds(sizes, 0, 0.9, kind, on_device=True)
    got = rounds(sizes, 20, 0.9, kind, on_device=True)
    assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("workers", [3, 8, 17])
@pytest.mark.parametrize("d", [5, 1025, 9000, 70_001])
def test_mean_forming_steps_off_the_lines_give_the_same_bits(workers, d):
    """Off the lines these steps take their tiles XCD by XCD, with another store policy; tiles in numbers that do and do
    not divide by the eight dies, k = 1 and 2 in one pass and k = 2 with the mean in the first step."""
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(d)
    base = [torch.from_numpy(rng.standard_normal((workers, d)).astype(np.float32)).to(dev) for _ in range(4)]
    want = None
    for extra in (0, 4, 20):
        stride = (d + 31) // 32 * 32 + extra
        xA, v, h, c = [torch.zeros((workers, stride), device=dev) for _ in range(4)]
        for t, src in zip((xA, v, h, c), base):
            t[:, :d] = src
        xB, mean = torch.zeros_like(xA), torch.zeros(stride, device=dev)
        s = torch.cuda.Stream(device=dev)
        torch.cuda.synchronize()
        ctx = P.Context(W=workers, d=d, stride=stride, xA=xA, xB=xB, v=v, mean=mean, h=h, c=c, momentum=0.9, compute_stream=s,
                        avg_stream=s, **HYPER)
        ctx.set_schedule(P.SCHED_HEAD)
        ctx.round_fused_tail(1)
        ctx.round_fused_tail(2)
        one_round(ctx, 2, True, True)
        ctx.sync()
        live = xA if ctx.live_model() == xA.data_ptr() else xB
        got = [live[:, :d].cpu(), v[:, :d].cpu(), mean[:d].cpu()]
        ctx.close()
        if want is None:
            want = got
        assert all(torch.equal(a, b) for a, b in zip(got, want)), extra
