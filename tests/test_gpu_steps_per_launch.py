"""Several local steps in one launch (built-in quadratic gradient): the same bits, in the models, the momentum, the mean and
the pads, as the same round with one launch per step, whatever the schedule and the way the round is closed."""
import numpy as np
import pytest
import torch

import paper_1906_12043_amd as P
from tests.gpu_harness import packed_positions

pytestmark = pytest.mark.gpu
HYPER = dict(lr=0.05, weight_decay=5e-4, seed=77)
SCHEDULES = [P.SCHED_OVERLAP, P.SCHED_SERIAL, P.SCHED_FUSED, P.SCHED_HEAD]
MOST = 16                        # steps of one launch


def run(W, sizes, k, call, schedule, one_by_one, extra=0, momentum=0.9, sigma=0.01, weighted=False, on_device=False):
    d = sum(sizes)
    packed = sizes if len(sizes) > 1 else None
    padded, _, _ = P.plan_layout(d, packed)
    stride = (padded + 31) // 32 * 32 + extra
    dev = torch.device("cuda:0")
    pos = torch.from_numpy(packed_positions(packed, d)).to(dev)
    gen = torch.Generator(device=dev if on_device else "cpu").manual_seed(d)

    def buf(scale):
        t = torch.full((W, stride), 7.0, device=dev)
        t[:, pos] = (scale * torch.randn((W, d), device=gen.device, generator=gen)).to(dev)
        return t
    xA, v, h, c = buf(0.5), buf(0.1), buf(1.0), buf(1.0)
    xB, mean = torch.full_like(xA, 7.0), torch.full((stride,), 7.0, device=dev)
    weights = [float(np.float32((1 + i % 3) / sum(1 + j % 3 for j in range(W)))) for i in range(W)] if weighted else None
    s = torch.cuda.Stream(device=dev)
    torch.cuda.synchronize()
    ctx = P.Context(W=W, d=d, stride=stride, xA=xA, xB=xB, v=v if momentum else None, mean=mean, h=h, c=c, momentum=momentum,
                    noise_sigma=sigma, tensor_numel=packed, weights=weights, compute_stream=s,
                    avg_stream=torch.cuda.Stream(device=dev), **HYPER)
    ctx.set_schedule(schedule)
    ctx.set_step(5)
    for _ in range(2):
        if one_by_one:
            if call != "idle":
                ctx.average_begin()
            for i in range(k):
                if call == "tail" and i == k - 1:
                    ctx.local_steps_end_apply(1)
                else:
                    ctx.local_steps(1)
            if call == "separate":
                ctx.average_end_apply()
            elif call == "idle":
                ctx.average_apply_fused()
        elif call == "tail":
            ctx.round_fused_tail(k)
        elif call == "separate":
            ctx.round(k)
        elif call == "graph":
            ctx.graph_round(k, True)
        else:
            ctx.local_steps(k)
            ctx.average_apply_fused()
    ctx.sync()
    assert ctx.get_step() == 5 + 2 * k
    live = xA if ctx.live_model() == xA.data_ptr() else xB
    out = [live.cpu(), v.cpu(), mean[pos].cpu()]
    ctx.close()
    return out


def same(got, want):
    return all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("schedule", SCHEDULES)
@pytest.mark.parametrize("call", ["tail", "separate", "graph", "idle"])
@pytest.mark.parametrize("k", [2, 3, MOST, MOST + 1, 2 * MOST + 3])
def test_one_launch_gives_the_bits_of_one_launch_per_step(k, call, schedule):
    sizes = [3, 29, 1024, 1055, 33, 2050]                          # tensors that start at every index modulo 4
    want = run(3, sizes, k, "tail" if call == "graph" else call, schedule, True)
    assert same(run(3, sizes, k, call, schedule, False), want)
    assert same(run(3, sizes, k, call, schedule, False, extra=12), [torch.nn.functional.pad(t, (0, 12), value=7.0) if t.dim() == 2 else t for t in want])


@pytest.mark.parametrize("schedule", [P.SCHED_OVERLAP, P.SCHED_HEAD])
@pytest.mark.parametrize("momentum,sigma,weighted", [(0.0, 0.01, False), (0.9, 0.0, False), (0.0, 0.0, True), (0.9, 0.01, True)])
@pytest.mark.parametrize("W", [1, 4, 17, 64])                     # one and two quads per lane of the mean-forming launches
def test_options_and_worker_counts(W, momentum, sigma, weighted, schedule):
    for d in (1, 6, 1283):
        for call in ("tail", "separate"):
            kw = dict(momentum=momentum, sigma=sigma, weighted=weighted)
            assert same(run(W, [d], 4, call, schedule, False, **kw), run(W, [d], 4, call, schedule, True, **kw)), (d, call)


@pytest.mark.parametrize("call", ["tail", "separate", "graph"])
@pytest.mark.parametrize("W,d,k", [(64, 3000, 4), (64, 70_001, 4), (64, 70_001, 8), (131, 1500, 3), (131, 1500, 8), (131, 70_001, 16),
                                   (48, 1283, 3), (48, 1283, 4), (16, 1283, 16)])
def test_mean_inside_and_apart_from_a_launch_of_several_steps(W, d, k, call):
    """Under the head schedule, with enough blocks or few enough element steps for the launch to form the mean, and with too
    few blocks for it."""
    want = run(W, [d], k, "tail" if call == "graph" else call, P.SCHED_HEAD, True)
    assert same(run(W, [d], k, call, P.SCHED_HEAD, False), want)


@pytest.mark.parametrize("call", ["tail", "separate"])
@pytest.mark.parametrize("W,d,k", [(64, 1500, 8), (131, 1500, 8), (64, 3000, 16)])
def test_one_launch_is_no_slower_than_one_launch_per_step_with_few_blocks(W, d, k, call):
    """Many workers on a short vector under the head schedule: blocks of all workers' rows would leave the chip idle (45 us
    against 37 with one launch per step at W = 64, d = 1500, k = 8 in such blocks, 9 us otherwise)."""
    dev = torch.device("cuda:0")
    stride = (d + 1023) // 1024 * 1024
    x, xB, v, h, c = [torch.zeros((W, stride), device=dev) for _ in range(5)]
    mean = torch.zeros(stride, device=dev)
    s = torch.cuda.Stream(device=dev)
    torch.cuda.synchronize()
    ctx = P.Context(W=W, d=d, stride=stride, xA=x, xB=xB, v=v, mean=mean, h=h, c=c, momentum=0.9, noise_sigma=0.01, compute_stream=s,
                    avg_stream=s, **HYPER)
    ctx.set_schedule(P.SCHED_HEAD)

    def step_by_step():
        ctx.average_begin()
        for i in range(k):
            ctx.local_steps_end_apply(1) if call == "tail" and i == k - 1 else ctx.local_steps(1)
        if call == "separate":
            ctx.average_end_apply()

    def milliseconds(body):
        times = []
        for _ in range(9):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(s)
            for _ in range(50):
                body()
            b.record(s)
            s.synchronize()
            times.append(a.elapsed_time(b))
        return sorted(times)[4]
    together = milliseconds(lambda: ctx.round_fused_tail(k) if call == "tail" else ctx.round(k))
    single = milliseconds(step_by_step)
    ctx.close()
    print("W=%d d=%d k=%d %s: %.1f us together, %.1f us step by step" % (W, d, k, call, together * 20, single * 20))
    assert together < single


@pytest.mark.parametrize("call", ["tail", "separate"])
@pytest.mark.parametrize("sizes,extra", [([3, 1_300_001, 1055, 2_750_002], 0), ([4_050_001], 12), ([34_000_003], 0)])
def test_streaming_and_panels(sizes, extra, call):
    """States above the size of the cached accesses, and a mean above the size from which line 6 goes panel by panel."""
    kw = dict(extra=extra, on_device=True)
    assert same(run(3, sizes, 3, call, P.SCHED_OVERLAP, False, **kw), run(3, sizes, 3, call, P.SCHED_OVERLAP, True, **kw))


def test_timed_steps_are_launches_of_their_own():
    dev = torch.device("cuda:0")
    t = [torch.zeros((2, 1024), device=dev) for _ in range(5)]
    s = torch.cuda.Stream(device=dev)
    torch.cuda.synchronize()
    ctx = P.Context(W=2, d=1000, stride=1024, xA=t[0], xB=t[1], v=t[2], mean=torch.zeros(1024, device=dev), h=t[3], c=t[4], momentum=0.9,
                    noise_sigma=0.01, compute_stream=s, avg_stream=s, **HYPER)
    ctx.step_timing(5)
    ctx.round_fused_tail(3)
    ctx.local_steps(6)                                               # two of them timed, the other four in one launch
    plain, tail, head = [n for _, n in ctx.step_timing_read()]
    assert (plain, tail, head) == (4, 1, 0) and ctx.get_step() == 9
    ctx.close()


def test_no_more_steps_are_timed_than_were_asked_for():
    """Armed for fewer steps than before: the event pool of the earlier call does not make it more."""
    dev = torch.device("cuda:0")
    t = [torch.zeros((2, 1024), device=dev) for _ in range(5)]
    s = torch.cuda.Stream(device=dev)
    torch.cuda.synchronize()
    ctx = P.Context(W=2, d=1000, stride=1024, xA=t[0], xB=t[1], v=t[2], mean=torch.zeros(1024, device=dev), h=t[3], c=t[4], momentum=0.9,
                    noise_sigma=0.01, compute_stream=s, avg_stream=s, **HYPER)
    ctx.step_timing(30)
    ctx.step_timing(2)
    for _ in range(2):                                               # reading rearms for two again
        ctx.local_steps(7)
        ctx.local_steps(3)
        assert [n for _, n in ctx.step_timing_read()] == [2, 0, 0]
    ctx.step_timing(0)
    ctx.local_steps(3)
    assert [n for _, n in ctx.step_timing_read()] == [0, 0, 0] and ctx.get_step() == 23
    ctx.close()
