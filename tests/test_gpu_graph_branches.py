"""Replayed rounds on either side of the size up to which the mean stays on the one branch of the graph: the bits of the same
rounds issued call by call, replay after replay."""
import numpy as np
import pytest
import torch

import paper_1906_12043_amd as P
import synth_inputs
from tests.gpu_harness import GpuMlp, GpuWorkers

pytestmark = pytest.mark.gpu
BRANCH = 16 << 20                # bytes of all models


def compare(eager, graph, k, fused_tail):
    for r in range(6):
        eager.ctx.round_fused_tail(k) if fused_tail else eager.ctx.round(k)
        if r == 3:                                       # an eager round and a synchronisation between replays
            graph.ctx.round_fused_tail(k) if fused_tail else graph.ctx.round(k)
            graph.ctx.sync()
        else:
            graph.ctx.graph_round(k, fused_tail)
    eager.ctx.sync(); graph.ctx.sync()
    assert eager.ctx.get_step() == graph.ctx.get_step() == 6 * k
    live = [w.xA if w.ctx.live_model() == w.xA.data_ptr() else w.xB for w in (eager, graph)]
    assert torch.equal(live[0][:, :eager.d], live[1][:, :eager.d])
    assert torch.equal(eager.v[:, :eager.d], graph.v[:, :eager.d]) and torch.equal(eager.mean[:eager.d], graph.mean[:eager.d])
    eager.close(); graph.close()


@pytest.mark.parametrize("k,fused_tail", [(2, True), (2, False), (18, True)])
@pytest.mark.parametrize("d", [838_860, 838_864, 1_000_003])          # W stride: one quad below, at and above the line
def test_quadratic_rounds(d, k, fused_tail):
    W = 5
    make = lambda: GpuWorkers(W, d, device_fill=True, lr=0.05, momentum=0.9, weight_decay=5e-4, noise_sigma=0.01, seed=91)
    a, b = make(), make()
    assert (W * a.stride * 4 <= BRANCH) == (d <= 838_860)
    compare(a, b, k, fused_tail)


@pytest.mark.parametrize("fused_tail", [True, False])
@pytest.mark.parametrize("shape,large", [((256, 192, 3), False), ((1024, 1152, 10), True)])
def test_perceptron_rounds(shape, large, fused_tail):
    W, batch = 4, 128
    theta = synth_inputs.mlp_he_init(3, *shape).astype(np.float32)
    make = lambda: GpuMlp(W, shape, batch, theta, lr=0.01, momentum=0.9, weight_decay=1e-3, seed=5)
    a, b = make(), make()
    assert (W * a.stride * 4 > BRANCH) == large
    compare(a, b, 2, fused_tail)
