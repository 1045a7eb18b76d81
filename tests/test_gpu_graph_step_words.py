"""The step counter of replayed rounds: a round leaves it for the next one in the other of two device words.  Any mixture of
replays, eager rounds, rounds without steps, idle steps and jumps of the counter gives the bits of eager calls."""
import numpy as np
import pytest
import torch

import paper_1906_12043_amd as P
import synth_inputs
from tests.gpu_harness import GpuMlp, GpuWorkers

pytestmark = pytest.mark.gpu
# (what, k): g = replayed round, e = eager round, s = steps outside a round, j = set the counter
SEQUENCES = [[("g", 2), ("g", 3), ("g", 2), ("e", 1), ("g", 2), ("g", 2), ("j", 40), ("g", 3), ("g", 0), ("g", 2), ("g", 2)],
             [("e", 2), ("g", 2), ("s", 3), ("g", 2), ("j", 2), ("g", 2), ("j", 0), ("g", 1), ("g", 0), ("g", 0), ("g", 1)],
             [("g", 0), ("g", 17), ("j", 0xffffff00), ("g", 17), ("g", 2), ("e", 2), ("e", 1), ("g", 2), ("j", 5), ("g", 2), ("g", 2)]]


def play(w, sequence, fused_tail, replay):
    for what, k in sequence:
        if what == "j":
            w.ctx.set_step(k)
        elif what == "s":
            w.ctx.local_steps(k)
        elif what == "g" and replay:
            w.ctx.graph_round(k, fused_tail)
        else:
            w.ctx.round_fused_tail(k) if fused_tail else w.ctx.round(k)
    w.ctx.sync()
    live = w.xA if w.ctx.live_model() == w.xA.data_ptr() else w.xB
    out = [live[:, :w.d].cpu(), w.v[:, :w.d].cpu(), w.mean[:w.d].cpu(), w.ctx.get_step()]
    w.close()
    return out


@pytest.mark.parametrize("sequence", SEQUENCES)
@pytest.mark.parametrize("schedule,fused_tail", [(P.SCHED_OVERLAP, True), (P.SCHED_OVERLAP, False), (P.SCHED_HEAD, True), (P.SCHED_SERIAL, False)])
def test_quadratic_rounds(sequence, schedule, fused_tail):
    out = []
    for replay in (False, True):
        h, c = synth_inputs.quadratic_data(8, 3, 5003)
        w = GpuWorkers(3, 5003, h=h, c=c, lr=0.05, momentum=0.9, weight_decay=5e-4, noise_sigma=0.01, seed=91)
        w.ctx.set_schedule(schedule)
        out.append(play(w, sequence, fused_tail, replay))
    assert all(torch.equal(a, b) for a, b in zip(out[0][:3], out[1][:3])) and out[0][3] == out[1][3]


@pytest.mark.parametrize("sequence", SEQUENCES[:2])
@pytest.mark.parametrize("fused_tail", [True, False])
def test_perceptron_rounds(sequence, fused_tail):
    shape = (128, 64, 3)
    theta = synth_inputs.mlp_he_init(3, *shape).astype(np.float32)
    out = [play(GpuMlp(2, shape, 128, theta, lr=0.01, momentum=0.9, weight_decay=1e-3, seed=5), sequence, fused_tail, replay)
           for replay in (False, True)]
    assert all(torch.equal(a, b) for a, b in zip(out[0][:3], out[1][:3])) and out[0][3] == out[1][3]
