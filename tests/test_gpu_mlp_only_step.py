"""A round's only step applies line 6 from the models that it has read: the bits of the step and line 6 on their own, in
64- and 128-column tiles, on and off the 128-byte lines, several rounds in a row."""
import pytest
import torch

import paper_1906_12043_amd as P
import synth_inputs
from tests.test_gpu_mlp_contractions import theta_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extra", [0, 12])
@pytest.mark.parametrize("shape,batch,W", [((128, 64, 3), 128, 3), ((512, 256, 10), 256, 3), ((1024, 192, 16), 128, 8)])
def test_round_of_one_step(shape, batch, W, extra):
    theta = theta_of(shape)
    d = synth_inputs.mlp_param_count(*shape)
    stride = (d + 31) // 32 * 32 + extra
    dev = torch.device("cuda:0")
    out = []
    for fused in (False, True):
        xA = torch.zeros((W, stride), device=dev)
        xA[:, :d] = torch.from_numpy(theta).to(dev) * torch.linspace(0.5, 1.5, W, device=dev)[:, None]
        xB, v, mean = torch.full_like(xA, float("nan")), torch.zeros_like(xA), torch.zeros(stride, device=dev)
        s = torch.cuda.Stream(device=dev)
        torch.cuda.synchronize()
        ctx = P.Context(W=W, d=d, stride=stride, xA=xA, xB=xB, v=v, mean=mean, grad=P.GRAD_MLP, mlp=(*shape, batch), lr=0.05,
                        momentum=0.9, weight_decay=1e-3, seed=9, compute_stream=s, avg_stream=torch.cuda.Stream(device=dev))
        for _ in range(3):
            ctx.round_fused_tail(1) if fused else ctx.round(1)
        ctx.sync()
        live = xA if ctx.live_model() == xA.data_ptr() else xB
        out.append([t[..., :d].cpu() for t in (live, v, mean)])
        ctx.close()
    assert all(torch.equal(a, b) for a, b in zip(*out))
