"""The perceptron workers' two big contractions (three bf16 planes per operand on the matrix cores, at fp32 accuracy) at
the sizes and values where their splitting, range, K splits, tiles and chunks can go wrong, against 64 bits on the device's
own operands."""
import numpy as np
import pytest
import torch

import paper_1906_12043_amd as P
import synth_inputs
from tests.gpu_harness import GpuMlp

pytestmark = pytest.mark.gpu
HYPER = dict(lr=0.05, momentum=0.9, weight_decay=0.0, seed=0x5EED0009)


def theta_of(shape, seed=3):
    theta = synth_inputs.mlp_he_init(seed, *shape).astype(np.float64)
    theta += 0.05 * np.random.default_rng(seed).standard_normal(theta.size)
    return theta.astype(np.float32)


def one_step(W, shape, batch, theta):
    """(work space, v) of one step from v = 0 and weight decay 0: v is then the gradient itself."""
    g = GpuMlp(W, shape, batch, theta, **HYPER)
    g.ctx.local_steps(1)
    ws, v, x = g.workspace(), g.vel(), g.x()
    g.close()
    return ws, v, x


def bound(K, a, b):
    """Largest error of an element of a @ b.  Every operand is split exactly (8 + 8 + 8 bits); the partial products left out
    are at most 2^-24 of the product; K / 16 sums of 16 leading products are rounded to fp32, each a few times inside, 5 K / 16
    sums of small ones (2^-7 of the leading ones) likewise; the two are added once."""
    return 2.0**-24 * (2 + 4 * K / 16 * (1 + 5 * 2.0**-7)) * (np.abs(a) @ np.abs(b))


# one and several K splits; 64- and 128-column tiles; one and several m-tiles; a hidden layer that passes through the
# output kernel's LDS in two chunks (the second one short); every octet of classes
@pytest.mark.parametrize("W,shape,batch", [(1, (128, 64, 1), 128), (2, (384, 192, 4), 256), (3, (1024, 128, 5), 128),
                                           (1, (256, 2176, 10), 384), (2, (640, 320, 16), 1024), (5, (2048, 256, 9), 128)])
def test_contractions_and_small_gradients_against_64_bits(W, shape, batch):
    n_in, n_hidden, n_out = shape
    theta = theta_of(shape)
    ws, v, _ = one_step(W, shape, batch, theta)
    th = theta.astype(np.float64)
    a, b, c = n_in * n_hidden, n_in * n_hidden + n_hidden, n_in * n_hidden + n_hidden + n_hidden * n_out
    W1, b1, W2 = th[:a].reshape(n_in, n_hidden), th[a:b], th[b:c].reshape(n_hidden, n_out)
    for i in range(W):
        X, H, dA, dZ = ws["X"][i], ws["H"][i], ws["dA"][i], ws["dZ"][i]
        H64 = np.maximum(X @ W1 + b1, 0)
        assert np.all(np.abs(H - H64) <= bound(n_in, X, W1) + 2.0**-22 * (np.abs(b1) + np.abs(H64)))
        # four sums of up to four products, two roundings each (largest seen 6.4 x 2^-24, at 16 classes)
        assert np.all(np.abs(dA - np.where(H > 0, dZ @ W2.T, 0)) <= 2.0**-21 * (np.abs(dZ) @ np.abs(W2.T)))
        assert np.all(np.abs(v[i, :a].reshape(n_in, n_hidden) - X.T @ dA) <= bound(batch, X.T, dA))
        small = (batch + 8) * 2.0**-24                       # a chain of fp32 additions over the batch
        assert np.all(np.abs(v[i, a:b] - dA.sum(0)) <= small * np.abs(dA).sum(0))
        assert np.all(np.abs(v[i, b:c].reshape(n_hidden, n_out) - H.T @ dZ) <= small * (np.abs(H.T) @ np.abs(dZ)))
        assert np.all(np.abs(v[i, c:] - dZ.sum(0)) <= small * np.abs(dZ).sum(0))


@pytest.mark.parametrize("scale", [1e-30, 1e-12, 1e12])
def test_weights_of_any_magnitude(scale):
    """A worker's W1 far from 1 (bias 0, so that H shows the product itself)."""
    W, shape, batch = 1, (512, 128, 3), 128
    theta = theta_of(shape)
    a = shape[0] * shape[1]
    theta[:a] *= np.float32(scale)
    theta[a:a + shape[1]] = 0
    ws, _, _ = one_step(W, shape, batch, theta)
    W1 = theta[:a].astype(np.float64).reshape(shape[0], shape[1])
    X = ws["X"][0]
    assert np.all(np.abs(ws["H"][0] - np.maximum(X @ W1, 0)) <= bound(shape[0], X, W1))


def test_columns_that_outgrow_their_first_rows():
    """A column that grows a millionfold after its first rows, one whose first rows are zero and one that is zero throughout
    are exact to the bound."""
    W, shape, batch = 1, (512, 256, 3), 128
    theta = theta_of(shape)
    a = shape[0] * shape[1]
    W1 = theta[:a].reshape(shape[0], shape[1])
    W1[40:, 5] *= 1e6
    W1[:64, 70] = 0
    W1[:, 131] = 0
    theta[a:a + shape[1]] = 0
    ws, _, _ = one_step(W, shape, batch, theta)
    X, W64 = ws["X"][0], W1.astype(np.float64)
    assert np.all(np.abs(ws["H"][0] - np.maximum(X @ W64, 0)) <= bound(shape[0], X, W64))


def test_infinities_and_nan_in_the_weights_go_where_fp32_takes_them():
    """An infinite weight makes its column's pre-activation +-inf by the sign of the input (0 or inf after the relu), a
    NaN weight makes it NaN (0 after the relu's maximum); the other columns are untouched."""
    W, shape, batch = 1, (256, 128, 3), 128
    clean = theta_of(shape)
    a = shape[0] * shape[1]
    theta = clean.copy()
    W1 = theta[:a].reshape(shape[0], shape[1])
    W1[7, 3], W1[200, 9], W1[100, 64] = np.inf, -np.inf, np.nan
    ws, _, _ = one_step(W, shape, batch, theta)
    X, H = ws["X"][0], ws["H"][0]
    assert np.array_equal(H[:, 3], np.where(X[:, 7] > 0, np.inf, 0)) and np.array_equal(H[:, 9], np.where(X[:, 200] < 0, np.inf, 0))
    assert np.all(H[:, 64] == 0)
    rest = [n for n in range(shape[1]) if n not in (3, 9, 64)]
    C1 = clean[:a].astype(np.float64).reshape(shape[0], shape[1])[:, rest]
    b1 = clean[a:a + shape[1]].astype(np.float64)[rest]
    assert np.all(np.abs(H[:, rest] - np.maximum(X @ C1 + b1, 0)) <= bound(shape[0], X, C1) + 2.0**-21 * (1 + np.abs(b1)))


def scale_rows(factors):
    def change(W1, W2):
        W2 *= factors(len(W2))[:, None].astype(np.float32)
    return change


@pytest.mark.parametrize("change", [scale_rows(lambda n: 2.0 ** (-45 * np.arange(n) / (n - 1))),      # rows of W2 over 2^-45 .. 1
                                    scale_rows(lambda n: np.where(np.arange(n) == 7, 1e8, 1.0)),       # one row above the others
                                    scale_rows(lambda n: np.full(n, 1e-34))])                          # near the smallest numbers
def test_every_column_of_the_gradient_has_its_own_accuracy(change):
    """W2 is the caller's and sets the columns of dA: the gradient of a column must not lose bits to a larger one."""
    W, shape, batch = 1, (256, 128, 10), 128
    theta = theta_of(shape)
    a, b, c = 256 * 128, 256 * 128 + 128, 256 * 128 + 128 + 128 * 10
    change(theta[:a].reshape(256, 128), theta[b:c].reshape(128, 10))
    ws, v, _ = one_step(W, shape, batch, theta)
    X, dA = ws["X"][0], ws["dA"][0]
    assert (np.abs(dA).max(0) > 0).sum() > 100
    assert np.all(np.abs(v[0, :a].reshape(256, 128) - X.T @ dA) <= bound(batch, X.T, dA))


def test_sums_of_one_term_are_products_of_whole_operands():
    """A column of W1 with one entry that is not zero, and units that are active on a few samples: no sum hides what an
    operand has lost.  One term: 2^-24 left out, 2^-24 for adding the small products, the last place of the fp32 result."""
    W, shape, batch = 2, (512, 256, 10), 128
    n_in, n_hidden, n_out = shape
    theta = theta_of(shape)
    a = n_in * n_hidden
    W1 = theta[:a].reshape(n_in, n_hidden)
    w = W1[2 * np.arange(n_hidden), np.arange(n_hidden)].copy()
    W1[:] = 0
    W1[2 * np.arange(n_hidden), np.arange(n_hidden)] = w
    theta[a:a + n_hidden] = 0
    ws, _, _ = one_step(W, shape, batch, theta)
    for i in range(W):
        exact = ws["X"][i][:, ::2] * w.astype(np.float64)
        assert np.all(np.abs(ws["H"][i] - np.maximum(exact, 0)) <= 2.1 * 2.0**-24 * np.abs(exact))
    theta = theta_of(shape)
    norm = np.sqrt((theta[:a].astype(np.float64).reshape(n_in, n_hidden) ** 2).sum(0))
    theta[a:a + n_hidden] = (-2.2 * norm).astype(np.float32)
    ws, v, _ = one_step(W, shape, batch, theta)
    for i in range(W):
        X, dA = ws["X"][i], ws["dA"][i]
        assert np.median((dA != 0).sum(0)) <= 4
        assert np.all(np.abs(v[i, :a].reshape(n_in, n_hidden) - X.T @ dA) <= bound(8, X.T, dA))


@pytest.mark.parametrize("which,scale", [("W1", 1e36), ("W1", 1e25), ("W1", 1e-37), ("W2", 1e36), ("W2", 1e25)])
def test_operands_at_the_ends_of_the_range(which, scale):
    """Beyond 2^104 the planes overflow and the tile is formed with fp32 products: n terms, n / 2 roundings of 2 each."""
    W, shape, batch = 1, (256, 192, 4), 128
    n_in, n_hidden, n_out = shape
    theta = theta_of(shape)
    a, b, c = n_in * n_hidden, n_in * n_hidden + n_hidden, n_in * n_hidden + n_hidden + n_hidden * n_out
    if which == "W1":
        theta[:a] *= np.float32(scale)
        theta[a:b] = 0
    else:
        theta[b:c] *= np.float32(scale)
    ws, v, _ = one_step(W, shape, batch, theta)
    X, dA, W1 = ws["X"][0], ws["dA"][0], theta[:a].astype(np.float64).reshape(n_in, n_hidden)
    if which == "W1":
        assert np.all(np.abs(ws["H"][0] - np.maximum(X @ W1, 0)) <= 2.0**-24 * (n_in + 8) * (np.abs(X) @ np.abs(W1)))
    assert np.isfinite(dA).all() and np.abs(dA).max() > 0
    assert np.all(np.abs(v[0, :a].reshape(n_in, n_hidden) - X.T @ dA) <= 2.0**-24 * (batch + 8) * (np.abs(X.T) @ np.abs(dA)))


def test_an_infinity_in_dA_leaves_the_other_columns_their_gradient():
    """W2 = -inf at a unit that is active on every sample: its class never occurs (probability 0), the unit's column of
    dA is inf where the class is the label and NaN elsewhere, every other dA is an ordinary number and so is its column
    of the gradient of W1, in the tile of the infinite column and in the others."""
    W, shape, batch = 1, (256, 384, 3), 128
    n_in, n_hidden, n_out = shape
    theta = theta_of(shape)
    a, b = n_in * n_hidden, n_in * n_hidden + n_hidden
    theta[a + 200] = 1e3                                         # active on every sample
    theta[b + 200 * n_out + 1] = -np.inf
    ws, v, _ = one_step(W, shape, batch, theta)
    X, dA = ws["X"][0], ws["dA"][0]
    assert np.isinf(dA[:, 200]).any() and np.isnan(dA[:, 200]).any()
    rest = np.arange(n_hidden) != 200
    assert np.isfinite(dA[:, rest]).all() and np.abs(dA[:, rest]).max() > 0
    dW1 = v[0, :a].reshape(n_in, n_hidden)
    assert np.isnan(dW1[:, 200]).all()
    assert np.all(np.abs(dW1[:, rest] - X.T @ dA[:, rest]) <= bound(batch, X.T, dA[:, rest]))


@pytest.mark.parametrize("shape,batch", [((128, 64, 3), 128), ((256, 256, 10), 256)])
def test_every_row_alignment_gives_the_same_bits(shape, batch):
    """The update's tiles are counted from the first 128-byte line of a worker's row: whatever the row's offset, and
    with line 6 inside the last step or alone, the result is the same."""
    W, theta = 3, theta_of(shape)
    d = synth_inputs.mlp_param_count(*shape)
    want = None
    for extra, fused_tail in [(e, tail) for e in (0, 4, 12, 20, 28, 32) for tail in (False, True)]:
        stride = (d + 31) // 32 * 32 + extra
        dev = torch.device("cuda:0")
        xA = torch.zeros((W, stride), device=dev)
        xA[:, :d] = torch.from_numpy(theta).to(dev) * torch.tensor([[1.0], [0.5], [2.0]], device=dev)
        xB, v, mean = torch.zeros_like(xA), torch.zeros_like(xA), torch.zeros(stride, device=dev)
        s = torch.cuda.Stream(device=dev)
        torch.cuda.synchronize()
        ctx = P.Context(W=W, d=d, stride=stride, xA=xA, xB=xB, v=v, mean=mean, grad=P.GRAD_MLP, mlp=(*shape, batch),
                        compute_stream=s, avg_stream=s, **HYPER)
        for _ in range(2):
            ctx.round_fused_tail(2) if fused_tail else ctx.round(2)
        ctx.sync()
        live = xA if ctx.live_model() == xA.data_ptr() else xB
        got = [t[..., :d].cpu() for t in (live, v, mean)]
        ctx.close()
        if want is None:
            want = got
        assert all(torch.equal(p, q) for p, q in zip(got, want)), (extra, fused_tail)
