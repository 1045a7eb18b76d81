"""Host-only check of the indexing of the contraction kernels on the 16-bit matrix instructions, of the output-layer
kernel and of the work that rides in the backward launch (csrc/mlp.hip), restated here: every operand access inside its
array for the last worker and the tightest buffers, every element of the results owned exactly once."""
import numpy as np
import pytest

SLICE, THREADS = 32, 256
SHAPES = [(n_in, n_hid, batch) for n_in in (128, 384, 3072) for n_hid in (64, 192, 256, 1024) for batch in (128, 384, 1024)]


def forward_splits(W, n_in, n_hid, batch, cus=256):
    tiles = W * (batch // 128) * (n_hid // (128 if n_hid % 128 == 0 else 64))
    return min(-(-cus // tiles), min(n_in // SLICE // 4, 8))


def split_slices(n_in, splits):
    pairs = n_in // SLICE // 2
    return [(2 * (pairs * s // splits), 2 * (pairs * (s + 1) // splits)) for s in range(splits)]


@pytest.mark.parametrize("n_in,n_hid,batch", SHAPES)
@pytest.mark.parametrize("W", [1, 3, 16, 400])
def test_forward_splits_cover_k_and_stay_inside(W, n_in, n_hid, batch):
    splits = forward_splits(W, n_in, n_hid, batch)
    ranges = split_slices(n_in, splits)
    assert 1 <= splits <= 8 and ranges[0][0] == 0 and ranges[-1][1] == n_in // SLICE
    assert all(a[1] == b[0] for a, b in zip(ranges, ranges[1:]))
    for first, end in ranges:
        n = end - first
        assert n >= 2 and n % 2 == 0                         # two register sets: slices come in pairs
        loaded = {0, 1} | {s + d for s in range(0, max(n - 2, 0), 2) for d in (2, 3)}
        assert loaded == set(range(n))
    BN = 128 if n_hid % 128 == 0 else 64
    t = np.arange(THREADS)
    rows = (t // 4)[:, None] + 64 * np.arange(2)
    assert sorted(rows[t % 4 == 0].ravel().tolist()) == list(range(128))
    k = (n_in // SLICE - 1) * SLICE + (t % 4) * 8 + 7
    assert (batch - 128 + rows.max()) * n_in + k.max() == batch * n_in - 1
    col = n_hid - BN + (t % 64) * (BN // 64) + BN // 64 - 1
    krow = (n_in // SLICE - 1) * SLICE + (t // 64) * 8 + 7
    assert krow.max() * n_hid + col.max() == n_in * n_hid - 1


@pytest.mark.parametrize("n_hid", [64, 128, 192, 256, 1024])
@pytest.mark.parametrize("lead", range(0, 32, 4))
def test_backward_columns_are_owned_once_whatever_the_row_offset(n_hid, lead):
    BN = 128 if n_hid % 128 == 0 else 64
    owned = []
    for n0 in range(0, n_hid, BN):
        c = n0 + lead + np.arange(BN)
        c = np.where(c < n_hid, c, c - n_hid)
        assert c.min() >= 0 and c.max() < n_hid
        assert np.all(np.diff(c.reshape(-1, 4), axis=1) == 1)          # a quad never wraps
        owned += c.tolist()
    assert sorted(owned) == list(range(n_hid))


@pytest.mark.parametrize("n_in,n_hid,batch", SHAPES)
def test_backward_tiles_small_update_and_mini_batch(n_in, n_hid, batch):
    W, BM = 3, 64
    BN = 128 if n_hid % 128 == 0 else 64
    nx, ny = n_hid // BN, n_in // BM
    total = nx * ny * W
    plain, line6 = set(), set()
    for linear in range(total):
        logical = (linear % 8) * (total // 8) + linear // 8 if total % 8 == 0 else linear
        plain.add((logical % nx, logical // nx % ny, logical // (nx * ny)))
        if ny % 8 == 0:
            rows, r = ny // 8, linear // 8
            line6.add((r % nx, (linear % 8) * rows + r // nx % rows, r // (nx * rows)))
    every = {(x, y, w) for x in range(nx) for y in range(ny) for w in range(W)}
    assert plain == every and (ny % 8 != 0 or line6 == every)
    # rows and columns of the update: BN / 4 threads per row
    per_pass, iters = THREADS // (BN // 4), BM * BN // 4 // THREADS
    t = np.arange(THREADS)
    got = {(r + it * per_pass, c) for it in range(iters) for r, c in zip(t // (BN // 4), t % (BN // 4) * 4)}
    assert got == {(r, c) for r in range(BM) for c in range(0, BN, 4)}
    # the small update's samples: wave w, quarter g, step s0 + 4 s
    per = batch // 4
    samples = [w * per + g + s0 + 4 * s for w in range(4) for g in range(4) for s0 in range(0, per, 16) for s in range(4)]
    assert sorted(samples) == list(range(batch))
    # the next mini-batch: groups of 256 quads, dealt to the tiles
    groups = (batch * n_in // 4 + 255) // 256 * W
    dealt = sorted(i for linear in range(total) for i in range(linear, groups, total))
    assert dealt == list(range(groups))


@pytest.mark.parametrize("n_hid", [64, 192, 1024, 2048, 2112, 4096 + 64])
def test_output_layer_chunks_rows_and_blocks(n_hid):
    chunk, waves, group = 2048, 16, 4
    pitch = min(n_hid, chunk) + 4
    seen = []
    for c0 in range(0, n_hid, chunk):
        width = min(chunk, n_hid - c0)
        cols = [n0 + 256 * i for lane in range(64) for n0 in range(4 * lane, width, 256 * group) for i in range(group) if n0 + 256 * i < width]
        assert sorted(cols) == list(range(0, width, 4)) and max(cols) + 4 <= pitch
        blocks = [b0 + waves * i for w in range(waves) for b0 in range(w, width // 16, waves * group) for i in range(group) if b0 + waves * i < width // 16]
        assert sorted(blocks) == list(range(width // 16))
        seen += [c0 + 16 * b for b in blocks]
    assert sorted(seen) == list(range(0, n_hid, 16))
    assert 16 * pitch * 4 + 17536 <= 160 * 1024                        # dynamic and static LDS of a block
