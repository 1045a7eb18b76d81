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


def tile_cols(n_hid):
    return 128 if n_hid % 128 == 0 else 64


def b_operand(K, n_hid, first_col):
    """(k, column) of every B element that the lanes of a block read in the last slice."""
    wave, lane, kb, j = np.meshgrid(np.arange(4), np.arange(64), np.arange(2), np.arange(8), indexing="ij")
    col = first_col + wave % (tile_cols(n_hid) // 32) * 32 + lane % 32
    return K - SLICE + 16 * kb + 8 * (lane // 32) + j, np.where(col < n_hid, col, col - n_hid)


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
        assert n >= 2 and n % 2 == 0                         # two LDS buffers: slices come in pairs
        loaded = [0] + [s + d for s in range(0, n - 2, 2) for d in (1, 2)] + [n - 1]
        assert loaded == list(range(n))
    t = np.arange(THREADS)
    rows = (t // 4)[:, None] + 64 * np.arange(2)
    assert sorted(rows[t % 4 == 0].ravel().tolist()) == list(range(128))
    k = (n_in // SLICE - 1) * SLICE + (t % 4) * 8 + 7
    assert (batch - 128 + rows.max()) * n_in + k.max() == batch * n_in - 1
    krow, col = b_operand(n_in, n_hid, n_hid - tile_cols(n_hid))
    assert krow.max() * n_hid + col.max() == n_in * n_hid - 1


@pytest.mark.parametrize("BN", [64, 128])
def test_b_operand_covers_a_slice_once_per_row_of_waves(BN):
    """Lane l of wave w: column 32 (w % waves along N) + l % 32, octets l / 32 and 2 + l / 32 of the slice."""
    seen = {}
    for wave in range(4):
        for lane in range(64):
            for kb in range(2):
                for j in range(8):
                    at = (wave // (BN // 32), 16 * kb + 8 * (lane // 32) + j, wave % (BN // 32) * 32 + lane % 32)
                    seen[at] = seen.get(at, 0) + 1
    assert seen == {(m, k, c): 1 for m in range(4 // (BN // 32)) for k in range(SLICE) for c in range(BN)}


@pytest.mark.parametrize("forward", [True, False])
def test_a_operand_is_read_where_it_was_written(forward):
    """A's pieces in LDS: [32-row block][octet][slot]; the eight lanes that write together use eight 16-byte groups."""
    rows = 128 if forward else 64
    slot = (lambda r, o: (r + 2 * o) & 31) if forward else (lambda r, o: r)
    lds = {}
    for i in range(rows // 64):
        for t in range(THREADS):
            row, octet = (t // 4 + 64 * i, t % 4) if forward else (t % 64, t // 64)
            key = (row // 32, octet, slot(row % 32, octet))
            assert key not in lds
            lds[key] = (row, octet)
        for first in range(0, THREADS, 8):
            together = [(t // 4 + 64 * i, t % 4) if forward else (t % 64, t // 64) for t in range(first, first + 8)]
            groups = {slot(r % 32, o) % 8 for r, o in together}
            assert len(groups) == 8
    assert len(lds) == rows * 4
    for block in range(rows // 32):
        for kb in range(2):
            for lane in range(64):
                octet = 2 * kb + lane // 32
                assert lds[(block, octet, slot(lane % 32, octet))] == (32 * block + lane % 32, octet)


@pytest.mark.parametrize("BM,BN", [(128, 128), (128, 64), (64, 128), (64, 64)])
def test_results_cover_the_tile_once(BM, BN):
    """Lane l, register r of a wave's 32-row block i: row l % 32, column 8 (r / 4) + 4 (l / 32) + r % 4 of its 32 columns."""
    nwn = BN // 32
    mb = BM // 32 // (4 // nwn)
    got = sorted(((w // nwn * mb + i) * 32 + l % 32, w % nwn * 32 + 8 * (r // 4) + 4 * (l // 32) + r % 4)
                 for w in range(4) for i in range(mb) for l in range(64) for r in range(16))
    assert got == [(r, c) for r in range(BM) for c in range(BN)]


@pytest.mark.parametrize("n_in,n_hid,batch", SHAPES)
def test_backward_operands_and_update_stay_inside(n_in, n_hid, batch):
    """X^T, dA with wrapped columns, and the update's x, v, stored model and mean, for the last worker and tile."""
    W, BM, BN = 3, 64, tile_cols(n_hid)
    t = np.arange(THREADS)
    x_row = (batch // SLICE - 1) * SLICE + (t // 64) * 8 + 7
    assert x_row.max() * n_in + (n_in - BM) + (t % 64).max() == batch * n_in - 1
    assert [0] + [s + d for s in range(0, batch // SLICE - 2, 2) for d in (1, 2)] + [batch // SLICE - 1] == list(range(batch // SLICE))
    stride = (n_in * n_hid + n_hid + 3) // 4 * 4
    for lead in range(0, 32, 4):
        for n0 in (0, n_hid - BN):
            krow, col = b_operand(batch, n_hid, n0 + lead)
            assert col.min() >= 0 and col.max() < n_hid and krow.max() == batch - 1
            quad = n0 + lead + (t % (BN // 4)) * 4
            quad = np.where(quad < n_hid, quad, quad - n_hid)
            per_pass, iters = THREADS // (BN // 4), BM * BN // 4 // THREADS
            last = (W - 1) * stride + (n_in - BM + (t // (BN // 4)).max() + (iters - 1) * per_pass) * n_hid + quad.max() + 3
            assert quad.min() >= 0 and last < (W - 1) * stride + n_in * n_hid


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


@pytest.mark.parametrize("n_in,n_hid,batch", SHAPES)
@pytest.mark.parametrize("n_out", [1, 10, 16])
def test_output_layer_and_small_update_stay_inside_their_arrays(n_in, n_hid, batch, n_out):
    """Last worker, tightest buffers: H, dA, dZ rows, the K splits behind H, W2 read by hidden unit and by class, and the
    next mini-batch."""
    W, pitch = 3, 16
    splits = forward_splits(W, n_in, n_hid, batch)
    group, wave = batch // 16 - 1, 15
    sample = (W - 1) * batch + group * 16 + wave
    assert sample == W * batch - 1
    assert sample * n_hid + n_hid - 1 == W * batch * n_hid - 1                                 # H and dA
    assert max(splits - 2, 0) * W * batch * n_hid + sample * n_hid + n_hid - 1 < max(splits - 1, 1) * W * batch * n_hid
    lane = np.arange(64)
    s16, g = lane % 16, lane // 16
    W2 = n_in * n_hid + n_hid
    end = W2 + n_hid * n_out
    for j in range(4):                                       # the last block of 16 hidden units
        by_unit = (n_hid - 16 + 4 * g + j) * n_out + s16
        by_class = (n_hid - 16 + s16) * n_out + 4 * j + g
        assert W2 + by_unit[s16 < n_out].max() < end and by_unit[s16 < n_out].max() + 1 <= n_hid * n_out
        ok = 4 * j + g < n_out
        assert not ok.any() or W2 + by_class[ok].max() < end
    own = n_hid // 64 - 1                                    # small update: 64 hidden units, quarter of the batch per wave
    s = (W - 1) * batch + 3 * (batch // 4) + (batch // 4 - 16) + 12 + g
    assert s.max() == W * batch - 1 and s.max() * pitch + s16.max() == W * batch * pitch - 1
    assert (s * n_hid + own * 64 + s16 + 48).max() == W * batch * n_hid - 1
    e = np.arange(64 * n_out)
    assert own * 64 * n_out + e.max() == n_hid * n_out - 1
    stride = (end + n_out + 3) // 4 * 4                      # the pads behind the last parameter, at most three
    assert end + n_out + ((end + n_out + 3) // 4 * 4 - (end + n_out)) <= stride
    groups = (batch * n_in // 4 + 255) // 256
    q = (groups - 1) * 256 + np.arange(256)
    q = q[q < batch * n_in // 4]
    assert q.max() * 4 + 3 == batch * n_in - 1 and batch // 4 <= 256
