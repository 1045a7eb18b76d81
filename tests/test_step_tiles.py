"""Host-only check of the step kernel's tiles (csrc/local_step.hip): the chunk table's entries and the rule that moves a
worker's tiles up to the 128-byte lines of its row are restated here; every element of every tensor must be served by
exactly one wave pass, inside its tensor, for every distance of the row from a line."""
import numpy as np
import pytest

CHUNK, TILE, LINE = 1024, 256, 32


def chunks_of(n):
    """(offset in the tensor, elements, elements behind the chunk (at most a line), first) per chunk."""
    out = []
    for off in range(0, n, CHUNK):
        here = min(CHUNK, n - off)
        out.append((off, here, min(LINE, n - off - here), off == 0))
    return out


def passes(n, lead):
    """(begin, end) inside the tensor of every wave pass of one worker row that lies `lead` elements before a line."""
    for off, here, after, first_chunk in chunks_of(n):
        for first in range(0, CHUNK, TILE):
            if first >= here:
                continue
            begin = first + lead
            count = min(TILE, max(0, here + after - begin))
            if first_chunk and first == 0 and lead:
                yield off, off + min(here, lead)
            if count:
                yield off + begin, off + begin + count


@pytest.mark.parametrize("lead", range(0, LINE, 4))
def test_every_element_is_served_once(lead):
    sizes = list(range(1, 70)) + [n + e for n in (256, 512, 768, 1024, 2048, 3072) for e in range(-33, 34)] + [12345, 99999]
    for n in sizes:
        count = np.zeros(n, dtype=np.int32)
        for begin, end in passes(n, lead):
            assert 0 <= begin < end <= n and end - begin <= TILE
            assert (begin + (LINE - lead)) % LINE == 0 or begin == 0          # on a line, or the head of the tensor
            assert begin % 4 == 0
            count[begin:end] += 1
        assert np.all(count == 1), (n, lead)
