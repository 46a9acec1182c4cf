"""Hand-over of the blocked Cholesky's pivot masks (CPU only).

chol_inv_blocked ends with every thread reading the masks of refused pivots
from the work area, with no barrier behind; the test for a second CholeskyQR
pass that may follow at once has each wave write a partial sum.  The words are
read from the kernel header, and the two steps are replayed in the orders in
which four waves can take them: whatever wave is ahead, the others have to read
the masks as they were.
"""
import itertools
import os
import re
import struct

HDR = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_22713_amd", "csrc",
                   "eodabe_kernels.hpp")


def _word(expr, src):
    """Offset in doubles of an expression like `work`, `work + 8` or `work + NAME`."""
    m = re.fullmatch(r"work(?:\s*\+\s*(\w+))?", expr.strip())
    assert m, expr
    if m.group(1) is None:
        return 0
    if m.group(1).isdigit():
        return int(m.group(1))
    return int(re.search(r"\b%s = (\d+)" % m.group(1), src).group(1))


def _layout():
    src = open(HDR).read()
    refused = re.search(r"uint32_t\* refused = reinterpret_cast<uint32_t\*>\(([^)]*)\)", src).group(1)
    dump = re.search(r"double\* dump = ([^;]*);", src).group(1)
    body = src[src.index("bool chol_tame_sum("):]
    body = body[:body.index("\n}")]
    m = re.search(r"double\* red = ([^;]*);", body)
    # without words of its own the sum takes the area it is handed from its start
    red = _word(m.group(1), src) if m else 0
    return _word(refused, src), red, _word(dump, src)


def _replay(refused, red, masks, order):
    """The masks each wave reads when the waves read them and then write their
    sums in the given interleaving of (wave, step)."""
    work = bytearray(8 * 128)
    struct.pack_into("<4I", work, 8 * refused, *masks)
    seen = {}
    for wave, step in order:
        if step == 0:
            seen[wave] = struct.unpack_from("<4I", work, 8 * refused)
        else:
            struct.pack_into("<d", work, 8 * (red + wave), 0.37 + wave)
    return seen


def _orders():
    steps = [(w, s) for w in range(4) for s in (0, 1)]
    for late in itertools.permutations(range(4)):
        yield [(w, s) for w in late for s in (0, 1)]             # one wave after the other
    for late in range(4):                                          # one wave behind all others
        yield [x for x in steps if x[0] != late] + [x for x in steps if x[0] == late]


def test_every_wave_reads_the_masks_as_written():
    refused, red, dump = _layout()
    for masks in ((0, 0, 0, 0), (1, 0, 0, 0x8000), (0xFFFF, 3, 0, 0)):
        for order in _orders():
            for wave, got in _replay(refused, red, masks, order).items():
                assert got == masks, (wave, got, masks, order)


def test_work_words_are_disjoint():
    refused, red, dump = _layout()
    words = [set(range(refused, refused + 2)), set(range(red, red + 4)), set(range(dump, dump + 64))]
    for a, b in itertools.combinations(words, 2):
        assert not a & b
