"""Host checks of integer-from-float shortcuts the HIP kernels rely on (no GPU)."""
import numpy as np


def _nudge(x, ulps):
    x = np.float32(x)
    step = np.float32(np.inf) if ulps > 0 else np.float32(-np.inf)
    for _ in range(abs(ulps)):
        x = np.nextafter(x, step, dtype=np.float32)
    return x


def test_rectangle_row_from_reciprocal():
    # instance emission: row = trunc(pos * rcp(rw) + 1/128) for a hit position pos < 64 in a
    # tile rectangle of width rw <= 64; exact for a reciprocal off by up to two ulps, with
    # the fused multiply-add rounded once or the product rounded first
    for rw in range(1, 65):
        r0 = np.float32(1.0) / np.float32(rw)
        for ulps in range(-2, 3):
            r = _nudge(r0, ulps)
            for pos in range(64):
                fused = np.float32(np.float64(pos) * np.float64(r) + 1.0 / 128.0)
                split = np.float32(np.float32(np.float32(pos) * r) + np.float32(1.0 / 128.0))
                assert int(fused) == pos // rw and int(split) == pos // rw, (rw, ulps, pos)


def test_cells_of_small_rectangles():
    # tile lists: the cells of 2x2 tiles of a rectangle of at most 64 tiles, at every offset from
    # the cells' grid, take at most 34 places (they are laid over 64 lanes, and a cell's row is
    # found from k * rcp(cw) + 1/128), and each tile's mask bit is taken exactly once
    most, widest = 0, 0
    for rw in range(1, 65):
        for rh in range(1, 64 // rw + 1):
            for x0, y0 in ((2, 4), (3, 4), (2, 5), (3, 5)):
                cx0, cy0 = x0 >> 1, y0 >> 1
                cw, ch = ((x0 + rw - 1) >> 1) - cx0 + 1, ((y0 + rh - 1) >> 1) - cy0 + 1
                most, widest = max(most, cw * ch), max(widest, cw)
                seen = []
                for k in range(cw * ch):
                    cr = int(np.float32(np.float64(k) * np.float64(np.float32(1.0) / np.float32(cw)) + 1.0 / 128.0))
                    assert cr == k // cw
                    dx, dy = 2 * (cx0 + k - cr * cw) - x0, 2 * (cy0 + cr) - y0
                    cols = (1 if dx >= 0 else 0) | (2 if dx + 1 < rw else 0)
                    for row in range(2):
                        y = dy + row
                        p = y * rw + dx
                        assert p >= -1 or not 0 <= y < rh
                        for bit in range(2):
                            if cols >> bit & 1 and 0 <= y < rh:
                                assert 0 <= p + bit < 64
                                seen.append(p + bit)
                assert sorted(seen) == list(range(rw * rh)), (rw, rh, x0, y0)
    assert (most, widest) == (34, 33)
