"""What the reconstruction's sweeps of a 64 x 64 tile rely on, in a plain model of
the same chunk order: a line is stable after one pair of opposite scans that run at
the same time, and a scan may skip the 16-wide chunks whose predecessors did not
change since it last ran, unless it changed the chunk before."""
import numpy as np
import pytest

T, CHUNK = 64, 16


def tile(rng, step, keep):
    I = (np.cumsum(rng.integers(-step, step + 1, (T, T)), axis=1) + 128).clip(0, 255)
    J = np.where(rng.random((T, T)) < keep, np.maximum(I, 40) - 40, I)
    return J.astype(np.int64), I.astype(np.int64)


def tiles(seed, n):
    rng = np.random.default_rng(seed)
    for k in range(n):
        yield tile(rng, (1, 3, 40, 120)[k % 4], (0.5, 0.97, 0.995)[k % 3])


def stable(J, I, conn):
    """No neighbour inside the tile can raise a pixel."""
    P = np.pad(J, 1)
    for dy in (-1, 0, 1):
        for dx in (-1, 0, 1):
            if (dy or dx) and (conn == 8 or not (dy and dx)):
                if (np.minimum(P[1 + dy:T + 1 + dy, 1 + dx:T + 1 + dx], I) > J).any():
                    return False
    return True


def lines_stable(J, I):
    return not ((np.minimum(J[:, :-1], I[:, 1:]) > J[:, 1:]).any() or (np.minimum(J[:, 1:], I[:, :-1]) > J[:, :-1]).any())


def preds(chunk, forward):
    lo = chunk * CHUNK + (-1 if forward else 1)
    return range(max(0, lo), min(T, lo + CHUNK))


def line_pair(J, I, dirty=None):
    """Both scans along axis 1, four passes of a chunk each; `dirty`: the columns
    changed since they last ran (None: take every chunk).  Returns the changed rows
    and the number of chunks scanned."""
    rows, scanned, f, b = set(), 0, False, False
    for c in range(T // CHUNK):
        cb = T // CHUNK - 1 - c
        if dirty is None:
            f = b = True
        else:
            f = f or any(p in dirty for p in preds(c, True))
            b = b or any(p in dirty for p in preds(cb, False))
        df, db = np.zeros(T, bool), np.zeros(T, bool)
        for k in range(CHUNK):  # a step of each, from the values before either
            x, y = c * CHUNK + k, T - 1 - (c * CHUNK + k)
            nf = np.minimum(np.maximum(J[:, x], J[:, x - 1] if x else 0), I[:, x]) if f else J[:, x].copy()
            nb = np.minimum(np.maximum(J[:, y], J[:, y + 1] if y < T - 1 else 0), I[:, y]) if b else J[:, y].copy()
            df |= nf != J[:, x]
            db |= nb != J[:, y]
            J[:, x], J[:, y] = nf, nb
        scanned += int(f) + int(b)
        f, b = bool(df.any()), bool(db.any())
        rows |= set(np.flatnonzero(df | db).tolist())
    return rows, scanned


def column_scan8(J, I, forward, dirty):
    """One 8-connected column scan by chunks of rows; returns changed columns, rows
    (whole chunks) and chunks scanned."""
    cols, rows, scanned, carry = set(), set(), 0, False
    for c in range(T // CHUNK) if forward else range(T // CHUNK - 1, -1, -1):
        if not carry and not any(p in dirty for p in preds(c, forward)):
            continue
        scanned += 1
        d = np.zeros(T, bool)
        for k in range(CHUNK):
            y = c * CHUNK + (k if forward else CHUNK - 1 - k)
            q = y - 1 if forward else y + 1
            p = J[q] if 0 <= q < T else np.zeros(T, np.int64)
            e = np.pad(p, 1)
            n = np.minimum(np.maximum(J[y], np.maximum(p, np.maximum(e[:-2], e[2:]))), I[y])
            d |= n != J[y]
            J[y] = n
        carry = bool(d.any())
        if carry:
            cols |= set(np.flatnonzero(d).tolist())
            rows |= set(range(c * CHUNK, (c + 1) * CHUNK))
    return cols, rows, scanned


def sweep8(J, I, r_cf, r_cb, c_r, columns_first=False, limit=400):
    """The 8-connected sweep with its dirty sets; returns the chunks scanned."""
    scanned = 0
    for n in range(limit):
        if not (r_cf or r_cb or c_r):
            return scanned
        if ((n & 1) != 0) == columns_first:
            if c_r:
                r, s = line_pair(J, I, c_r)
                c_r = set()
                r_cf, r_cb, scanned = r_cf | r, r_cb | r, scanned + s
        elif r_cf or r_cb:
            c, rows, s = column_scan8(J, I, True, r_cf)
            r_cb, r_cf, c_r, scanned = r_cb | rows, set(), c_r | c, scanned + s
            c, rows, s = column_scan8(J, I, False, r_cb)
            r_cf, r_cb, c_r, scanned = r_cf | rows, set(), c_r | c, scanned + s
    raise AssertionError("not stable")


def test_a_line_is_stable_after_one_pair():
    for J, I in tiles(1, 60):
        for axis in (0, 1):
            j, i = (J.T.copy(), I.T.copy()) if axis else (J.copy(), I.copy())
            line_pair(j, i)
            assert lines_stable(j, i)


def test_four_connected_tile_is_stable_when_a_later_pair_changes_nothing():
    for J, I in tiles(2, 24):
        for n in range(400):
            j, i = (J.T, I.T) if n & 1 else (J, I)
            before = J.copy()
            line_pair(j, i)
            if n > 0 and np.array_equal(J, before):
                break
        assert stable(J, I, 4)


@pytest.mark.parametrize("columns_first", [False, True])
def test_skipped_chunks_leave_eight_connected_tiles_stable(columns_first):
    rng = np.random.default_rng(3)
    everything = set(range(T))
    saved = 0
    for J, I in tiles(3, 12):
        sweep8(J, I, set(everything), set(everything), set(everything), columns_first)
        assert stable(J, I, 8)
        for _ in range(3):  # then a few pixels of a stable tile rise, as border pixels do
            rows, cols = set(), set()
            for _ in range(int(rng.integers(1, 4))):
                y, x = (int(v) for v in rng.integers(0, T, 2))
                if J[y, x] < I[y, x]:
                    J[y, x] = I[y, x]
                    rows.add(y)
                    cols.add(x)
            full = J.copy()
            scanned = sweep8(J, I, set(rows), set(rows), set(cols), columns_first)
            assert stable(J, I, 8)
            complete = sweep8(full, I, set(everything), set(everything), set(everything), columns_first)
            assert np.array_equal(full, J)
            saved += complete - scanned
    assert saved > 0  # the sets do skip chunks
