"""Which feature the exact distance transform names: among those at the exact
distance the one in the smallest column, and of that column the upper one.
Compared with a plain evaluation over all columns, at sizes around the row
pass's anchors, its two workgroup sizes and both of its paths (dense rows, and
rows whose features lie farther away than an anchor's own search goes)."""
import numpy as np
import pytest

from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


def by_columns(B):
    h, w = B.shape
    y = np.arange(h)[:, None]
    up = np.maximum.accumulate(np.where(B == 0, y, -1), axis=0)
    down = np.minimum.accumulate(np.where(B == 0, y, 1 << 20)[::-1], axis=0)[::-1]
    r = np.where((up >= 0) & ((down >= 1 << 20) | (y - up <= down - y)), up, np.where(down < 1 << 20, down, -1))
    sq, nr = np.full((h, w), -1, np.int64), np.full((h, w), -1, np.int64)
    cols = np.arange(w, dtype=np.int64)
    for i in range(h):
        f = np.where(r[i] < 0, 1 << 40, (i - r[i]).astype(np.int64) ** 2)
        if f.min() >= 1 << 40:
            continue
        for a in range(0, w, 512):
            x = cols[a:a + 512]
            d = (x[:, None] - cols[None, :]) ** 2 + f[None, :]
            c = d.argmin(axis=1)  # the first minimum: the smallest column
            sq[i, a:a + 512], nr[i, a:a + 512] = d[np.arange(x.size), c], r[i, c].astype(np.int64) * w + c
    return sq, nr


@pytest.mark.parametrize("h,w,p", [(1, 1, 0.5), (65, 2, 0.2), (64, 15, 0.1), (63, 16, 0.1), (66, 17, 0.05),
                                   (130, 33, 0.02), (7, 1023, 0.01), (200, 129, 0.3), (1100, 70, 0.0003),
                                   (257, 300, 0.00005), (3, 8192, 0.002), (3, 8193, 0.002), (2, 9001, 0.0002)])
def test_named_feature(h, w, p):
    torch, iw = require_gpu()
    rng = np.random.default_rng(h * 10007 + w)
    B = (rng.random((h, w)) >= p).astype(np.uint8)
    B[rng.integers(h), rng.integers(w)] = 0
    B[0, w - 1] = 0
    announce("edt exact named feature", h, w, p)
    ctx = iw.Context(0)
    try:
        sq, nr = ctx.edt_exact(torch.from_numpy(B).cuda())
        sq, nr = sq.cpu().numpy(), nr.cpu().numpy()
    finally:
        ctx.close()
    es, en = by_columns(B)
    assert np.array_equal(sq, es) and np.array_equal(nr, en)
