"""Change records of the propagation EDT in tile columns of every word width (1,
2, 4 and 8 bytes a row), with changes that cross from and into the last column
and rows cut by the image's end; and a server whose scratch area just holds an
image a few pixels high or wide by 344 bytes per 26 x 26 pixels."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("conn", [4, 8])
@pytest.mark.parametrize("cols", [1, 8, 9, 16, 17, 32, 33, 47, 48])
def test_record_widths(cols, conn, waves):
    torch, iw = require_gpu()
    rng = np.random.default_rng(cols * 10 + conn)
    ctx = iw.Context(0, wg_waves=waves)
    try:
        for h, full in ((1, 0), (7, 1), (101, 0), (97, 1), (150, 2)):
            w = 48 * full + cols
            for p in (0.0, 0.004):
                B = (rng.random((h, w)) >= p).astype(np.uint8)
                B[rng.integers(h), 0 if p else w - 1] = 0
                announce("edt record widths", h, w, conn, waves, p)
                sq, nr = ctx.edt(torch.from_numpy(B).cuda(), conn)
                st = ctx.stats()
                so, no, ost = oracle.edt_rounds(B, conn, return_stats=True)
                assert st["status"] == 0 and np.array_equal(sq.cpu().numpy(), so) and np.array_equal(nr.cpu().numpy(), no)
                assert st["rounds"] == ost["rounds"] and st["items"] == ost["items"]
    finally:
        ctx.close()


@pytest.mark.parametrize("h,w", [(1, 40000), (40000, 1), (10, 40000), (26, 49)])
def test_server_admits_thin_images(h, w):
    torch, iw = require_gpu()
    rng = np.random.default_rng(h + w)
    B = (rng.random((h, w)) >= 0.002).astype(np.uint8)
    B[0, 0] = 0
    job = {"op": "edt", "conn": 8, "binary": torch.from_numpy(B).pin_memory(),
           "sqdist": torch.empty((h, w), dtype=torch.int32).pin_memory(),
           "nearest": torch.empty((h, w), dtype=torch.int32).pin_memory()}
    need = 344 * (-(-h // 26) * -(-w // 26)) + 20 * 256 + 8 * h * w + 2 * 256 + 56 + 64 * 256
    announce("server thin", h, w, need)
    ctx = iw.Context(0)
    try:
        with iw.Server(ctx, hbm_budget_bytes=64 << 20, scratch_bytes=-(-need // 256) * 256) as srv:
            srv.submit(job)
            srv.drain()
    finally:
        ctx.close()
    so, no = oracle.edt_rounds(B, 8)
    assert np.array_equal(job["sqdist"].numpy(), so) and np.array_equal(job["nearest"].numpy(), no)
