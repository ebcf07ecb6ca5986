"""The propagation EDT at the edges of its 48 x 48 tiles and their 64 x 64
regions: sides around the multiples of 48, images with more changes in a round
than a wave lists at a time, both coordinate widths and workgroup sizes.
Distances, indices and work counts equal the oracle's (whole numbers)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves", [0, 8])
@pytest.mark.parametrize("h,w,conn,density", [
    (47, 49, 8, 0.02), (48, 48, 4, 0.02), (49, 97, 8, 0.002), (96, 95, 4, 0.002), (145, 40, 8, 0.01),
    (8, 300, 4, 0.003), (200, 200, 8, 0.7), (200, 200, 4, 0.35), (150, 149, 8, 0.0002), (5, 33000, 8, 0.01),
    (33000, 3, 4, 0.02)])
def test_tile_edges(h, w, conn, density, waves):
    torch, iw = require_gpu()
    rng = np.random.default_rng(h * 131 + w + conn)
    B = (rng.random((h, w)) >= density).astype(np.uint8)
    B[rng.integers(h), rng.integers(w)] = 0
    announce("edt tile edges", h, w, conn, density, waves)
    ctx = iw.Context(0, wg_waves=waves)
    try:
        sq, nr = ctx.edt(torch.from_numpy(B).cuda(), conn)
        st = ctx.stats()
        sq, nr = sq.cpu().numpy(), nr.cpu().numpy()
    finally:
        ctx.close()
    so, no, ost = oracle.edt_rounds(B, conn, return_stats=True)
    assert st["status"] == 0 and np.array_equal(sq, so) and np.array_equal(nr, no)
    assert st["rounds"] == ost["rounds"] and st["items"] == ost["items"]


def test_long_runs_of_changes():
    """Straight fronts (one feature row, one feature column) and a diagonal:
    whole rows and columns of a region change in one round."""
    torch, iw = require_gpu()
    ctx = iw.Context(0)
    try:
        for k in range(3):
            B = np.ones((260, 310), np.uint8)
            if k == 0:
                B[131, :] = 0
            elif k == 1:
                B[:, 77] = 0
            else:
                B[np.arange(260), np.arange(260)] = 0
            for conn in (4, 8):
                announce("edt straight fronts", k, conn)
                sq, nr = ctx.edt(torch.from_numpy(B).cuda(), conn)
                so, no = oracle.edt_rounds(B, conn)
                assert np.array_equal(sq.cpu().numpy(), so) and np.array_equal(nr.cpu().numpy(), no)
    finally:
        ctx.close()


@pytest.mark.parametrize("blocks", [1, 3, 8, 9, 20])
def test_more_tiles_than_workgroups(blocks):
    """Steps that list more tiles than the grid has workgroups: tiles dealt by
    group, taken as workgroups get to them, and taken from other groups; with
    fewer workgroups than groups some groups have none.  One image and a batch."""
    torch, iw = require_gpu()
    rng = np.random.default_rng(blocks)
    imgs = [(rng.random(s) >= d).astype(np.uint8) for s, d in (((400, 500), 0.01), ((49, 300), 0.3), ((700, 60), 0.001))]
    imgs[2][10, 10] = 0
    ctx = iw.Context(0, persistent_blocks=blocks)
    try:
        announce("edt dealing", blocks)
        for B in imgs:
            sq, nr = ctx.edt(torch.from_numpy(B).cuda(), 8)
            st = ctx.stats()
            so, no, ost = oracle.edt_rounds(B, 8, return_stats=True)
            assert st["status"] == 0 and np.array_equal(sq.cpu().numpy(), so) and np.array_equal(nr.cpu().numpy(), no)
            assert st["rounds"] == ost["rounds"] and st["items"] == ost["items"]
        out = [[torch.empty(B.shape, dtype=torch.int32, device="cuda") for _ in range(2)] for B in imgs]
        ctx.run_batch([{"op": "edt", "binary": torch.from_numpy(B).cuda(), "sqdist": sq, "nearest": nr, "conn": 8}
                       for B, (sq, nr) in zip(imgs, out)])
        for B, (sq, nr) in zip(imgs, out):
            so, no = oracle.edt_rounds(B, 8)
            assert np.array_equal(sq.cpu().numpy(), so) and np.array_equal(nr.cpu().numpy(), no)
    finally:
        ctx.close()
