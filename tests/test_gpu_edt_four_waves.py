"""The propagation EDT's two workgroup sizes, each by name, where the automatic
size takes only one of them: tile edges and images with more changes in a round than
a wave of four lists at a time (256), whole rows and columns changing in one round,
and steps with more tiles than the grid has workgroups.  Distances, indices and work
counts equal the oracle's."""
import numpy as np
import pytest

import oracle
from paper_1209_3314_amd import synth
from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


def check(torch, ctx, B, conn):
    sq, nr = ctx.edt(torch.from_numpy(B).cuda(), conn)
    st = ctx.stats()
    so, no, ost = oracle.edt_rounds(B, conn, return_stats=True)
    assert st["status"] == 0 and np.array_equal(sq.cpu().numpy(), so) and np.array_equal(nr.cpu().numpy(), no)
    assert st["rounds"] == ost["rounds"] and st["items"] == ost["items"]


@pytest.mark.parametrize("h,w,conn,density", [
    (47, 49, 8, 0.02), (48, 48, 4, 0.02), (49, 97, 8, 0.002), (96, 95, 4, 0.002), (145, 40, 8, 0.01),
    (8, 300, 4, 0.003), (200, 200, 8, 0.7), (200, 200, 8, 0.35), (200, 200, 4, 0.35), (200, 200, 4, 0.12),
    (150, 149, 8, 0.0002)])
def test_tile_edges_four_waves(h, w, conn, density):
    torch, iw = require_gpu()
    rng = np.random.default_rng(h * 131 + w + conn)
    B = (rng.random((h, w)) >= density).astype(np.uint8)
    B[rng.integers(h), rng.integers(w)] = 0
    announce("edt four waves", h, w, conn, density)
    ctx = iw.Context(0, wg_waves=4)
    try:
        check(torch, ctx, B, conn)
    finally:
        ctx.close()


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("conn", [4, 8])
def test_straight_fronts(conn, waves):
    torch, iw = require_gpu()
    ctx = iw.Context(0, wg_waves=waves)
    try:
        for k in range(4):
            B = np.ones((260, 310), np.uint8)
            if k == 0:
                B[131, :] = 0
            elif k == 1:
                B[:, 77] = 0
            elif k == 2:
                B[np.arange(260), np.arange(260)] = 0
            else:
                B[::16, :] = 0  # four fronts of 64 pixels a region: more than 256 sources a wave of four
                B[:, ::16] = 0
            announce("edt fronts", k, conn, waves)
            check(torch, ctx, B, conn)
    finally:
        ctx.close()


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("blocks", [1, 3, 8, 9, 20])
def test_dealing(blocks, waves):
    torch, iw = require_gpu()
    rng = np.random.default_rng(blocks)
    imgs = [(rng.random(s) >= d).astype(np.uint8) for s, d in (((400, 500), 0.01), ((49, 300), 0.3), ((700, 60), 0.001))]
    imgs[2][10, 10] = 0
    ctx = iw.Context(0, persistent_blocks=blocks, wg_waves=waves)
    try:
        announce("edt dealing", blocks, waves)
        for B in imgs:
            check(torch, ctx, B, 8)
        out = [[torch.empty(B.shape, dtype=torch.int32, device="cuda") for _ in range(2)] for B in imgs]
        ctx.run_batch([{"op": "edt", "binary": torch.from_numpy(B).cuda(), "sqdist": sq, "nearest": nr, "conn": 4}
                       for B, (sq, nr) in zip(imgs, out)])
        for B, (sq, nr) in zip(imgs, out):
            so, no = oracle.edt_rounds(B, 4)
            assert np.array_equal(sq.cpu().numpy(), so) and np.array_equal(nr.cpu().numpy(), no)
    finally:
        ctx.close()


@pytest.mark.parametrize("conn,depth", [(8, 0), (8, 1), (4, 16)])
def test_stage_depths_four_waves(conn, depth):
    torch, iw = require_gpu()
    B = synth.edt_input(700, 533, seed=12, coverage=0.25)
    ctx = iw.Context(0, wg_waves=4, stage_depth=depth)
    try:
        announce("edt stage depth, four waves", conn, depth)
        check(torch, ctx, B, conn)
    finally:
        ctx.close()
