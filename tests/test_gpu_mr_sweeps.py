"""Reconstruction sweeps of a tile where only some chunks of its lines have
anything to do: few raised pixels in smooth and in rough masks, sides at and
around the tile's, and every cap of sweep iterations down to one.  Bytes equal
the oracle's."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("conn", [4, 8])
@pytest.mark.parametrize("cap", [0, 1, 2, 3, 8])
@pytest.mark.parametrize("h,w", [(40, 40), (64, 64), (63, 65), (200, 130)])
def test_sparse_changes(h, w, cap, conn):
    torch, iw = require_gpu()
    rng = np.random.default_rng(h * 997 + w + 10 * cap + conn)
    ctx = iw.Context(0, mr_max_sweeps=cap, mr_seed_sweeps=cap)
    try:
        announce("sparse sweeps", h, w, conn, cap)
        for step, keep in ((3, 0.97), (40, 0.999), (1, 0.9), (3, 0.5)):
            I = (np.cumsum(rng.integers(-step, step + 1, (h, w)), axis=1) + 128).clip(0, 255).astype(np.uint8)
            J = np.where(rng.random((h, w)) < keep, np.maximum(I, 40) - 40, I).astype(np.uint8)
            got = ctx.morph_recon(torch.from_numpy(J).cuda(), torch.from_numpy(I).cuda(), conn).cpu().numpy()
            assert np.array_equal(got, oracle.mr_fh(J, I, conn))
    finally:
        ctx.close()
