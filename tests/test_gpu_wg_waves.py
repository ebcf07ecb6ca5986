"""The automatic workgroup size and both explicit ones give the same results:
reconstructions, and distance transforms on both sides of 512 tiles."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves", [0, 4, 8])
@pytest.mark.parametrize("conn", [4, 8])
def test_workgroup_sizes(waves, conn):
    torch, iw = require_gpu()
    rng = np.random.default_rng(conn)
    ctx = iw.Context(0, wg_waves=waves)
    try:
        for h, w in ((150, 333), (24 * 48, 21 * 48), (24 * 48, 22 * 48 + 1)):  # 504 and 552 tiles
            announce("workgroup size", waves, conn, h, w)
            B = (rng.random((h, w)) >= 0.003).astype(np.uint8)
            sq, nr = ctx.edt(torch.from_numpy(B).cuda(), conn)
            st = ctx.stats()
            so, no, ost = oracle.edt_rounds(B, conn, return_stats=True)
            assert st["status"] == 0 and np.array_equal(sq.cpu().numpy(), so) and np.array_equal(nr.cpu().numpy(), no)
            assert st["rounds"] == ost["rounds"] and st["items"] == ost["items"]
            I = (np.cumsum(rng.integers(-3, 4, (h, w)), axis=1) + 128).clip(0, 255).astype(np.uint8)
            J = np.where(rng.random((h, w)) < 0.99, np.maximum(I, 40) - 40, I).astype(np.uint8)
            got = ctx.morph_recon(torch.from_numpy(J).cuda(), torch.from_numpy(I).cuda(), conn).cpu().numpy()
            assert np.array_equal(got, oracle.mr_fh(J, I, conn))
    finally:
        ctx.close()
