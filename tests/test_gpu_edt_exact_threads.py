"""Exact distance transforms of rows whose column data exceed 64 KB of LDS, of two
widths at once from two threads with a context and a stream each, and of the widest
row accepted: no call fails, and each result is what the call gives alone."""
import threading

import numpy as np
import pytest

from tests.gpu_util import announce, require_gpu
from tests.test_gpu_edt_exact_index import by_columns

pytestmark = pytest.mark.gpu


def image(h, w):
    rng = np.random.default_rng(w)
    B = (rng.random((h, w)) >= 0.01).astype(np.uint8)
    B[0, 0] = 0
    return B


def test_two_widths_at_once():
    torch, iw = require_gpu()
    announce("edt exact, two threads")
    widths, errors, alone = (22000, 40000), [], {}
    inputs = {w: torch.from_numpy(image(2, w)).cuda() for w in widths}
    torch.cuda.synchronize()
    ctxs = {w: iw.Context(0) for w in widths}
    try:
        for w in widths:
            alone[w] = [t.clone() for t in ctxs[w].edt_exact(inputs[w])]
        torch.cuda.synchronize()

        def work(w):
            try:
                with torch.cuda.stream(torch.cuda.Stream()):
                    for _ in range(400):
                        got = ctxs[w].edt_exact(inputs[w])
                    torch.cuda.current_stream().synchronize()
                if not all(torch.equal(a, b) for a, b in zip(got, alone[w])):
                    errors.append((w, "differs"))
            except Exception as e:  # reported by the assertion below
                errors.append((w, repr(e)))

        threads = [threading.Thread(target=work, args=(w,)) for w in widths]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
    finally:
        torch.cuda.synchronize()
        for c in ctxs.values():
            c.close()
    assert not errors, errors[:3]


@pytest.mark.parametrize("w", [21845, 21846, 46340])
def test_widest_rows(w):
    torch, iw = require_gpu()
    announce("edt exact, widest rows", w)
    B = image(1, w)
    ctx = iw.Context(0)
    try:
        sq, nr = (t.cpu().numpy() for t in ctx.edt_exact(torch.from_numpy(B).cuda()))
    finally:
        ctx.close()
    es, en = by_columns(B)
    assert np.array_equal(sq, es) and np.array_equal(nr, en)
