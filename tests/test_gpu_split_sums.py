"""The backward-weight partial sums of few and of many pixel splits (64 is
where more threads share an element), with and without the bias gradient,
against the oracle."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_within, dev, host

pytestmark = pytest.mark.gpu


# First layers (no output tile but one): the splits grow with the pixels.
@pytest.mark.parametrize("shape", [
    (1, 3, 9, 9, 16, 3, 3, 1, 1, 1),
    (1, 3, 64, 65, 17, 3, 3, 1, 1, 1),
    (2, 3, 95, 97, 16, 3, 3, 1, 1, 1),
    (2, 1, 180, 181, 20, 3, 3, 1, 1, 1),
    (4, 3, 224, 224, 16, 3, 3, 2, 1, 1),
    (4, 4, 224, 224, 24, 3, 3, 1, 1, 1),
], ids=lambda s: "x".join(map(str, s)))
def test_splits(shape):
    import paper_1903_06934_amd as m
    N, C, H, W, K, R, S, st, pad, G = shape
    P, Q = oracle.out_size(H, R, st, pad), oracle.out_size(W, S, st, pad)
    d = workloads.make_inputs(shape, P, Q, seed=(81, H), init="he")
    x, dy = dev(d["x"]), dev(d["dy"])
    dw, db = m.conv_bwd_weight(x, dy, (R, S), st, pad, G)
    dw_ref, adw, db_ref, adb = oracle.conv_bwd_weight(shape, d["x"], d["dy"])
    assert_within(host(dw), dw_ref, adw, "dw")
    assert_within(host(db), db_ref, adb, "db")
    alone, _ = m.conv_bwd_weight(x, dy, (R, S), st, pad, G, with_bias=False)
    assert np.array_equal(host(alone).view(np.uint32), host(dw).view(np.uint32))
