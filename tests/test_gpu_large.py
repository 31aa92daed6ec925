"""Launch-splitting paths at sizes where they occur, on sampled elements
against the oracle's gather forms:

* batch chunking: a batch whose input tensor exceeds 2^29 elements runs as
  several launches of whole images (here 2 + 1 images of 176 x 1024 x 1024);
* the explicit plan's column chunks: 256 MB of column tensor a chunk (here
  2 + 1 images of a 64-channel 224 x 224 layer), for each pass."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_within, dev, host, sample_indices

pytestmark = pytest.mark.gpu


def _gpu_all(shape, d, ws=None):
    import paper_1903_06934_amd as m
    N, C, H, W, K, R, S, st, pad, G = shape
    y = host(m.conv_fwd(dev(d["x"]), dev(d["w"]), dev(d["b"]), st, pad, G))
    dx = host(m.conv_bwd_data(dev(d["dy"]), dev(d["w"]), (H, W), st, pad, G))
    dw, db = m.conv_bwd_weight(dev(d["x"]), dev(d["dy"]), (R, S), st, pad, G)
    return y, dx, host(dw), host(db)


def _check_sampled(shape, d, y, dx, dw, db, what, dw_count=256):
    N, C, H, W, K, R, S, st, pad, G = shape
    rng = np.random.default_rng(list(shape))
    idx = sample_indices(y.shape, rng, groups=G)
    v, a = oracle.conv_fwd_at(shape, d["x"], d["w"], d["b"], idx)
    assert_within(y.ravel()[idx], v, a, f"{what} fwd")
    idx = sample_indices(dx.shape, rng, groups=G)
    v, a = oracle.conv_bwd_data_at(shape, d["dy"], d["w"], idx)
    assert_within(dx.ravel()[idx], v, a, f"{what} bwd_data")
    idx = sample_indices(dw.shape, rng, count=dw_count, groups=1, channel_axis=0)
    v, a = oracle.conv_bwd_weight_at(shape, d["x"], d["dy"], idx)
    assert_within(dw.ravel()[idx], v, a, f"{what} bwd_weight")
    v, a = oracle.bias_grad(d["dy"])
    assert_within(db, v, a, f"{what} bias_grad")


def test_batch_chunking():
    shape = (3, 176, 1024, 1024, 16, 3, 3, 1, 1, 1)
    d = workloads.make_inputs(shape, 1024, 1024, seed=(90, 1), init="he")
    y, dx, dw, db = _gpu_all(shape, d)
    _check_sampled(shape, d, y, dx, dw, db, "chunked")


def test_explicit_plan_column_chunks():
    import paper_1903_06934_amd as m
    shape = (3, 64, 224, 224, 32, 3, 3, 1, 1, 1)
    d = workloads.make_inputs(shape, 224, 224, seed=(91, 1), init="he")
    try:
        for p in (m.PASS_FWD, m.PASS_BWD_DATA, m.PASS_BWD_WEIGHT):
            n = m.plan_count(p, shape)
            ex = [i for i in range(n) if m.plan_name(p, shape, i).startswith("explicit")]
            assert ex and "(2 images a chunk)" in m.plan_name(p, shape, ex[0])
            m.plan_set(p, shape, ex[0])
        y, dx, dw, db = _gpu_all(shape, d)
    finally:
        m.plan_clear()
    _check_sampled(shape, d, y, dx, dw, db, "explicit")


def test_fast_filtering_just_below_the_offset_limit():
    """Outputs of 2^29 - 512 elements on a map of odd height and width, whose
    last tiles have no second row or column: nothing that lies past them may
    come back to the start of the buffer.  Forward, and the same layer's
    mirror image backward; backward-weight reads the large tensor."""
    import torch
    import paper_1903_06934_amd as m
    H, W, few, many = 1025, 1023, 32, 512
    gen = torch.Generator(device="cuda").manual_seed(92)
    small = torch.randn(1, few, H, W, device="cuda", generator=gen)
    plane = np.arange(2 * W), np.arange((H - 2) * W, H * W)
    rng = np.random.default_rng(92)
    at = lambda c, i: c * H * W + i  # noqa: E731
    idx = np.unique(np.concatenate([at(0, plane[0]), at(0, plane[1]), at(many - 1, plane[0]),
                                    at(many - 1, plane[1]), rng.integers(0, many * H * W, 2048)]))

    def fast(p, shape):
        return [m.plan_name(p, shape, i).startswith("fast filtering")
                for i in range(m.plan_count(p, shape))].index(True)

    try:
        shape = (1, few, H, W, many, 3, 3, 1, 1, 1)
        w = torch.randn(many, few, 3, 3, device="cuda", generator=gen)
        m.plan_set(m.PASS_FWD, shape, fast(m.PASS_FWD, shape))
        got = host(m.conv_fwd(small, w, None, 1, 1, 1))
        v, a = oracle.conv_fwd_at(shape, host(small), host(w), None, idx)
        assert_within(got.ravel()[idx], v, a, "fwd")
        del got

        shape = (1, many, H, W, few, 3, 3, 1, 1, 1)
        w = torch.randn(few, many, 3, 3, device="cuda", generator=gen)
        m.plan_set(m.PASS_BWD_DATA, shape, fast(m.PASS_BWD_DATA, shape))
        got = host(m.conv_bwd_data(small, w, (H, W), 1, 1, 1))
        v, a = oracle.conv_bwd_data_at(shape, host(small), host(w), idx)
        assert_within(got.ravel()[idx], v, a, "bwd_data")
        del got

        x = torch.randn(1, many, H, W, device="cuda", generator=gen)
        m.plan_set(m.PASS_BWD_WEIGHT, shape, fast(m.PASS_BWD_WEIGHT, shape))
        got = host(m.conv_bwd_weight(x, small, (3, 3), 1, 1, 1, with_bias=False)[0])
        idx = np.unique(np.concatenate([np.arange(0, got.size, 3001), np.arange(got.size - 9, got.size)]))
        v, a = oracle.conv_bwd_weight_at(shape, host(x), host(small), idx)
        assert_within(got.ravel()[idx], v, a, "bwd_weight")
    finally:
        m.plan_clear()
