"""GPU parity at the sizes where a kernel's tiles, splits or dispatch rules end."""
import numpy as np
import pytest

import oracle
from workloads import make_cache

import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_q_heads", [1, 5, 16, 20])
def test_dense_decode_at_tile_and_split_edges(n_q_heads):
    """16-row tiles, 64-row steps of a workgroup, 256-row splits, and passes of 16 heads."""
    ctx = [1, 15, 16, 17, 63, 64, 65, 255, 256, 257, 511, 513, 1100]
    c = make_cache(batch=len(ctx), n_kv_heads=1, n_q_heads=n_q_heads, context=ctx, mean_cluster=16, q_scale=0.7, seed=61)
    out, lse = H.gpu_dense_decode(c, H.segment_rows(c))
    ref, ref_lse, _ = oracle.Oracle(c).dense_step(n_threads=4)
    # fp32 sums of at most 1100 weighted values of size ~1 (weights sum to 1): a few times 2^-24 x sqrt(rows), the
    # scores' own rounding times their size (|x| <= 40: 40 x 2^-23) above it
    assert np.abs(out - ref).max() <= 2e-5
    assert np.abs(lse - ref_lse).max() <= 2e-5 * np.abs(ref_lse).max()


def test_dense_decode_deals_rows_out_over_ragged_segments():
    """Shares of 64-row chunks that end one segment and begin the next, empty segments between them, and (512 heads: 32
    partial slots each) a segment with more chunks than slots."""
    ctx = [4000, 1, 700, 64, 2500, 65, 3000, 128]
    c = make_cache(batch=len(ctx), n_kv_heads=4, n_q_heads=64, context=ctx, mean_cluster=16, q_scale=0.7, seed=62)
    rows = H.segment_rows(c)
    rows[[5, 6, 30]] = 0   # these heads attend to nothing
    out, lse = H.gpu_dense_decode(c, rows)
    ref, ref_lse, _ = oracle.Oracle(c).dense_step(n_threads=4)
    empty = np.repeat(rows == 0, 16).reshape(out.shape[:2])
    assert (out[empty] == 0).all() and np.isneginf(lse[empty]).all()
    # as above; 4000 rows
    assert np.abs(out - ref)[~empty].max() <= 2e-5
    assert np.abs(lse - ref_lse)[~empty].max() <= 2e-5 * np.abs(ref_lse).max()
