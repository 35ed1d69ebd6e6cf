"""GPU parity of the split decode where its units, items and partials begin and end: rows per wave (16, 32, 64), items of
several units, heads of one item and of many, in a launch of its own and inside the selection's launch."""
import numpy as np
import pytest

import oracle
from workloads import make_cache

import harness as H

pytestmark = pytest.mark.gpu

# fp32 sums of up to 10^4 weighted values of size ~1 (weights sum to 1), the scores' own rounding (|x| <= 40: 40 x 2^-23)
# above it; the bar that the other parity tests hold this path to as well
TIGHT = 2e-4
MOST_INLINE = 512  # a head that keeps this many rows or fewer may be attended by the workgroup that selects it


def _whole(cache, exact_share=1.0, seed=0):
    """Every cluster of every segment retained, the first `exact_share` of a random order exact."""
    rng = np.random.default_rng(seed)
    exact, approx = [], []
    for i in range(cache.batch * cache.n_q_heads):
        b, h = divmod(i, cache.n_q_heads)
        seg = b * cache.n_kv_heads + h // cache.group
        n = int(cache.seg_cluster_ptr[seg + 1] - cache.seg_cluster_ptr[seg])
        order = rng.permutation(n)
        k = int(round(exact_share * n))
        exact.append(np.sort(order[:k]))
        approx.append(np.sort(order[k:]))
    return exact, approx


def _check_sets(cache, exact, approx):
    out, lse = H.gpu_sparse_decode(cache, exact, approx)
    g = H.GpuStep(out=out, lse=lse, exact=exact, approx=approx, n_exact_tokens=np.zeros(len(exact)))
    H.check_outputs(cache, oracle.Oracle(cache), g, tight=TIGHT)
    return out, lse


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 1023, 1025])
@pytest.mark.parametrize("share", [1.0, 0.5, 0.0])
def test_split_decode_of_few_rows(n, share):
    """Rows around every unit and item size, as tokens, as pseudo-tokens and mixed."""
    c = make_cache(batch=2, n_kv_heads=1, n_q_heads=2, context=[n, n + 7], mean_cluster=1 if share == 0.0 else 5,
                   size_lo=1, size_hi=16, q_scale=0.4, seed=101)
    _check_sets(c, *_whole(c, share, seed=n))


@pytest.mark.parametrize("heads, context", [(2, 9000), (32, 3000), (128, 700)])
def test_split_decode_inside_the_selection_launch(heads, context):
    """p1 = p2 = 1 leaves every row of every head to the queue: items of many units, of few, and many heads; heads with
    one row, none beyond the inline limit, and empty ones between them."""
    import paper_2602_05191_amd as dp
    n_seg = heads // 2
    ctx = [context + 61 * i for i in range(n_seg)]
    if n_seg > 3:
        ctx[0], ctx[1], ctx[2] = 1, 64, 65
    c = make_cache(batch=n_seg, n_kv_heads=1, n_q_heads=2, context=ctx, mean_cluster=7, size_hi=32, q_scale=0.4, seed=102)
    if n_seg > 3:
        c.cluster_sizes[int(c.seg_cluster_ptr[3]):int(c.seg_cluster_ptr[4])] = 0   # a segment with nothing in it
    orc = oracle.Oracle(c)
    for flags in (0, dp.DP_FLAG_SEPARATE_DECODE_LAUNCH):
        g = H.gpu_decode_attention(c, 1.0, 1.0, flags=flags)
        assert (g.n_exact_tokens > MOST_INLINE).sum() >= (heads - 8 if n_seg > 3 else heads)
        H.check_outputs(c, orc, g, tight=TIGHT)
        again = H.gpu_decode_attention(c, 1.0, 1.0, flags=flags)
        assert np.array_equal(g.out.view(np.uint32), again.out.view(np.uint32))
    # some heads flat, some peaked: both kinds of workgroup serve
    g = H.gpu_decode_attention(c, 0.9, 0.6)
    H.check_outputs(c, orc, g, tight=TIGHT)


@pytest.mark.parametrize("n", [70, 100, 300, MOST_INLINE + 3, MOST_INLINE + 65, 2000])
def test_split_decode_keeps_an_infinite_value_in_its_dimension(n):
    """An infinity in the segment's last V row, which the lanes without a row of their own name as well.  Lists given by
    the caller are never attended anywhere else; heads of a step are where they have more rows than their own workgroup
    takes."""
    import paper_2602_05191_amd as dp
    c = make_cache(batch=1, n_kv_heads=1, n_q_heads=4, context=n, mean_cluster=8, size_hi=32, q_scale=0.3, seed=103)
    c.v_cache[n - 1, 5] = 0x7F80
    outs = [H.gpu_sparse_decode(c, *_whole(c))[0]]
    for flags in (0, dp.DP_FLAG_SEPARATE_DECODE_LAUNCH):
        g = H.gpu_decode_attention(c, 1.0, 1.0, flags=flags)
        assert (g.n_exact_tokens == n).all()
        outs.append(g.out)
    for out in outs:
        assert np.isposinf(out[..., 5]).all() and np.isfinite(np.delete(out, 5, axis=-1)).all()


def test_split_decode_of_sets_with_an_empty_cluster():
    """A caller's exact list that names clusters without rows (they add nothing)."""
    c = make_cache(batch=1, n_kv_heads=1, n_q_heads=2, context=900, mean_cluster=6, size_hi=16, q_scale=0.4, seed=104)
    exact, approx = _whole(c, 0.8)
    empty = [int(e) for e in exact[0][[0, 3, 4, 40, -1]]]
    c.cluster_sizes[empty] = 0
    approx = [np.array([a for a in ap if a not in empty], dtype=np.int64) for ap in approx]
    _check_sets(c, exact, approx)


@pytest.mark.parametrize("at", [62, 63, 64])
def test_split_decode_of_sets_with_an_empty_cluster_behind_one_row_ones(at):
    """A wave looks 64 list entries up at a time: one-row clusters up to where the 64 end, then one without rows."""
    c = make_cache(batch=1, n_kv_heads=1, n_q_heads=2, context=1200, mean_cluster=6, size_hi=16, q_scale=0.4, seed=105)
    n = int(c.seg_cluster_ptr[1])
    c.cluster_sizes[:at] = np.minimum(c.cluster_sizes[:at], 1)
    c.cluster_sizes[at] = 0
    _check_sets(c, [np.arange(n - 20)] * 2, [np.arange(n - 20, n)] * 2)


@pytest.mark.parametrize("batch", [1, 33])
@pytest.mark.parametrize("budget", [(50, 2), (105, 4), (120, 4), (160, 4)])
def test_budget_heads_around_the_rows_their_own_workgroup_attends(budget, batch):
    """Launches of few and of many heads, budgets of some 80 to 220 rows: attended with the selection, by the decode
    launch, or some heads here and some there."""
    c = make_cache(batch=batch, n_kv_heads=1, n_q_heads=4, context=6000, mean_cluster=16, q_scale=0.4, seed=106)
    g = H.gpu_decode_attention(c, 0, 0, budget=budget)
    rows = np.array([t + len(a) for t, a in zip(g.n_exact_tokens, g.approx)])
    assert rows.min() > 64 and (budget[0] < 150 or rows.max() > 200)
    H.check_outputs(c, oracle.Oracle(c), g, tight=TIGHT)


@pytest.mark.parametrize("p1, fewest, most", [(0.1, 190, 300), (0.15, 330, 512), (0.18, 420, 600), (0.35, 1000, 1400)])
def test_flat_heads_around_the_rows_their_own_workgroup_attends(p1, fewest, most):
    """The search of 1024 threads per head (more than 4096 clusters): heads below 512 rows, on both sides, and beyond."""
    c = make_cache(batch=1, n_kv_heads=1, n_q_heads=16, context=9000, mean_cluster=2, size_hi=4, q_scale=0.3, seed=107)
    assert c.max_clusters_per_seg > 4096
    g = H.gpu_decode_attention(c, p1, 0.5, sm_scale=0.02)
    rows = np.array([t + len(a) for t, a in zip(g.n_exact_tokens, g.approx)])
    assert fewest < rows.min() and rows.max() < most, rows
    H.check_outputs(c, oracle.Oracle(c, sm_scale=0.02), g, tight=TIGHT)


@pytest.mark.parametrize("n", [128, 449, 512, 513, 640])
@pytest.mark.parametrize("lo, hi", [(0, 0), (0, 64), (64, 128)])
def test_split_decode_merges_few_and_many_partials(n, lo, hi):
    """Items of 64 rows in a launch this light: 2, 8, 9 and 10 partials, one of them without any weight (every row of it
    scores -inf)."""
    c = make_cache(batch=1, n_kv_heads=1, n_q_heads=2, context=n, mean_cluster=1, size_lo=1, size_hi=1, q_scale=0.4, seed=108)
    if hi > lo:
        c.q[..., 7] = 0x3F80
        c.k_cache[lo:hi, 7] = 0xFF80
    _check_sets(c, *_whole(c))
