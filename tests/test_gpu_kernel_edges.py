"""GPU parity at the sizes where a kernel's tiles, splits or dispatch rules end."""
import numpy as np
import pytest

import oracle
from workloads import make_cache

import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_q_heads", [1, 5, 16, 20])
def test_dense_decode_at_tile_and_split_edges(n_q_heads):
    """16-row tiles, 64-row chunks (here one per workgroup), and passes of 16 heads."""
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


@pytest.mark.parametrize("n_seg, lengths", [
    (9, [1, 320]), (9, [1, 321]), (127, [17, 64, 512]), (128, [17, 64, 512]), (128, [16, 513]), (511, [1, 65, 1024]),
    (512, [1, 65, 1024]), (512, [1, 63, 1025]), (64, [1, 64, 129, 1500]), (65, [1, 64, 129, 1500]), (4096, [1, 2, 1030]),
    (4097, [1, 2, 1030])])
def test_dense_decode_of_many_segments(n_seg, lengths):
    """Segments taken whole by a workgroup and segments whose chunks are dealt out, at the lengths and counts where one
    form ends; looked up by one lane each, by several, by all; segments without rows."""
    rng = np.random.default_rng(n_seg)
    ctx = [int(x) for x in rng.choice(lengths, size=n_seg)]
    if n_seg > 4000:   # (few long ones)
        ctx = [n if n < 1000 or i % 97 == 0 else 3 for i, n in enumerate(ctx)]
    ctx[-1] = max(lengths)
    heads = 20 if n_seg < 10 else 2   # (two passes over a group of 20)
    c = make_cache(batch=n_seg, n_kv_heads=1, n_q_heads=heads, context=ctx, mean_cluster=64, size_hi=256, q_scale=0.7,
                   seed=67)
    rows = H.segment_rows(c)
    rows[rng.choice(n_seg - 1, n_seg // 8, replace=False)] = 0
    out, lse = H.gpu_dense_decode(c, rows)
    ref, ref_lse, _ = oracle.Oracle(c).dense_step(n_threads=4)
    full = rows > 0
    assert (out[~full] == 0).all() and np.isneginf(lse[~full]).all()
    assert np.abs(out - ref)[full].max() <= 2e-5
    assert np.abs(lse - ref_lse)[full].max() <= 2e-5 * np.abs(ref_lse).max()


BF16 = {"inf": 0x7F80, "-inf": 0xFF80, "one": 0x3F80, "huge": 0x7F62}   # huge = 3.004e38


def _dense_against_oracle(c, rtol=2e-5):
    """Equal non-finite elements, the others as above (relative to their size where that is above 1)."""
    out, lse = H.gpu_dense_decode(c, H.segment_rows(c))
    ref, ref_lse, _ = oracle.Oracle(c).dense_step(n_threads=4)
    assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.array_equal(np.isinf(out), np.isinf(ref))
    fin = np.isfinite(ref)
    assert (np.abs(out[fin] - ref[fin]) <= rtol * np.maximum(np.abs(ref[fin]), 1.0)).all()
    assert np.abs(lse - ref_lse).max() <= 2e-5 * np.maximum(np.abs(ref_lse).max(), 1.0)
    return out


@pytest.mark.parametrize("n", [1, 37, 48, 64, 100, 1000])
def test_dense_decode_keeps_an_infinite_value_in_its_dimension(n):
    """An infinity in the segment's last V row, at lengths that are and are not multiples of the tile of 16."""
    c = make_cache(batch=1, n_kv_heads=1, n_q_heads=4, context=n, mean_cluster=16, q_scale=0.3, seed=63)
    c.v_cache[n - 1, 5] = BF16["inf"]
    out = _dense_against_oracle(c)
    assert np.isposinf(out[..., 5]).all() and np.isfinite(np.delete(out, 5, axis=-1)).all()


@pytest.mark.parametrize("n, lo, hi", [(300, 64, 128), (300, 0, 16), (1000, 0, 900), (37, 32, 37)])
def test_dense_decode_rows_that_score_minus_infinity_have_no_weight(n, lo, hi):
    """Whole tiles and whole 64-row chunks whose every row scores -inf, in front of, between and behind the others."""
    c = make_cache(batch=1, n_kv_heads=1, n_q_heads=4, context=n, mean_cluster=16, q_scale=0.3, seed=64)
    c.q[..., 7] = BF16["one"]
    c.k_cache[lo:hi, 7] = BF16["-inf"]
    assert np.isfinite(_dense_against_oracle(c)).all()


@pytest.mark.parametrize("gap", [86, 90, 95])
def test_dense_decode_weights_below_the_normal_range_count(gap):
    """One row of weight e^-gap (below 2^-126 from 88 on) with values of 3e38: the product is of ordinary size."""
    c = make_cache(batch=1, n_kv_heads=1, n_q_heads=4, context=40, mean_cluster=16, q_scale=0.3, seed=65)
    c.q[:], c.k_cache[:], c.v_cache[:] = 0, 0, 0
    c.q[..., 0] = BF16["one"]
    c.k_cache[1:, 0] = np.float32([-gap * 128 ** 0.5]).view(np.uint32)[0] >> 16
    c.v_cache[1, 5] = BF16["huge"]
    # the weight is a multiple of 2^-149, so it is off by up to 2^-150 / e^-gap of itself; the score (up to 137 in base
    # 2) is rounded to 2^-17 at each of three steps, and that is what the weight is off by as well
    bar = 2.0 ** -150 / np.exp(-gap) + 3 * 2.0 ** -17
    out = _dense_against_oracle(c, rtol=bar)
    assert (out[..., 5] > 0).all()


@pytest.mark.parametrize("seed", [66, 67])
def test_dense_decode_long_sums_keep_fp32_precision(seed):
    """One segment of 16384 rows among 128 (2048 heads: 8 partial slots each, so a wave sums 592 rows one after the
    other) with weights of similar size and values of both signs."""
    ctx = [16384] + [1] * 127
    c = make_cache(batch=128, n_kv_heads=1, n_q_heads=16, context=ctx, mean_cluster=16, q_scale=0.05, seed=seed)
    out, _ = H.gpu_dense_decode(c, H.segment_rows(c))
    ref, _, _ = oracle.Oracle(c).dense_step(n_threads=4)
    rel = np.linalg.norm(out[0] - ref[0]) / np.linalg.norm(ref[0])
    # A chain of n fp32 sums of random sign is off by 2^-24 / sqrt(3) x sqrt(n / 2) of the result: 16 rows of a tile and
    # 37 tiles give 1.8e-7, one chain over 592 rows 5.9e-7.  Scores of rms 3 (base 2), off by 6e-8 and rounded twice,
    # add 2.5e-7: together 3.1e-7 against 6.4e-7.
    assert rel <= 4.2e-7, rel


@pytest.mark.parametrize("n", [40001, 40017])
@pytest.mark.parametrize("n_q_heads", [5, 20])
def test_dense_decode_shares_of_several_chunks(n, n_q_heads):
    """One segment with more chunks than partial slots: shares of three chunks, so a wave has several tiles, in passes of
    5, 16 and 4 heads; scores grow along the rows, so the maximum moves in late tiles."""
    c = make_cache(batch=1, n_kv_heads=1, n_q_heads=n_q_heads, context=n, mean_cluster=64, size_hi=256, q_scale=0.3,
                   seed=68)
    c.q[..., 0] = BF16["one"]
    c.k_cache[:, 0] = np.linspace(-60, 60, n).astype(np.float32).view(np.uint32) >> 16
    _dense_against_oracle(c)


def _tokens(rows, clusters, spread, seed):
    """Token-order K / V with ids drawn as ``spread`` says."""
    from workloads import TokenOrderInput
    rng = np.random.default_rng(seed)
    ids = []
    for n, kc in zip(rows, clusters):
        if spread == "uniform":
            a = rng.integers(0, kc, size=n)
        elif spread == "one_bin":       # (nearly) everything in the last 16 clusters: one long run
            a = np.where(rng.random(n) < 0.98, kc - 1 - rng.integers(0, min(kc, 16), size=n), rng.integers(0, kc, size=n))
        else:                           # runs of equal ids, some of them invalid
            a = np.repeat(rng.integers(-1, kc + 1, size=n // 50 + 1), 50)[:n]
        ids.append(a)
    rows = np.asarray(rows, np.int32)
    bits = rng.integers(0, 1 << 16, size=(2, int(rows.sum()), 128), dtype=np.uint16)
    bits = (bits & 0x807F) | np.uint16(0x3F80) - (bits & 0x0300)   # finite values of a few exponents, both signs
    return TokenOrderInput(n_seg=len(rows), head_dim=128, k_tokens=bits[0].copy(), v_tokens=bits[1].copy(),
                           assignment=np.concatenate(ids).astype(np.int32),
                           seg_row_base=np.concatenate([[0], np.cumsum(rows)[:-1]]).astype(np.int64), seg_rows=rows,
                           seg_cluster_ptr=np.concatenate([[0], np.cumsum(clusters)]).astype(np.int32))


@pytest.mark.parametrize("spread", ["uniform", "one_bin", "runs"])
@pytest.mark.parametrize("clusters", [1, 16, 17, 33, 1000, 1024, 1025])
def test_build_at_block_bin_and_list_edges(clusters, spread):
    """Token blocks of 4096, waves of 64, bins of 16 clusters, runs above and below the 1024 tokens whose list stays in
    LDS, chunks of 64 rows.  Bit-exact, as in test_gpu_build."""
    from test_gpu_build import check_build, gpu_build
    rows = [1, 63, 65, 1023, 1025, 4095, 4096, 4097, 9000]
    t = _tokens(rows, [clusters] * len(rows), spread, seed=70 + clusters)
    check_build(t, gpu_build(t), oracle.build_cluster_cache(t))


@pytest.mark.parametrize("longest", [64, 1024, 1025, 4096, 4097, 8192, 8193])
@pytest.mark.parametrize("clusters", [1, 17, 700])
def test_build_of_short_segments(longest, clusters):
    """Segments that a workgroup sorts alone (up to 1024, 4096 and 8192 tokens) and the first length beyond, with tokens
    that have no valid cluster and a segment without rows.  Bit-exact, as above."""
    from test_gpu_build import check_build, gpu_build
    rng = np.random.default_rng(longest + clusters)
    rows = [longest, 1, max(1, longest // 2), 0, longest - 1, 63]
    t = _tokens(rows, [clusters] * len(rows), "runs" if clusters == 17 else "uniform", seed=longest)
    t.assignment[rng.choice(len(t.assignment), max(1, len(t.assignment) // 50), replace=False)] = -1
    check_build(t, gpu_build(t), oracle.build_cluster_cache(t))


def test_build_without_any_cluster_leaves_every_token_out():
    from test_gpu_build import gpu_build
    t = _tokens([5, 4097], [1, 1], "uniform", seed=79)
    t.seg_cluster_ptr[:] = 0
    assert (gpu_build(t)["token_row"] == -1).all()


def test_build_with_words_of_64_bits():
    """A bound of 2^28 rows per segment: the sort's words take 64 bits.  Same outputs as with the exact bound."""
    import torch
    import paper_2602_05191_amd as dp
    t = _tokens([5000], [100], "one_bin", seed=81)
    up = lambda a, dt: torch.from_numpy(np.ascontiguousarray(a).view(dt)).cuda()
    out = []
    for bound in (5000, 1 << 28):
        pf = dp.Prefill(up(t.k_tokens, np.int16), up(t.v_tokens, np.int16), up(t.assignment, np.int32),
                        up(t.seg_row_base, np.int64), up(t.seg_rows, np.int32), up(t.seg_cluster_ptr, np.int32),
                        100, 100, bound)
        bufs = [torch.full(s, -7, dtype=d, device="cuda") for s, d in
                (((5000, 128), torch.int16), ((5000, 128), torch.int16), ((100,), torch.int32), ((100,), torch.int32),
                 ((100, 128), torch.int16), ((100, 128), torch.int16))]
        row = torch.full((5000,), -7, dtype=torch.int32, device="cuda")
        ws = torch.empty(dp.dp_build_workspace_bytes(pf), dtype=torch.uint8, device="cuda")
        dp.dp_build_cluster_cache(pf, *bufs, ws, token_row=row)
        torch.cuda.synchronize()
        out.append(bufs + [row])
    for a, b in zip(*out):
        assert torch.equal(a, b)


def test_build_without_any_row_needs_no_workspace():
    import torch
    import paper_2602_05191_amd as dp
    dev = lambda *a, **k: torch.full(*a, device="cuda", **k)
    k = dev((1, 128), 0x7FC0, dtype=torch.int16)
    ptr = torch.tensor([0, 3, 40], dtype=torch.int32, device="cuda")
    pf = dp.Prefill(k, k, dev((1,), 0, dtype=torch.int32), dev((2,), 0, dtype=torch.int64),
                    dev((2,), 0, dtype=torch.int32), ptr, 40, 37, 0)
    assert dp.dp_build_workspace_bytes(pf) == 0
    off, size = (dev((40,), -7, dtype=torch.int32) for _ in range(2))
    kc, vc = (dev((40, 128), 0x7FC0, dtype=torch.int16) for _ in range(2))
    dp.dp_build_cluster_cache(pf, k.clone(), k.clone(), off, size, kc, vc, torch.empty(0, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    for out in (off, size, kc, vc):
        assert (out == 0).all()


@pytest.mark.parametrize("clusters", [2, 17])
def test_kmeans_update_on_long_clusters(clusters):
    """The keys-only move (two halves of a workgroup take the clusters in turn) over runs of 64 to 9000 rows: after
    one round from given, well separated centroids the new centroids are the oracle's bits."""
    import paper_2602_05191_amd as dp
    from test_gpu_kmeans import gpu_fit, grouped_keys
    rows = [64, 65, 1500, 9000]
    t = grouped_keys(83, rows=rows, clusters=[clusters] * len(rows), groups=clusters)
    ref_c, ref_a = oracle.kmeans_fit(t, None, 1, oracle.KMEANS_INIT_STRIDED)
    got_c, got_a, _ = gpu_fit(t, None, 1, dp.DP_KMEANS_INIT_STRIDED)
    assert np.array_equal(got_a, ref_a) and np.array_equal(got_c, ref_c)


@pytest.mark.parametrize("last", [6010, 1908, 1907, 60])
def test_kmeans_assign_same_bits_whatever_the_launch(last):
    """Eight segments together take 128 tokens per wave (2048 or 1536 centroids per segment on average) or 64 (fewer);
    one alone takes 32.  The same products are summed in the same order: index and score are equal to the bit, at token
    and centroid counts around the tiles, for equal centroids in one quad and far apart, and with NaN and inf."""
    import torch
    import paper_2602_05191_amd as dp
    rows = [32769, 1, 127, 128, 129, 511, 513, 2049]
    clusters = [4099, 2048, 1, 3, 0, 66, 4163, last]
    g = torch.Generator().manual_seed(91)
    keys = torch.randn(sum(rows), 128, generator=g).bfloat16()
    cent = torch.randn(sum(clusters), 128, generator=g).bfloat16()
    cent[[5, 6, 70, 4098]] = cent[4].clone()          # one quad and the next, another block, the last
    cent[4099 + 17, 3], cent[4099 + 18, 4], cent[4099 + 40, 5] = float("nan"), float("inf"), float("-inf")
    keys[100, 7], keys[101, 8] = float("nan"), float("inf")
    keys, cent = keys.cuda(), cent.cuda()
    base, ptr = np.concatenate([[0], np.cumsum(rows)]), np.concatenate([[0], np.cumsum(clusters)])

    def assign(segs):
        first, end = ptr[segs[0]], ptr[segs[-1] + 1]
        dev = lambda a, dt: torch.from_numpy(np.asarray(a, dt)).cuda()
        pf = dp.Prefill(keys, keys, torch.zeros(len(keys), dtype=torch.int32, device="cuda"), dev(base[segs], np.int64),
                        dev([rows[s] for s in segs], np.int32), dev(ptr[segs[0]:segs[-1] + 2] - first, np.int32),
                        int(end - first), max(clusters[s] for s in segs), max(rows[s] for s in segs))
        ws = torch.empty(max(dp.dp_kmeans_workspace_bytes(pf), 256), dtype=torch.uint8, device="cuda")
        asg = torch.full((len(keys),), -7, dtype=torch.int32, device="cuda")
        score = torch.full((len(keys),), -7.0, device="cuda")
        dp.dp_kmeans_assign(pf, cent[first:max(end, first + 1)].contiguous(), asg, ws, best_score=score)
        torch.cuda.synchronize()
        return asg, score

    asg, score = assign(list(range(8)))
    assert not torch.isin(asg[:rows[0]], torch.tensor([5, 6, 70, 4098], device="cuda")).any()
    for s in range(8):
        one, one_score = assign([s])
        at = slice(int(base[s]), int(base[s + 1]))
        assert torch.equal(asg[at], one[at]) and torch.equal(score[at], one_score[at]), f"segment {s}"


@pytest.mark.parametrize("rows", [100, 20000])
@pytest.mark.parametrize("clusters", [1, 63, 64, 65, 1024, 1025])
def test_kmeans_assign_same_bits_whoever_works_out_the_norms(rows, clusters):
    """A segment by itself (up to 1024 centroids: every workgroup takes the norms of the centroids it stages) and beside
    one with so many centroids that a launch in front does; a centroid with a NaN, one with an infinity, one of zeros."""
    import torch
    import paper_2602_05191_amd as dp
    g = torch.Generator().manual_seed(92)
    keys = torch.randn(rows + 10, 128, generator=g).bfloat16().cuda()
    cent = (torch.randn(clusters + 9000, 128, generator=g) * 3).bfloat16()
    if clusters > 60:
        cent[5, 3], cent[6, 127], cent[7] = float("nan"), float("inf"), 0.0
    cent = cent.cuda()
    got = []
    for segs in (1, 2):
        dev = lambda a, dt: torch.from_numpy(np.asarray(a, dt)[:segs + (len(a) == 3)]).cuda()
        pf = dp.Prefill(keys, keys, torch.zeros(len(keys), dtype=torch.int32, device="cuda"), dev([0, rows], np.int64),
                        dev([rows, 10], np.int32), dev([0, clusters, clusters + 9000], np.int32),
                        clusters + 9000 * (segs - 1), 9000 if segs == 2 else clusters, rows)
        ws = torch.empty(max(dp.dp_kmeans_workspace_bytes(pf), 256), dtype=torch.uint8, device="cuda")
        asg = torch.full((len(keys),), -7, dtype=torch.int32, device="cuda")
        score = torch.full((len(keys),), -7.0, device="cuda")
        dp.dp_kmeans_assign(pf, cent, asg, ws, best_score=score)
        torch.cuda.synchronize()
        got.append((asg[:rows], score[:rows]))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
