"""Host-side check of the sampler's plan (no GPU): over random layer structures of the kind
the workloads are drawn from, the speculative threshold that the plan's sample would give
keeps at least k and at most `capacity` entries of the row - the condition under which a
worker is served from its candidate list and not from its dense row.

The plan (tile positions, target rank, list capacity) comes from the library through
gtopk_debug_plan; the estimate is modelled here with numpy: the threshold is the plan's
target-th largest magnitude among the sampled elements, rounded down to the edge of a
histogram bucket (the sampler's buckets are at most 1/64 of the magnitude wide).  A miss
would cost time only (the select is exact whatever it filters with), so this is a check of
the margin, not of correctness.  The same for both ends of the brackets that steps of large densities take instead."""
import numpy as np
import pytest

from paper_1901_04359_amd import binding as B


def _row(rng, m, nseg):
    """Gaussian row in `nseg` contiguous segments: lengths from weights exp(U(0, ln 1000)),
    standard deviations log-uniform in [1e-5, 1e-2] (the recipe of the large configurations)."""
    w = np.exp(rng.uniform(0.0, np.log(1000.0), nseg))
    lens = np.maximum(1, (w / w.sum() * m).astype(np.int64))
    lens[-1] = m - lens[:-1].sum()
    assert lens[-1] > 0
    sig = np.exp(rng.uniform(np.log(1e-5), np.log(1e-2), nseg)).astype(np.float32)
    x = rng.standard_normal(m, dtype=np.float32)
    x *= np.repeat(sig, lens)
    return x


# rank: expected sample rank of the k-th key; most: candidates per k, at most.  At rank r the target lies 5.5 standard
# deviations above r, and the number of candidates varies about that by some standard deviations of the target.
@pytest.mark.parametrize("nseg", [8, 54, 400])
@pytest.mark.parametrize("m,k,P,tile,most", [
    (2_555_703, 2_556, 32, 64, 2.5),          # the large sample, rank 256
    (3_000_017, 30_000, 32, 64, 2.5),
    (2_000_000, 2_000, 8, 16, 4.5),           # one block per worker: rank 16 for k <= 4096
    (1_000_003, 4_096, 4, 16, 3.0),           # (rank 67: the sample of a short row is large for its k)
    (1_000_003, 4_097, 4, 16, 3.0),
    (8_000_003, 16_500, 4, 16, 3.0),          # rank 64
    (3_000_017, 5_860, 8, 16, 3.0),
    (3_000_017, 4_096, 8, 16, 4.5),           # rank 22 at the shortest list for it (5 k)
])
def test_sample_plan_keeps_between_k_and_capacity(m, k, P, tile, most, nseg):
    try:
        plan = B.gtopk_debug_plan(m, k, P)
    except OSError as e:          # library not built
        pytest.skip(str(e))
    assert plan["tile_len"] == tile
    t = np.arange(plan["n_tiles"], dtype=np.int64)[:, None] * plan["tile_stride"]
    pos = (t + np.arange(plan["tile_len"], dtype=np.int64)[None, :]).ravel()
    pos = pos[pos < m]
    assert pos.size < m and plan["target"] <= pos.size
    ratios = []
    for trial in range(6):
        rng = np.random.default_rng(100 * nseg + trial)
        mag = np.abs(_row(rng, m, nseg))
        thr = np.sort(mag[pos])[::-1][plan["target"] - 1]
        kept = int((mag >= thr).sum())                               # with the exact sample key
        kept_lo = int((mag >= thr * np.float32(1.0 - 1.0 / 64)).sum())   # with a bucket edge below it
        assert kept >= k, f"trial {trial}: the threshold keeps {kept} < k = {k}"
        assert kept_lo <= plan["capacity"], f"trial {trial}: {kept_lo} > capacity {plan['capacity']}"
        ratios.append(kept_lo / k)
    assert max(ratios) < most, ratios     # the margin is a fraction of k (a multiple for the smallest samples)


@pytest.mark.parametrize("m,k,P", [(8_193, 20, 4), (9_000, 64, 64), (16_384, 50, 4), (269_722, 270, 8)])
def test_the_plan_of_the_few_launch_path_has_one_tile_length(m, k, P):
    """plan[8] .. plan[10] describe a sampler whose tiles are tile_len long, as the general kernels' are there."""
    try:
        plan = B.gtopk_debug_plan(m, k, P)
    except OSError as e:          # library not built
        pytest.skip(str(e))
    assert plan["small_path"] == 1 and plan["tile_len"] == 64
    covered = (plan["small_n_tiles"] - 1) * plan["small_tile_stride"] + plan["tile_len"]
    assert m - plan["small_tile_stride"] < covered                    # tiles up to the row's end
    assert plan["small_n_tiles"] * plan["tile_len"] >= 8_192


def _edges(sampled, lo_rank, hi_rank):
    """A bracket's ends as the kernels take them: the lower edge of the histogram bucket (2^17 keys wide) that lo_rank of the
    sampled keys reach (0 if the sample is smaller), the lowest edge that at most hi_rank do."""
    desc = np.sort(sampled)[::-1]
    lo = int(desc[lo_rank - 1]) >> 17 << 17 if lo_rank <= desc.size else 0
    return lo, ((int(desc[hi_rank]) >> 17) + 1) << 17


@pytest.mark.parametrize("nseg", [1, 8, 54, 400])
@pytest.mark.parametrize("m,k,P", [
    (1_048_579, 209_720, 32),                 # the shortest rows, the smallest density for them
    (1_500_003, 500_000, 16),                 # the largest
    (4_200_001, 525_001, 2),
])
def test_brackets_of_index_groups_hold_the_kth_key(m, k, P, nseg):
    """Steps of large densities: the k-th key of a row, and of the union of two sets, lies between both ends of its bracket,
    and the keys inside fit a row's storage.  Rows by the sampler's plan; the union by as many random elements of every
    group of 8192 as the kernels take scattered ones."""
    try:
        plan, routes = B.gtopk_debug_plan(m, k, P), B.gtopk_debug_routes(m, k, P)
    except OSError as e:          # library not built
        pytest.skip(str(e))
    groups = -(-m // 8192)
    assert routes["index_groups"] == groups
    t = np.arange(plan["n_tiles"], dtype=np.int64)[:, None] * plan["tile_stride"]
    pos = (t + np.arange(plan["tile_len"], dtype=np.int64)[None, :]).ravel()
    pos = pos[pos < m]
    for trial in range(3):
        rng = np.random.default_rng(1000 * nseg + trial)
        first = _row(rng, m, nseg)
        rows = first, first * rng.uniform(0.5, 1.5, m).astype(np.float32) * np.where(rng.random(m) < 0.5, -1, 1).astype(np.float32)
        union = np.zeros(m, np.float32)
        held = np.zeros(m, bool)
        for row in rows:
            key = np.abs(row).view(np.uint32)
            kth = int(np.partition(key, m - k)[m - k])
            lo, hi = _edges(key[pos], plan["target"], routes["row_target_hi"])
            assert lo <= kth < hi, (trial, lo, kth, hi)
            inside = int(((key >= lo) & (key < hi)).sum())
            assert inside + 4 * groups <= plan["capacity"] and inside < 0.6 * k, (trial, inside)
            union += np.where(key >= kth, row, np.float32(0.0))
            held |= key >= kth
        key = np.abs(union).view(np.uint32)
        kth = int(np.sort(key[held])[held.sum() - k])
        at = (np.arange(groups)[:, None] * 8192 + rng.integers(0, 8192, (groups, routes["union_samples"]))).ravel()
        at = at[at < m]
        lo, hi = _edges(key[at[held[at]]], routes["union_target_lo"], routes["union_target_hi"])
        assert lo <= kth < hi, (trial, lo, kth, hi)
