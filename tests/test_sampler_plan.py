"""Host-side check of the sampler's plan (no GPU): over random layer structures of the kind
the workloads are drawn from, the speculative threshold that the plan's sample would give
keeps at least k and at most `capacity` entries of the row - the condition under which a
worker is served from its candidate list and not from its dense row.

The plan (tile positions, target rank, list capacity) comes from the library through
gtopk_debug_plan; the estimate is modelled here with numpy: the threshold is the plan's
target-th largest magnitude among the sampled elements, rounded down to the edge of a
histogram bucket (the sampler's buckets are at most 1/64 of the magnitude wide).  A miss
would cost time only (the select is exact whatever it filters with), so this is a check of
the margin, not of correctness."""
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
