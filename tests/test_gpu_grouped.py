"""gtopk_step at large densities (index groups, two-sided brackets), GPU against the oracle, bit for bit: sizes around
the edges of groups and stretches, rows that start at any offset in a 16-byte vector, value kinds that make brackets
long, empty or useless, and inputs that mislead the samplers, so that sets are selected outside their brackets."""
import numpy as np
import pytest

from tests.gpu_harness import Device, bits_equal, first_diff, idx_np, say, val_np
from tests.test_gpu_fullsize import oracle_step_parallel

pytestmark = pytest.mark.gpu

GROUP = 8192


def sampled_positions(m, k, P):
    """Elements that the rows' sampler reads, by the layout that gtopk_debug_plan reports."""
    from paper_1901_04359_amd import binding as B
    plan = B.gtopk_debug_plan(m, k, P)
    first = np.arange(plan["n_tiles"], dtype=np.int64) * plan["tile_stride"]
    at = (first[:, None] + np.arange(plan["tile_len"], dtype=np.int64)).ravel()
    return at[at < m]


def rows(kind, P, m, k, rng):
    layers = np.exp(rng.uniform(np.log(1e-5), np.log(1e-2), 24)).astype(np.float32)
    scale = np.repeat(layers, -(-m // 24))[:m]
    g = rng.standard_normal((P, m), dtype=np.float32) * scale
    if kind == "layers":
        return g
    if kind == "flat":
        return rng.standard_normal((P, m), dtype=np.float32)
    if kind == "zeros":                     # fewer non-zeros than k; zeros of either sign
        keep = rng.random((P, m)) < 0.5 * k / m
        return np.where(keep, g, np.where(rng.random((P, m)) < 0.5, np.float32(-0.0), np.float32(0.0))).astype(np.float32)
    if kind == "some_zero_rows":
        g[::2] = 0.0
        return g
    if kind == "signs":
        return np.sign(g).astype(np.float32) + (g == 0)
    if kind == "rounded":
        return np.rint(rng.standard_normal((P, m)) * 2).astype(np.float32)
    if kind == "denormal":
        return (rng.integers(-5000, 5000, (P, m)).astype(np.int32).astype(np.float64) * 1.4e-45).astype(np.float32)
    if kind == "cancel":                    # each pair's sums cancel
        g[1::2] = -g[0::2]
        return g
    if kind == "same":
        return np.broadcast_to(g[:1], g.shape).copy()
    if kind == "plateau":                   # masses at one magnitude around the k-th key
        mag = np.sort(np.abs(g[0]))[-k]
        g[rng.random((P, m)) < 0.3] = mag
        return g
    if kind == "apart":                     # the workers' large entries lie in different parts of the row
        for w in range(P):
            lo = m * w // P
            g[w, lo:lo + m // P] *= 1e4
        return g
    if kind == "infinite":                  # fewer than k of a row, more of a pair's union
        return np.where(rng.random((P, m)) < 0.6 * k / m, np.float32(np.inf), g).astype(np.float32)
    if kind == "nan":
        return np.where(rng.random((P, m)) < 0.9, np.float32(np.nan), g).astype(np.float32)
    at = sampled_positions(m, k, P)
    if kind == "sample_large":              # fewer than k keys reach the threshold
        g[:, at] *= 1e4
    elif kind == "sample_small":            # far more than k keys are above the bracket
        g[:, at] *= 1e-4
    elif kind == "sample_cancels":          # pairs: the sampled sums are nothing
        g[1::2, at] = -g[0::2, at]
    elif kind == "sample_doubles":          # pairs: more than half of the sums are nothing, but none of the sampled
        off = rng.random(m) < 0.7
        off[at] = False
        g[1::2] = np.where(off, -g[0::2], g[1::2])
    elif kind == "sample_two_values":       # .. and the other keys around the k-th are too many for a list
        two = np.where(rng.random((P, m)) < 0.5, np.float32(1.0), np.float32(1.0625))
        g = np.where(rng.random((P, m)) < 0.95, two, g)
        g[:, at] *= 1e-4
    else:
        raise ValueError(kind)
    return g.astype(np.float32)


KINDS = ("zeros", "some_zero_rows", "signs", "rounded", "denormal", "cancel", "same", "plateau", "apart", "sample_large",
         "sample_small", "sample_cancels", "sample_doubles", "infinite", "nan")
CASES = [
    # P, m, k, kind, elements from the end of a row to the start of the next
    (32, 128 * GROUP, 209_716, "layers", 0),            # the shortest rows, the smallest k for them
    (16, 128 * GROUP, 314_573, "layers", 0),            # the fewest entries of all workers
    (16, 128 * GROUP + 1, 349_525, "flat", 0),          # the largest k
    (16, 129 * GROUP - 1, 330_001, "layers", 2),
    (32, 128 * GROUP + 255, 262_000, "layers", 258),
    (8, 256 * GROUP + 3, 530_001, "layers", 0),
    (2, 512 * GROUP + 1, 524_289, "layers", 0),         # one round; the smallest density
    (4, 520 * GROUP - 3, 532_480, "flat", 1),
] + [(16, 1_050_003, 316_000, kind, pad) for pad, kind in enumerate(KINDS)] + [
    (2, 4_200_001, 530_000, kind, 0) for kind in ("zeros", "sample_large", "sample_small", "sample_cancels")] + [
    (16, 1_050_003, 316_000, "sample_two_values", 1)]


# Kinds that make every worker's set miss its bracket / every pair's of the first round; none of the others' sets do
MISS_WORKERS = ("sample_large", "sample_small", "sample_two_values", "denormal", "nan")
MISS_PAIRS = ("sample_large", "sample_small", "sample_two_values", "sample_cancels", "sample_doubles", "signs", "plateau", "infinite",
              "nan")


def check_missed(kind, P, missed):
    first = missed[P:P + P // 2]
    assert all(missed[:P]) if kind in MISS_WORKERS else not any(missed[:P]), missed
    assert all(first) if kind in MISS_PAIRS else not any(missed[P:]), missed
    if kind == "plateau":                   # (pairs of later rounds too)
        assert any(missed[P + P // 2:]), missed


@pytest.mark.parametrize("P,m,k,kind,pad", CASES)
def test_step_by_index_groups(P, m, k, kind, pad):
    from paper_1901_04359_amd import binding as B
    assert B.gtopk_debug_routes(m, k, P)["index_groups"] == -(-m // GROUP)
    rng = np.random.default_rng(P * 7 + m + k)
    dev = Device(P, m, k, stride=m + pad if pad else None)
    res = (rng.standard_normal((P, m), dtype=np.float32) * np.float32(1e-6) if kind == "layers"
           else np.zeros((P, m), dtype=np.float32))
    dev.set_res(res)
    for it in range(2 if kind in ("layers", "zeros") else 1):
        g = rows(kind, P, m, k, rng)
        dev.set_grad(g)
        say(f"index groups P={P} m={m} k={k} kind={kind} pad={pad} it={it}")
        gi, gv = dev.step()
        missed = dev.B.gtopk_debug_missed_brackets(dev.ws, m, k, P)
        say(f"  missed brackets: workers {sum(missed[:P])} of {P}, pairs {sum(missed[P:])} of {P - 1}")
        check_missed(kind, P, missed)
        exp = dict(zip(("loc_idx", "loc_val", "g_idx", "g_val", "residual"), oracle_step_parallel(res, g, k)))
        li, lv = idx_np(dev.loc_idx), val_np(dev.loc_val)
        for w in range(P):
            assert np.array_equal(li[w], exp["loc_idx"][w]), (w, first_diff(li[w], exp["loc_idx"][w]))
            assert bits_equal(lv[w], exp["loc_val"][w]), (w, first_diff(lv[w], exp["loc_val"][w]))
        assert np.array_equal(gi, exp["g_idx"]), first_diff(gi, exp["g_idx"])
        assert bits_equal(gv, exp["g_val"]), first_diff(gv, exp["g_val"])
        out = dev.residual()
        for w in range(P):
            assert bits_equal(out[w], exp["residual"][w]), (w, first_diff(out[w], exp["residual"][w]))
        res = np.stack(list(exp["residual"]))


# The longest rows that go by groups: the last group's ties are found at the end of the groups' table.
# ties: of either worker, equal to the k-th key, in front of the last group / in it (six of them are selected)
@pytest.mark.parametrize("m,ties", [(8192 * GROUP, ((3, 9), (6, 5))), (8191 * GROUP + 40, ((0, 9), (2, 7)))])
def test_ties_in_the_last_of_the_most_groups(m, ties):
    P, k, need = 2, m // 8 + 1, 6
    last = 8191 * GROUP
    rng = np.random.default_rng(m)
    large = rng.choice(last, k - need + 100, replace=False)      # (the first k - need, the others are free for ties)
    base = rng.random(m, dtype=np.float32) * np.float32(0.3) + np.float32(0.1)
    base[large[:k - need]] = rng.random(k - need, dtype=np.float32) * np.float32(2.0) + np.float32(2.0)
    # the workers share their large entries, so that the k-th key of the pair is that of their ties too
    g = np.stack([base, base])
    behind = rng.permutation(np.arange(last, m))
    for w, (before, inside) in enumerate(ties):
        g[w, large[k - need + 50 * w:][:before]] = 1.0
        g[w, behind[20 * w:][:inside]] = -1.0
    dev = Device(P, m, k)
    dev.set_grad(g)
    say(f"index groups, ties in the last group P={P} m={m} k={k}")
    assert dev.B.gtopk_debug_routes(m, k, P)["index_groups"] == 8192
    gi, gv = dev.step()
    assert not any(dev.B.gtopk_debug_missed_brackets(dev.ws, m, k, P))
    exp = dict(zip(("loc_idx", "loc_val", "g_idx", "g_val", "residual"), oracle_step_parallel(np.zeros_like(g), g, k)))
    li, lv = idx_np(dev.loc_idx), val_np(dev.loc_val)
    for w in range(P):
        assert np.array_equal(li[w], exp["loc_idx"][w]), (w, first_diff(li[w], exp["loc_idx"][w]))
        assert bits_equal(lv[w], exp["loc_val"][w]), (w, first_diff(lv[w], exp["loc_val"][w]))
    assert np.array_equal(gi, exp["g_idx"]), first_diff(gi, exp["g_idx"])
    assert bits_equal(gv, exp["g_val"]), first_diff(gv, exp["g_val"])
    out = dev.residual()
    for w in range(P):
        assert bits_equal(out[w], exp["residual"][w]), (w, first_diff(out[w], exp["residual"][w]))
