"""The local selection of medium rows by one block per worker (rows that cannot be filtered: by up to eight), GPU
against the oracle, bit for bit, through gtopk_local_select, gtopk_step and gtopk_step_carry: both sides of every size at
which a thread holds more entries and of the largest, and rows whose list cannot be used or does not fit a block's registers."""
import numpy as np
import pytest

from oracle import gtopk_oracle as orc
from tests.gpu_harness import Device, bits_equal, first_diff, idx_np, say, val_np
from tests.test_gpu_grouped import rows

pytestmark = pytest.mark.gpu

# P, m, k, elements from the end of a row to the start of the next, entries that a thread holds (0: several kernels)
SIZES = [(8, 30_001, 960, 0, 4), (8, 30_001, 961, 1, 8), (4, 99_999, 1984, 0, 8), (4, 100_000, 1985, 3, 16), (2, 524_288, 4032, 0, 16),
         (2, 524_289, 4032, 0, 0), (2, 524_288, 4033, 2, 0), (16, 60_007, 600, 0, 4), (2, 4_097, 4_000, 1, 16), (8, 524_285, 4032, 2, 16),
         # a row is shared by several blocks: from 2^17 elements on, fewer than 8 workers, eight blocks to four
         (4, 131_072, 1000, 0, 8), (4, 131_073, 1000, 3, 8), (8, 131_073, 520, 0, 4), (1, 262_145, 1638, 0, 8), (2, 200_003, 1639, 1, 8),
         (4, 150_001, 2731, 0, 16), (2, 140_000, 20, 1, 4)]


@pytest.mark.parametrize("kind", ["layers", "flat", "rounded", "zeros", "plateau", "levels", "two_values", "sample_large",
                                  "sample_small", "infinite", "nan"])
@pytest.mark.parametrize("P,m,k,pad,entries", SIZES)
def test_local_select_in_one_block(P, m, k, pad, entries, kind):
    from paper_1901_04359_amd import binding as B
    assert B.gtopk_debug_routes(m, k, P)["select_entries"] == entries
    rng = np.random.default_rng(P * 31 + m + k)
    dev = Device(P, m, k, stride=m + pad if pad else None)
    res = (rng.standard_normal((P, m), dtype=np.float32) * np.float32(1e-5)).astype(np.float32)
    if kind == "levels":                    # runs of equal values, the largest behind the others: cut twice for the k-th key
        g = np.repeat(np.arange(1, m // 100 + 2), 100)[:m].clip(max=m // 400 + 1).astype(np.float32) * np.ones((P, 1), np.float32)
        g[1::2] *= -1
    elif kind == "two_values":              # mixed in every step, close together: more in the k-th key's bin than a list holds
        g = np.where(rng.random((P, m)) < 0.5, np.float32(1.0), np.float32(1.0 + 2.0 ** -20))
    else:
        g = rows(kind, P, m, k, rng)
    if kind != "layers":
        res[:] = 0.0
    exp = orc.step(res, g, k)
    acc = res + g
    for call in ("local_select", "step", "step_carry"):
        dev.set_grad(g)
        dev.set_res(res)
        dev.loc_idx.zero_()
        say(f"select in one block {call} P={P} m={m} k={k} kind={kind} pad={pad}")
        if call == "local_select":
            dev.local_select()
        else:
            gi, gv = getattr(dev, call)()
            assert np.array_equal(gi, exp["g_idx"]), first_diff(gi, exp["g_idx"])
            assert bits_equal(gv, exp["g_val"]), first_diff(gv, exp["g_val"])
        li, lv, out = idx_np(dev.loc_idx), val_np(dev.loc_val), dev.residual()
        assert np.array_equal(li, exp["loc_idx"]), first_diff(li, exp["loc_idx"])
        assert bits_equal(lv, exp["loc_val"]), first_diff(lv, exp["loc_val"])
        if call == "local_select":
            want = acc.copy()
            np.put_along_axis(want, exp["loc_idx"].astype(np.int64), np.float32(0.0), axis=1)
            assert bits_equal(out, want), first_diff(out, want)
        else:
            assert bits_equal(out, exp["residual"]), first_diff(out, exp["residual"])
