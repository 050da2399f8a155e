"""The tree in one block (few-launch path), GPU against the oracle, bit for bit: a wave per pair and every number
of threads per pair, more pairs than waves, the largest sets, and value kinds whose sums cancel or whose keys crowd into one bin."""
import numpy as np
import pytest

from oracle import gtopk_oracle as orc
from tests.gpu_harness import Device, bits_equal, first_diff, idx_np, say, val_np
from tests.test_gpu_grouped import rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["layers", "cancel", "same", "rounded", "signs", "zeros", "plateau", "apart", "denormal",
                                  "infinite", "nan"])
@pytest.mark.parametrize("P,k", [(2, 1), (2, 512), (4, 33), (4, 512), (8, 270), (8, 512), (16, 256), (32, 128), (64, 64), (64, 3),
                                 # both sides of the lengths at which a wave of the short sets' rounds holds more, and of the longest
                                 (16, 32), (64, 33), (2, 64), (8, 65), (2, 127), (16, 128), (16, 129), (2, 129)])
def test_tree_of_small_sets(P, k, kind):
    from paper_1901_04359_amd import binding as B
    m = 20_011
    assert B.gtopk_debug_plan(m, k, P)["small_path"] == 1
    rng = np.random.default_rng(P * 1000 + k)
    if kind in ("infinite", "nan"):         # most of every set, at indices of its own: a pair's union holds more than k of them
        g = rows("layers", P, m, k, rng)
        n = (3 * k + 3) // 4
        at = rng.permutation(m)[:P * n].reshape(P, n)
        for w in range(P):
            g[w, at[w]] = np.inf if kind == "infinite" else np.uint32(0x7FFFFFFF).view(np.float32)
    else:
        g = rows(kind, P, m, k, rng)
    if kind == "cancel":                    # the second half of the workers undoes the first in the last round
        g[P // 2:] = -g[:P // 2]
    dev = Device(P, m, k)
    dev.set_grad(g)
    say(f"tree of small sets P={P} k={k} kind={kind}")
    gi, gv = dev.step()
    exp = orc.step(np.zeros((P, m), np.float32), g, k)
    assert np.array_equal(idx_np(dev.loc_idx), exp["loc_idx"]) and bits_equal(val_np(dev.loc_val), exp["loc_val"])
    assert np.array_equal(gi, exp["g_idx"]), first_diff(gi, exp["g_idx"])
    assert bits_equal(gv, exp["g_val"]), first_diff(gv, exp["g_val"])
    out = dev.residual()
    assert bits_equal(out, exp["residual"]), first_diff(out, exp["residual"])
