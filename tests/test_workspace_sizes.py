"""Host-side check (no GPU): the workspace of given k and P does not shrink as the rows get
longer, so that gtopk_tree, which is sized as for m = k, fits the workspace of any m >= k."""
import random

import pytest

from paper_1901_04359_amd import binding as B


@pytest.mark.parametrize("P", [1, 4, 32, 512])
def test_workspace_grows_with_m(P):
    try:
        B.load()
    except (OSError, RuntimeError) as e:          # library not built
        pytest.skip(str(e))
    rng = random.Random(P)
    for _ in range(60):
        k = int(2 ** rng.uniform(0, 22))
        sizes = sorted({int(k * 2 ** rng.uniform(0, 14)) + d for d in (0, 1) for _ in range(20)} | {k, k + 1})
        need = [B.gtopk_workspace_bytes(m, k, P) for m in sizes if k <= m <= 2 ** 31]
        assert all(n >= need[0] for n in need), (k, P, need)
