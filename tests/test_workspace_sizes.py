"""Host-side check (no GPU): a workspace serves smaller k, and the tree, of the same P too.  Programs allocate
once for the largest k they will meet (a density that comes down during the first epochs) and run
gtopk_tree, which is sized as for m = k, on the workspace of their step."""
import random

import pytest

from paper_1901_04359_amd import binding as B


@pytest.fixture(autouse=True)
def _library():
    try:
        B.load()
    except (OSError, RuntimeError) as e:          # library not built
        pytest.skip(str(e))


@pytest.mark.parametrize("P", [1, 4, 8, 32, 512])
def test_workspace_of_any_rows_serves_the_tree(P):
    rng = random.Random(P)
    for _ in range(60):
        k = int(2 ** rng.uniform(0, 22))
        sizes = sorted({int(k * 2 ** rng.uniform(0, 14)) + d for d in (0, 1) for _ in range(20)} | {k, k + 1})
        need = [B.gtopk_workspace_bytes(m, k, P) for m in sizes if k <= m <= 2 ** 31]
        assert all(n >= need[0] for n in need), (k, P, need)


@pytest.mark.parametrize("P", [1, 4, 8, 32, 512])
def test_workspace_grows_with_k(P):
    """k' <= 0.98 k: closer than that the group tables, whose slots per group go up in steps, may make a
    difference of some KB either way."""
    rng = random.Random(P)
    for _ in range(400):
        m = int(2 ** rng.uniform(4, 26))
        k = max(2, int(m * 2 ** rng.uniform(-12, 0)))
        less = max(1, min(int(k * rng.uniform(0.02, 0.98)), k - 1))
        assert B.gtopk_workspace_bytes(m, less, P) <= B.gtopk_workspace_bytes(m, k, P), (m, k, less, P)


@pytest.mark.parametrize("m,k,less,P", [
    (3_000_017, 5_860, 5_859, 8),              # one-block sampler / a kernel of its own for the sample
    (3_000_017, 4_097, 4_096, 8),
    (4_729, 3, 1, 1024),
    (8_191, 513, 512, 32),                     # general kernels / few-launch path
    (25_557_032, 6_389_258, 25_557, 32),
    (25_557_032, 1_277_852, 1_277_851, 32),    # chunks of 2^14 / 2^15 elements
])
def test_workspace_of_neighbouring_plans(m, k, less, P):
    assert B.gtopk_workspace_bytes(m, less, P) <= B.gtopk_workspace_bytes(m, k, P)
