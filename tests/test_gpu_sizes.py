"""Parity at the sizes where the library changes kernels, against the CPU oracle, bit for bit."""
import numpy as np
import pytest

from oracle import gtopk_oracle as orc
from paper_1901_04359_amd import workloads as W
from tests.gpu_harness import Device, bits_equal, first_diff, say
from tests.test_gpu_parity import _check_two_iterations, check_select, run_merge

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["gauss", "ties", "cancel"])
@pytest.mark.parametrize("k,batch", [(16_383, 25), (16_384, 24), (24_577, 16), (24_575, 16)])
def test_merge_batches_at_the_unions_border(kind, k, batch):
    """Either side of the batch sizes at which a merge's union is cut by output position."""
    m = 200_003
    idx, val = W.ksets(2 * batch, k, m, seed=k + batch, overlap=0.4, value_kind=kind)
    say(f"merge batches: kind={kind} k={k} batch={batch}")
    gi, gv = run_merge(idx[0::2].copy(), val[0::2].copy(), idx[1::2].copy(), val[1::2].copy(), k)
    for b in range(batch):
        oi, ov = orc.merge(idx[2 * b], val[2 * b], idx[2 * b + 1], val[2 * b + 1], k)
        assert np.array_equal(gi[b], oi), f"b={b} idx: {first_diff(gi[b], oi)}"
        assert bits_equal(gv[b], ov), f"b={b} val: {first_diff(gv[b], ov)}"


@pytest.mark.parametrize("kind", ["gauss", "ties"])
@pytest.mark.parametrize("P,m,k,pad,tile,chunk_log2,in_place", [
    # few blocks: chunks down to 4096 elements
    (2, 33_001, 900, 1, 16, 12, 0),      # (one block selects)
    (2, 33_001, 9000, 1, 16, 12, 1),
    (4, 900_001, 4000, 0, 16, 12, 0),    # runs put into index order
    (4, 1_500_003, 300_000, 3, 16, 12, 1),
    (8, 1_100_003, 5000, 2, 16, 13, 0),
    (16, 1_048_581, 5000, 0, 16, 14, 0),
    (2, 3_000_001, 4500, 5, 64, 12, 0),  # the large sample
    # blocks enough: chunks by the density
    (32, 2_200_003, 120_000, 1, 64, 13, 1),
    (32, 2_200_003, 12_000, 0, 64, 15, 0),
    (32, 3_000_017, 20_000, 3, 64, 14, 1),
])
def test_step_at_every_chunk_size(P, m, k, pad, tile, chunk_log2, in_place, kind):
    """Each size of the pass's chunks by either rule, with runs selected in place and put into index order, after
    the one-block sampler (tiles of 16) and the large one, on rows of ragged length and alignment."""
    from paper_1901_04359_amd import binding as B
    plan = B.gtopk_debug_plan(m, k, P)
    assert plan["tile_len"] == tile and plan["small_path"] == 0
    assert plan["chunk_log2"] == chunk_log2 and plan["run_groups"] == in_place
    _check_two_iterations(P, m, k, kind, pad, "chunk sizes")


@pytest.mark.parametrize("kind", ["gauss", "sparse", "ties", "zeros", "special", "hidden"])
@pytest.mark.parametrize("m,k", [
    ((1 << 19) - 1, 700),                # read as it stands
    (1 << 19, 700),                      # filtered
    ((1 << 20) + 1, 300_000),            # the select finished once per set
    (1_500_003, 1_500_003),              # everything selected
    (3_000_001, 1000),                   # the large sample
    (3_000_001, 4500),                   # chunks whose runs the pass histograms
    (3_000_001, 200_000),
])
def test_dense_topk_filtered(m, k, kind):
    """Rows that are filtered before the selection, and rows whose filter has nothing to go by (fewer
    than k non-zeros, masses of ties, the largest entries where the sample does not look)."""
    import torch
    from paper_1901_04359_amd import binding as B
    rng = np.random.default_rng(m + k)
    d = rng.standard_normal(m).astype(np.float32)
    if kind == "sparse":
        d[rng.random(m) < 0.9] = 0.0
    elif kind == "ties":
        d = np.round(d).astype(np.float32)
    elif kind == "zeros":                # -0.0 among them
        d *= np.float32(0.0)
        at = rng.choice(m, max(1, k // 2), replace=False)
        d[at] = rng.standard_normal(at.size).astype(np.float32)
    elif kind == "special":
        for j, x in enumerate([np.inf, -np.inf, 1e-45, -1e-45, -0.0, 3.4e38, np.nan]):
            d[rng.integers(0, m, 5)] = np.float32(x)
    elif kind == "hidden":               # large entries everywhere but in the sampled tiles, then the reverse
        plan = B.gtopk_debug_plan(m, k, 1)
        at = np.arange(m) % plan["tile_stride"] < plan["tile_len"]
        d = np.where(at if k % 8 else ~at, d * np.float32(100.0), d).astype(np.float32)
    say(f"dense top-k: m={m} k={k} kind={kind}")
    row = torch.from_numpy(d).cuda()
    gi = torch.zeros(k, dtype=torch.int32, device="cuda")
    gv = torch.zeros(k, device="cuda")
    B.gtopk_dense_topk(row, k, gi, gv, B.alloc_workspace(m, k, 1))
    oi, ov = orc.dense_topk(d, k)
    gi, gv = gi.cpu().numpy().view(np.uint32), gv.cpu().numpy()
    assert np.array_equal(gi, oi), first_diff(gi, oi)
    assert bits_equal(gv, ov), first_diff(gv, ov)
    assert bits_equal(row.cpu().numpy(), d), "the row was written to"


@pytest.mark.parametrize("k", [1, 1023, 16_384, 16_385])
@pytest.mark.parametrize("batch", [1, 3])
def test_merge_smallest_keys(k, batch):
    """Either side of the set size up to which one block finds a set's smallest key; the smallest
    key lies at either end of the set, or is 0."""
    m = 40_000
    idx, val = W.ksets(2 * batch, k, m, seed=k, overlap=0.5, value_kind="gauss")
    val[0, 0] = val[1, -1] = np.float32(1e-6)
    val[-1, -1] = np.float32(-0.0)
    say(f"merge smallest keys: k={k} batch={batch}")
    gi, gv = run_merge(idx[0::2].copy(), val[0::2].copy(), idx[1::2].copy(), val[1::2].copy(), k)
    for b in range(batch):
        oi, ov = orc.merge(idx[2 * b], val[2 * b], idx[2 * b + 1], val[2 * b + 1], k)
        assert np.array_equal(gi[b], oi), f"b={b} idx: {first_diff(gi[b], oi)}"
        assert bits_equal(gv[b], ov), f"b={b} val: {first_diff(gv[b], ov)}"


@pytest.mark.parametrize("m", [2047, 2048, 2049, 8191, 8193, 30_001])
@pytest.mark.parametrize("P", [1, 31, 32])
def test_dense_average_of_crowded_blocks(m, P):
    """Up to 32 workers whose entries fill whole blocks of the dense average and their borders."""
    import torch
    from paper_1901_04359_amd import binding as B
    k = max(1, m // 2)
    rng = np.random.default_rng(m + P)
    idx = np.stack([np.sort(rng.choice(m, k, replace=False)) for _ in range(P)]).astype(np.uint32)
    idx[0] = np.arange(m - k, m)         # a run up to the row's end, across every border before it
    idx[P - 1] = np.arange(k)
    val = rng.standard_normal((P, k)).astype(np.float32)
    say(f"dense average: m={m} P={P}")
    dense = torch.full((m,), 7.0, device="cuda")
    B.gtopk_topk_allreduce(torch.from_numpy(idx.view(np.int32)).cuda(), torch.from_numpy(val).cuda(), P, k, dense,
                           B.alloc_allreduce_workspace(m, P))
    exp = np.zeros(m, dtype=np.float32)
    for w in range(P):                   # rank order, one fp32 add each
        exp[idx[w]] += val[w]
    exp /= np.float32(P)
    got = dense.cpu().numpy()
    assert bits_equal(got, exp), first_diff(got, exp)


@pytest.mark.parametrize("kind", ["gauss", "ties"])
@pytest.mark.parametrize("P,m,k", [
    (4, 8_192, 3), (4, 8_193, 3),        # sizes of the few-launch path, in the general kernels
    (2, 8_192, 8_192),
    (1, 1, 1), (8, 63, 2),
    (128, 8_192, 3), (128, 8_195, 3),
])
def test_rows_no_longer_than_the_sample(P, m, k, kind):
    """Either side of the row length up to which the whole row is the one-block sampler's sample."""
    from paper_1901_04359_amd import binding as B
    assert B.gtopk_debug_plan(m, k, P)["tile_len"] == (16 if m <= 8_192 else 64)
    rng = np.random.default_rng(P + m + k)
    dev = Device(P, m, k)
    res = rng.standard_normal((P, m)).astype(np.float32)
    g = rng.standard_normal((P, m)).astype(np.float32)
    if kind == "ties":
        res, g = np.round(res), np.round(g)
    check_select(dev, res, g, f"short rows P={P} m={m} k={k} kind={kind}")
    dev.set_res(res)
    dev.set_grad(g)
    for _ in range(3):                   # the thresholds are carried over from the second call on
        gi, gv = dev.step_carry()
        exp = orc.step(res, g, k)
        assert np.array_equal(gi, exp["g_idx"]) and bits_equal(gv, exp["g_val"])
        assert bits_equal(dev.residual(), exp["residual"])
        res = exp["residual"]


def _us(call, reps=5):
    import torch
    call(), call()
    best = float("inf")
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


@pytest.mark.parametrize("P,m,k", [(8, 1_000_003, 125_000), (2, 4_000_003, 240_000)])
def test_rows_of_few_magnitudes_are_not_read_per_block(P, m, k):
    """Values rounded to integers: the bin of the k-th key holds more than 100,000 equal keys.  Reading
    that list in every block of the emit takes over thirty times as long as a row of distinct values; the
    bound leaves the few times as long that writing the list and reading it once would take."""
    dev = Device(P, m, k)
    rng = np.random.default_rng(m)
    res = rng.standard_normal((P, m)).astype(np.float32)
    zero = np.zeros((P, m), dtype=np.float32)
    us = {}
    for kind, rows in (("distinct", res), ("rounded", np.round(2 * res))):
        check_select(dev, rows, zero, f"few magnitudes P={P} m={m} k={k} kind={kind}")
        # the selected entries are cleared by every call: the rows are put back in between
        rows_d = dev.torch.from_numpy(rows).cuda()

        def call():
            dev.res.copy_(rows_d)
            dev.B.gtopk_local_select(dev.grad, dev.res, k, dev.loc_idx, dev.loc_val, dev.ws)

        us[kind] = _us(call)
    say(f"us per call: {us}")
    assert us["rounded"] < 5 * us["distinct"], us


@pytest.mark.parametrize("kind", ["one key", "two keys", "none above"])
@pytest.mark.parametrize("P,m,k", [
    (2, 3_000_001, 10_000),              # candidates put into index order
    (2, 3_000_001, 100_000),             # runs selected in place
    (1, 700_001, 20_000),
])
def test_long_lists_of_equal_keys(P, m, k, kind):
    """Either side of the list length (4096) from which equal in-bin keys are counted and not listed; a
    second key in the bin (the next float) sends the finish back to the list."""
    for n_eq in (4095, 4096, 4097, 9000):
        rng = np.random.default_rng(m + n_eq)
        rows = (1e-3 * rng.standard_normal((P, m))).astype(np.float32)
        for w in range(P):
            at = rng.permutation(m)
            n_top = 0 if kind == "none above" else k - n_eq // 2
            rows[w, at[:n_top]] = (2.0 + rng.random(n_top)).astype(np.float32)
            plateau = at[n_top:n_top + (n_eq if n_top else k + n_eq)]
            rows[w, plateau] = np.where(rng.random(plateau.size) < 0.5, np.float32(1.0), np.float32(-1.0))
            if kind == "two keys":
                rows[w, plateau[::3]] = np.nextafter(np.float32(1.0), np.float32(2.0))
        check_select(Device(P, m, k), rows, np.zeros_like(rows), f"equal keys P={P} m={m} k={k} {kind} n_eq={n_eq}")


def test_one_dense_row_among_many_lists():
    """A worker whose row is all zeros is selected from its dense row, 25 million elements, which 32 blocks take as
    long to histogram as all the lists of the other workers: a fifth of the call.  With its own number of blocks
    it is less than half of that."""
    import torch
    P, m, k = 32, 25_557_032, 1_852_885
    dev = Device(P, m, k)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    rows = torch.empty((P, m), device="cuda")
    us = {}
    for kind in ("ordinary", "one of zeros"):
        rows.normal_(generator=gen)
        if kind != "ordinary":
            rows[5].zero_()
        say(f"dense row among lists P={P} m={m} k={k} kind={kind}")
        us[kind] = float("inf")
        for _ in range(7):
            dev.res.copy_(rows)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            dev.B.gtopk_local_select(dev.grad, dev.res, k, dev.loc_idx, dev.loc_val, dev.ws)
            b.record()
            b.synchronize()
            us[kind] = min(us[kind], a.elapsed_time(b) * 1e3)
    assert torch.equal(dev.loc_idx[5], torch.arange(k, dtype=torch.int32, device="cuda"))
    assert int(dev.loc_val[5].count_nonzero()) == 0
    top = rows[6].abs().topk(k).indices.sort().values.int()
    assert torch.equal(dev.loc_idx[6], top)              # (with this seed the border is no tie)
    say(f"us per call: {us}")
    assert us["one of zeros"] < 1.12 * us["ordinary"], us          # 1.06; with the lists' blocks 1.18


@pytest.mark.parametrize("kind", ["zeros", "few", "just k", "one magnitude", "powers of two", "most of one"])
@pytest.mark.parametrize("m,k", [
    (1 << 19, 700),                      # one-block sampler, the pass histograms
    (700_001, 5000),                     # one-block sampler, it does not
    (3_000_001, 1000),                   # the large sample
    (3_000_001, 30_000),
])
def test_dense_topk_of_rows_that_cannot_be_filtered(m, k, kind):
    """Rows whose sample shows fewer than k non-zeros, or more entries at one magnitude than the candidate list
    holds: the pass filters nothing (no candidate is counted) and histograms the row instead."""
    import torch
    from paper_1901_04359_amd import binding as B
    rng = np.random.default_rng(m + k)
    d = np.zeros(m, dtype=np.float32)
    if kind == "few":
        at = rng.choice(m, k // 2, replace=False)
        d[at] = rng.standard_normal(at.size)
    elif kind == "just k":
        at = rng.choice(m, k, replace=False)
        d[at] = rng.standard_normal(at.size)
    elif kind == "one magnitude":
        d = np.where(rng.random(m) < 0.5, np.float32(0.25), np.float32(-0.25)).astype(np.float32)
    elif kind == "powers of two":
        x = rng.standard_normal(m)
        d = (np.sign(x) * np.exp2(np.minimum(np.floor(np.log2(np.abs(x) + 1e-9)), 0.0))).astype(np.float32)
    elif kind == "most of one":
        d = (1e-3 * rng.standard_normal(m)).astype(np.float32)
        d[rng.random(m) < 0.6] = np.float32(3.0)
        d[rng.choice(m, k // 3, replace=False)] = np.float32(5.0)
    d[::7] *= np.float32(-1.0)           # -0.0 among the zeros
    say(f"dense top-k that cannot be filtered: m={m} k={k} kind={kind}")
    row = torch.from_numpy(d).cuda()
    gi = torch.zeros(k, dtype=torch.int32, device="cuda")
    gv = torch.zeros(k, device="cuda")
    ws = B.alloc_workspace(m, k, 1)
    ws.fill_(0xA5)
    B.gtopk_dense_topk(row, k, gi, gv, ws)
    torch.cuda.synchronize()
    counts, _ = B.gtopk_debug_candidate_counts(ws, m, k, 1)
    assert counts == [0], (counts, kind)
    oi, ov = orc.dense_topk(d, k)
    gi, gv = gi.cpu().numpy().view(np.uint32), gv.cpu().numpy()
    assert np.array_equal(gi, oi), first_diff(gi, oi)
    assert bits_equal(gv, ov), first_diff(gv, ov)
    assert bits_equal(row.cpu().numpy(), d), "the row was written to"
