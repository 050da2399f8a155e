"""The Top-k operation on sets that one block merges (k <= 8192), GPU against the oracle, bit for bit: both sides of
every size at which a thread gets more slots, and of the largest; shared indices from none to all; plus trees of such
sets, whose last round divides, and whose rounds hand their smallest keys on."""
import numpy as np
import pytest

from oracle import gtopk_oracle as orc
from paper_1901_04359_amd import workloads as W
from tests.gpu_harness import bits_equal, first_diff, idx_np, say, to_dev, val_np

pytestmark = pytest.mark.gpu


def _sets(n, k, kind, overlap, seed):
    rng = np.random.default_rng(seed)
    if kind in ("gauss", "ties", "cancel"):
        return W.ksets(n, k, 4 * k + 3, seed=seed, overlap=overlap, value_kind=kind)
    idx, val = W.ksets(n, k, 4 * k + 3, seed=seed, overlap=overlap, value_kind="gauss")
    if kind == "zeros":
        val = np.where(rng.random(val.shape) < 0.7, np.where(rng.random(val.shape) < 0.5, 0.0, -0.0), val).astype(np.float32)
    elif kind == "equal":
        val = np.copysign(np.float32(0.25), val)
    elif kind == "wide":                        # keys over the whole range of the type, denormals and huge ones
        val = (val * np.exp2(rng.integers(-148, 120, val.shape))).astype(np.float32)
    elif kind in ("infinite", "nan"):           # fewer than k of a set, more of a pair's union
        val = np.where(rng.random(val.shape) < 0.7, np.float32(np.inf if kind == "infinite" else np.nan), val)
    return idx, val


@pytest.mark.parametrize("kind,overlap", [("gauss", 0.0), ("gauss", 0.5), ("ties", 0.4), ("cancel", 1.0), ("zeros", 0.3),
                                          ("equal", 0.5), ("wide", 0.2), ("infinite", 0.1), ("nan", 0.1)])
@pytest.mark.parametrize("k", [1, 3, 511, 512, 1023, 1024, 1025, 2048, 2049, 4095, 4096, 4097, 6001, 8191, 8192, 8193])
def test_merge_in_one_block(k, kind, overlap):
    import torch
    from paper_1901_04359_amd import binding as B
    assert B.gtopk_debug_routes(k, k, 2)["merge_block"] == (1 if k <= 8192 else 0)
    batch, pad = 3, 5
    idx, val = _sets(2 * batch, k, kind, overlap, 100 * k + len(kind))
    stride = k + pad                            # rows apart, so that none but the first is aligned
    a_i, b_i = (np.zeros((batch, stride), np.uint32) for _ in range(2))
    a_v, b_v = (np.zeros((batch, stride), np.float32) for _ in range(2))
    a_i[:, :k], b_i[:, :k], a_v[:, :k], b_v[:, :k] = idx[0::2], idx[1::2], val[0::2], val[1::2]
    ws = B.alloc_merge_workspace(k, batch)
    ws.fill_(0x5A)
    out_i = torch.full((batch, stride), 77, dtype=torch.int32, device="cuda")
    out_v = torch.full((batch, stride), 77.0, device="cuda")
    say(f"merge in one block k={k} kind={kind} overlap={overlap}")
    B.gtopk_merge(to_dev(a_i), to_dev(a_v), to_dev(b_i), to_dev(b_v), k, batch, stride, out_i, out_v, stride, ws)
    torch.cuda.synchronize()
    gi, gv = idx_np(out_i), val_np(out_v)
    for p in range(batch):
        oi, ov = orc.merge(a_i[p, :k], a_v[p, :k], b_i[p, :k], b_v[p, :k], k)
        assert np.array_equal(gi[p, :k], oi), first_diff(gi[p, :k], oi)
        assert bits_equal(gv[p, :k], ov), first_diff(gv[p, :k], ov)
    assert (gi[:, k:] == 77).all() and (gv[:, k:] == 77.0).all()


@pytest.mark.parametrize("P,k,kind", [(2, 1024, "gauss"), (8, 8192, "ties"), (16, 1025, "cancel"), (32, 300, "wide"),
                                      (8, 4097, "zeros"), (64, 2049, "equal")])
def test_tree_of_sets_merged_in_one_block(P, k, kind):
    import torch
    from paper_1901_04359_amd import binding as B
    idx, val = _sets(P, k, kind, 0.5, P + k)
    ws = B.alloc_workspace(k, k, P)
    ws.fill_(0x5A)
    g_i = torch.zeros(k, dtype=torch.int32, device="cuda")
    g_v = torch.zeros(k, device="cuda")
    say(f"tree in one block per pair P={P} k={k} kind={kind}")
    B.gtopk_tree(to_dev(idx), to_dev(val), P, k, g_i, g_v, ws)
    torch.cuda.synchronize()
    sets = [(idx[p], val[p]) for p in range(P)]
    while len(sets) > 1:
        sets = [orc.merge(*sets[i], *sets[i + 1], k) for i in range(0, len(sets), 2)]
    assert np.array_equal(idx_np(g_i), sets[0][0])
    assert bits_equal(val_np(g_v), sets[0][1] / np.float32(P))
