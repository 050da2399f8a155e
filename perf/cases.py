"""The calls that a program using this library makes, at the sizes it makes them, for timing
them and for comparing two builds of the library.

Five kinds of call ("call" of a case):
  step      one gTop-k S-SGD iteration by gtopk_step: the whole hot path in one call
  carry     the same by gtopk_step_carry, the thresholds carried from call to call
  parts     the same iteration put together by hand, with the model update behind it:
            gtopk_local_select, gtopk_tree, gtopk_residual_restore, gtopk_apply_update
  merge     the Top-k operation alone on `P` pairs of k-sets (gtopk_merge)
  naive     the paper's comparison aggregation of P workers' k-sets: the dense average of
            Algorithm 1 (gtopk_topk_allreduce), then Algorithm 2's top-k of it
            (gtopk_dense_topk)

Sizes are those of the repository's own workloads (its benchmark and its full-size tests):
m gradients per worker, P workers, k selected, and values with a layer-wise scale.  Every
result is a copy or one fp32 add or divide in a fixed order, so outputs agree to the bit.
"""
import math
import random

import torch

from paper_1901_04359_amd import binding as B

# A pass takes its gradients from a window into a longer vector, the next pass from the
# window kShift elements further on: every pass sees fresh gradients, as in training, and a
# residual that is carried over hundreds of passes stays the random walk that it is there.
WINDOWS = 512
SHIFT = 64

LR = 0.05


def _case(name, call, m, P, k, layers, lo, hi, kind="gauss"):
    return {"name": name, "call": call, "m": m, "P": P, "k": k, "layers": layers,
            "sigma_lo": lo, "sigma_hi": hi, "kind": kind}


def listed():
    return [
        # a toy model: latency and the number of launches
        _case("tiny", "step", 65_536, 4, 66, 1, 1e-3, 1e-3, "laplace"),
        # ResNet-20 on Cifar-10: the smallest real model of the paper
        _case("resnet20", "step", 269_722, 8, 270, 22, 1e-4, 1e-2),
        # an odd row length at a density of one half percent, thresholds carried along
        _case("odd_carry", "carry", 3_000_017, 8, 15_001, 12, 1e-4, 1e-2),
        # VGG-16, heavy tails
        _case("vgg16", "step", 14_728_266, 16, 14_728, 16, 1e-5, 1e-2, "heavy"),
        # VGG-16 in separate calls, for a program that does other work in between
        _case("vgg16_parts", "parts", 14_728_266, 16, 14_728, 16, 1e-5, 1e-2, "heavy"),
        # ResNet-50 on 32 workers: the benchmark's default, at both of its densities
        _case("resnet50", "step", 25_557_032, 32, 25_557, 54, 1e-5, 1e-2),
        _case("resnet50_1pc", "step", 25_557_032, 32, 255_570, 54, 1e-5, 1e-2),
        # the same in the warm-up epochs, when the density comes down from 25 %
        _case("warmup_7pc", "step", 25_557_032, 32, 1_852_885, 54, 1e-5, 1e-2),
        _case("warmup_25pc", "step", 25_557_032, 32, 6_389_258, 54, 1e-5, 1e-2),
        # AlexNet, with repeated magnitudes: the largest
        _case("alexnet", "step", 61_100_840, 32, 61_101, 8, 1e-4, 1e-2, "ties"),
        # one tree round on its own: sixteen pairs of sets of an odd size
        _case("merge16", "merge", 25_557_032, 16, 100_003, 54, 1e-5, 1e-2),
        # Algorithms 1 and 2 on 32 workers' sets
        _case("naive", "naive", 25_557_032, 32, 25_557, 54, 1e-5, 1e-2),
    ]


def draw(rng):
    call = rng.choice(["step"] * 6 + ["carry", "parts", "merge", "naive"])
    P = 2 ** rng.randint(1, 5)
    most = min(61_100_840, (3 << 28) // P)
    m = int(math.exp(rng.uniform(math.log(20_000), math.log(most))))
    k = max(1, int(m * math.exp(rng.uniform(math.log(5e-4), math.log(0.25)))))
    if call in ("merge", "naive"):       # sets of a running job: densities of two percent at most
        k = max(1, int(m * math.exp(rng.uniform(math.log(5e-4), math.log(0.02)))))
    lo = 10.0 ** rng.randint(-5, -3)
    c = _case("", call, m, P, k, rng.randint(1, 64), lo, rng.choice([lo, 1e-2]),
              rng.choice(["gauss", "gauss", "laplace", "heavy", "ties"]))
    del c["name"]
    return c


# ---- inputs -------------------------------------------------------------------------

def _scales(case):
    """Scale of every element of a row: the layers of the case's model (not of the seed)."""
    m, n = case["m"], min(case["layers"], case["m"])
    r = random.Random("%d %d" % (m, n))
    w = [math.exp(r.uniform(0.0, math.log(1000.0))) for _ in range(n)]
    if case["kind"] == "ties":           # few leading layers with large gradients, the rest behind
        w = [1.0] * (n - n // 3) + [24.0 * (n - n // 3) / max(1, n // 3)] * (n // 3)
    cum, ends = 0.0, []
    for x in w:
        cum += x
        ends.append(int(round(m * cum / sum(w))))
    ends[-1] = m
    lo, hi = math.log(case["sigma_lo"]), math.log(case["sigma_hi"])
    s = torch.empty(m, device="cuda")
    first = 0
    for i, e in enumerate(ends):
        if case["kind"] == "ties":
            v = hi if i < n - n // 3 else lo
        else:
            v = r.uniform(lo, hi)
        s[first:e] = math.exp(v)
        first = e
    return s


def _laplace(n, gen):
    u = torch.rand(n, device="cuda", generator=gen).sub_(0.5)
    return u.sign() * -torch.log1p(-(2 * u.abs()).clamp_(max=1 - 2.0 ** -24))


def _fill(out, scale, kind, gen):
    n = out.numel()
    if kind == "laplace":
        torch.mul(_laplace(n, gen), scale, out=out)
        return
    out.normal_(generator=gen)
    out.mul_(scale)
    if kind == "heavy":                  # one value in twenty from a tail ten times as wide
        heavy = torch.rand(n, device="cuda", generator=gen) < 0.05
        torch.where(heavy, _laplace(n, gen) * (10 * scale), out, out=out)
    elif kind == "ties":                 # one value in a thousand from eight magnitudes per binade
        q = torch.rand(n, device="cuda", generator=gen) < 0.001
        bits = out.view(torch.int32)
        torch.where(q, bits & -0x100000, bits, out=bits)


def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) & 0xFFFFFFFF) * 8 + stream)
    return g


def _rows(case, seed):
    """Gradient windows (flat) and the residual [P][m] of a run some ten iterations old."""
    m, P = case["m"], case["P"]
    scale = _scales(case)
    gen = _gen(seed, 1)
    grads = torch.empty(P * m + WINDOWS * SHIFT, device="cuda")
    for w in range(P):
        _fill(grads[w * m:(w + 1) * m], scale, case["kind"], gen)
    tail, first = grads[P * m:], 0
    while first < tail.numel():
        n = min(m, tail.numel() - first)
        _fill(tail[first:first + n], scale[:n], case["kind"], gen)
        first += n
    res = torch.empty((P, m), device="cuda")
    gen = _gen(seed, 2)
    for w in range(P):
        res[w].normal_(generator=gen)
        res[w].mul_(scale).mul_(3.0)
    return grads, res


def _sets(case, n, seed):
    """n k-sets as n workers select them from gradients of the case: at the indices of a
    worker's largest magnitudes, every worker's alike in the layers that they fall in."""
    m, k = case["m"], case["k"]
    scale = _scales(case)
    gen = _gen(seed, 3)
    idx = torch.empty((n, k), dtype=torch.int32, device="cuda")
    val = torch.empty((n, k), device="cuda")
    row = torch.empty(m, device="cuda")
    for s in range(n):
        _fill(row, scale, case["kind"], gen)
        i = torch.topk(row.abs(), k, sorted=False).indices.sort().values
        idx[s] = i.to(torch.int32)
        val[s] = row[i]
    return idx, val


def prepare(case, seed):
    m, P, k = case["m"], case["P"], case["k"]
    call = case["call"]
    s = {"case": case, "pass": 0}
    i32 = dict(dtype=torch.int32, device="cuda")
    if call in ("step", "carry", "parts"):
        s["grads"], s["res"] = _rows(case, seed)
        s["ws"] = B.alloc_workspace(m, k, P)
        s["loc_idx"] = torch.zeros((P, k), **i32)
        s["loc_val"] = torch.zeros((P, k), device="cuda")
        s["g_idx"] = torch.zeros(k, **i32)
        s["g_val"] = torch.zeros(k, device="cuda")
        if call == "carry":
            s["thr"] = torch.zeros((P, 4), **i32)
        if call == "parts":
            s["weights"] = torch.empty(m, device="cuda").normal_(generator=_gen(seed, 4)).mul_(0.05)
    elif call == "merge":
        idx, val = _sets(case, 2 * P, seed)         # pair p: sets p and P + p
        s["a_idx"], s["b_idx"] = idx[:P].clone(), idx[P:].clone()
        s["a_val"], s["b_val"] = val[:P].clone(), val[P:].clone()
        s["out_idx"] = torch.zeros((P, k), **i32)
        s["out_val"] = torch.zeros((P, k), device="cuda")
        s["ws"] = B.alloc_merge_workspace(k, P)
    else:
        s["idx"], s["val"] = _sets(case, P, seed)
        s["dense"] = torch.zeros(m, device="cuda")
        s["ws"] = B.alloc_allreduce_workspace(m, P)
        s["ws_top"] = B.alloc_workspace(m, k, 1)
        s["g_idx"] = torch.zeros(k, **i32)
        s["g_val"] = torch.zeros(k, device="cuda")
    return s


def run(s):
    c = s["case"]
    m, P, k, call = c["m"], c["P"], c["k"], c["call"]
    if call == "merge":
        B.gtopk_merge(s["a_idx"], s["a_val"], s["b_idx"], s["b_val"], k, P, k,
                      s["out_idx"], s["out_val"], k, s["ws"])
        return {"idx": s["out_idx"], "val": s["out_val"]}
    if call == "naive":
        B.gtopk_topk_allreduce(s["idx"], s["val"], P, k, s["dense"], s["ws"])
        B.gtopk_dense_topk(s["dense"], k, s["g_idx"], s["g_val"], s["ws_top"])
        return {"dense": s["dense"], "g_idx": s["g_idx"], "g_val": s["g_val"]}
    off = (s["pass"] % WINDOWS) * SHIFT
    s["pass"] += 1
    grad = s["grads"][off:off + P * m].view(P, m)
    out = {n: s[n] for n in ("loc_idx", "loc_val", "g_idx", "g_val")}
    out["residual"] = s["res"]
    if call == "step":
        B.gtopk_step(grad, s["res"], k, s["g_idx"], s["g_val"], s["loc_idx"], s["loc_val"], s["ws"])
    elif call == "carry":
        B.gtopk_step_carry(grad, s["res"], k, s["g_idx"], s["g_val"], s["loc_idx"], s["loc_val"],
                           s["thr"], s["ws"])
    else:
        B.gtopk_local_select(grad, s["res"], k, s["loc_idx"], s["loc_val"], s["ws"])
        B.gtopk_tree(s["loc_idx"], s["loc_val"], P, k, s["g_idx"], s["g_val"], s["ws"])
        B.gtopk_residual_restore(s["res"], k, s["loc_idx"], s["loc_val"], s["g_idx"])
        B.gtopk_apply_update(s["weights"], k, s["g_idx"], s["g_val"], LR)
        out["weights"] = s["weights"]
    return out


def work(case):
    m, P, k, call = case["m"], case["P"], case["k"], case["call"]
    if call == "merge":
        return {"bytes": 8 * P * (2 * k + k), "flops": P * k}
    if call == "naive":
        return {"bytes": 8 * P * k + 4 * m + 8 * k, "flops": P * k + m}
    n = 12 * P * m + 8 * P * k + 8 * k       # two rows in, one out; the local sets; the global set
    if call == "parts":                      # the sets come in again for the tree, then for the restore
        n += 8 * P * k + 8 * P * k + 8 * P * k + 8 * k + 8 * k
    return {"bytes": n, "flops": P * m + P * k}


def tolerance(case):
    # every value is a copy or one IEEE fp32 operation in a fixed order, every index follows
    # from those by an order without ties
    return "exact"


# ---- the same in 64 bits ------------------------------------------------------------
# Which entries are selected is defined on the fp32 magnitudes (of the fp32 sums) and,
# among equals, on the index; the values are carried in 64 bits.

def _top(mag, k):
    """Positions, ascending, of the k largest of `mag` (fp32, >= 0), the lower position first
    among equals."""
    if k >= mag.numel():
        return torch.arange(mag.numel(), device=mag.device)
    kth = torch.topk(mag, k, sorted=False).values.min()
    above = (mag > kth).nonzero().view(-1)
    ties = (mag == kth).nonzero().view(-1)[:k - above.numel()]
    return torch.cat([above, ties]).sort().values


def _merge(a, b, k):
    """Top-k operation on two sets (idx, fp32 value, fp64 value)."""
    idx, inv = torch.unique(torch.cat([a[0], b[0]]), return_inverse=True)
    n = a[0].numel()
    v32 = torch.zeros(idx.numel(), device=idx.device)
    v64 = torch.zeros(idx.numel(), device=idx.device, dtype=torch.float64)
    v32[inv[:n]] = a[1]
    v64[inv[:n]] = a[2]
    v32[inv[n:]] += b[1]
    v64[inv[n:]] += b[2]
    at = _top(v32.abs(), k)
    return idx[at], v32[at], v64[at]


def exact(case, seed):
    m, P, k, call = case["m"], case["P"], case["k"], case["call"]
    if call == "merge":
        idx, val = _sets(case, 2 * P, seed)
        sets = [(idx[i].long(), val[i], val[i].double()) for i in range(2 * P)]
        got = [_merge(sets[p], sets[P + p], k) for p in range(P)]
        return {"idx": torch.stack([g[0] for g in got]).to(torch.int32),
                "val": torch.stack([g[2] for g in got])}
    if call == "naive":
        idx, val = _sets(case, P, seed)
        d32 = torch.zeros(m, device="cuda")
        d64 = torch.zeros(m, device="cuda", dtype=torch.float64)
        for w in range(P):
            d32[idx[w].long()] += val[w]
            d64[idx[w].long()] += val[w].double()
        d32, d64 = d32 / P, d64 / P
        at = _top(d32.abs(), k)
        return {"dense": d64, "g_idx": at.to(torch.int32), "g_val": d64[at]}
    grads, res = _rows(case, seed)
    residual = torch.empty((P, m), device="cuda", dtype=torch.float64)
    sets = []
    for w in range(P):
        acc = res[w].double() + grads[w * m:(w + 1) * m].double()
        acc32 = acc.float()
        at = _top(acc32.abs(), k)
        sets.append((at, acc32[at], acc[at]))
        residual[w] = acc
    del grads, res
    level = sets
    while len(level) > 1:
        level = [_merge(level[i], level[i + 1], k) for i in range(0, len(level), 2)]
    g = (level[0][0], level[0][1] / P, level[0][2] / P)
    lost = torch.zeros(m, dtype=torch.bool, device="cuda")
    lost[g[0]] = True
    for w in range(P):
        at = sets[w][0]
        residual[w, at[lost[at]]] = 0.0
    out = {"loc_idx": torch.stack([x[0] for x in sets]).to(torch.int32),
           "loc_val": torch.stack([x[2] for x in sets]),
           "g_idx": g[0].to(torch.int32), "g_val": g[2], "residual": residual}
    if call == "parts":
        w = torch.empty(m, device="cuda").normal_(generator=_gen(seed, 4)).mul_(0.05).double()
        w[g[0]] -= LR * g[2]
        out["weights"] = w
    return out
