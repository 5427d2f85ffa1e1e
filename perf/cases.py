"""The work that programs have this library do, as cases that can be timed and compared.

Each case is one pass through the public entry points of `paper_2103_00130_amd.binding` at one size: a checked layer
(`abft_gemm_u8s8s32_checked`), a checked embedding lookup (`abft_eb_u8_checked`), or a weight that is encoded anew and put to use
(`abft_pack_b_checksum`).  `listed()` names the sizes that stand for each kind of use, `draw()` gives more sizes of the same ranges,
`prepare()` makes what the program holds before the call, `run()` is the call.

Values follow the paper's recipe as `workloads.py` and `eb_workloads.py` draw them: uniform uint8 activations (or 40 % zeros after a
ReLU), uniform int8 weights, multipliers log-uniform on [1e-4, 1e-2]; embedding tables of uniform codes with one scale and bias per row.
"""
from __future__ import annotations

import math

import torch

from paper_2103_00130_amd import binding as b

DENSE = 4096 ** 3      # multiply-adds of the largest listed layer
WEIGHT = 16384 ** 2    # entries of the largest listed weight
GATHER = 16384 * 100 * 80   # record bytes of the largest listed lookup


def layer(name, M, N, K, out="C", scale="none", relu=False, count="overwrite", hit=False):
    """A fully connected layer: M requests, N outputs, K inputs.  out: "C" (32-bit), "q" (requantized only) or "both"; scale: one
    multiplier per tensor or per output channel (with a bias); relu: activations as after a ReLU; count: errCount overwritten by the
    call or kept as a running counter; hit: one bit of the packed weight is inverted, so that rows are flagged."""
    return {"name": name, "kind": "layer", "M": M, "N": N, "K": K, "out": out, "scale": scale, "relu": relu, "count": count, "hit": hit}


def lookup(name, rows, d, bags, pool, bits=8, lengths="spread", weighted=False, aligned=False):
    """An embedding lookup: `bags` index sets of `pool` rows on average from a table of rows x d codes."""
    return {"name": name, "kind": "lookup", "rows": rows, "d": d, "bags": bags, "pool": pool, "bits": bits, "lengths": lengths,
            "weighted": weighted, "aligned": aligned}


def refresh(name, M, N, K):
    """A weight of N x K (a torch Linear weight) replaced in a running program: encoded and packed, then used on M rows."""
    return {"name": name, "kind": "refresh", "M": M, "N": N, "K": K}


def listed():
    return [
        # the smallest layer of the benchmark: a call of a few microseconds, where launches and host work count
        layer("fc_64x256x512", 64, 256, 512),
        # a bottom-MLP layer of a recommendation model, requantized for the next layer
        layer("fc_bottom_256x512x1024", 256, 512, 1024, out="q", scale="tensor"),
        # one request: the shape that the paper names
        layer("fc_one_row_1x800x3200", 1, 800, 3200),
        # a small batch against a weight of 8 MiB
        layer("fc_tall_skinny_16x4096x2048", 16, 4096, 2048, count="accumulate"),
        # a top-MLP layer with a multiplier and a bias per output channel
        layer("fc_top_1024x1024x4096", 1024, 1024, 4096, out="q", scale="channel", relu=True),
        # a top MLP's first layer: its input is the feature interaction, whose width has no even factor; the weight has been hit
        layer("fc_ragged_2000x1000x479", 2000, 1000, 479, out="both", scale="channel", hit=True),
        # a small batch against a weight that fills memory, not caches
        layer("fc_stream_16x16384x16384", 16, 16384, 16384),
        # the dense layer that the benchmark quotes
        layer("fc_dense_4096", 4096, 4096, 4096),
        # the paper's embedding lookup (its Table I): ten index sets
        lookup("eb_table1_d64_batch10", 4_000_000, 64, 10, 100),
        # the same table under a serving batch
        lookup("eb_d64_batch16384", 4_000_000, 64, 16384, 100),
        # a 4-bit table, weighted sum, index sets of very different lengths (empty ones among them)
        lookup("eb_int4_d128_ragged", 2_000_000, 128, 3000, 60, bits=4, lengths="ragged", weighted=True, aligned=True),
        # a weight of 16 MiB replaced while the program runs, and its first batch
        refresh("refresh_64x4096x4096", 64, 4096, 4096),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(("layer", "layer", "layer", "layer", "lookup", "lookup", "refresh"))
    if kind == "lookup":
        bits = rng.choice((8, 8, 4))
        d = rng.choice((32, 64, 128, 256)) * (1 if bits == 8 else 2)
        record = d * bits // 8 + 16
        pool = _log_int(rng, 1, 200)
        bags = _log_int(rng, 1, min(16384, GATHER // (2 * pool * record)))
        case = lookup("", rng.randrange(100_000, 4_000_001), d, bags, pool, bits, rng.choice(("spread", "fixed", "ragged")),
                      rng.random() < 0.4, rng.random() < 0.3)
    elif kind == "refresh":
        case = refresh("", _log_int(rng, 16, 64), _log_int(rng, 256, 4096), _log_int(rng, 256, 4096))
    else:
        K = _log_int(rng, 64, 16384)
        aligned = rng.random() < 0.7
        if aligned:
            K = (K + 15) // 16 * 16    # most layers: widths that keep rows aligned
        N = _log_int(rng, 64, min(16384, WEIGHT // K))
        if rng.random() < 0.5:
            N = (N + 15) // 16 * 16
        M = _log_int(rng, 1, min(4096, max(1, DENSE // ((1 if aligned else 8) * N * K))))
        out, count = rng.choice((("C", "overwrite"), ("C", "accumulate"), ("q", "overwrite"), ("both", "overwrite")))
        case = layer("", M, N, K, out, "none" if out == "C" else rng.choice(("tensor", "channel")), rng.random() < 0.3, count,
                     count == "overwrite" and rng.random() < 0.3)
    del case["name"]
    return case


# ---- inputs, from the seed alone -------------------------------------------------------------

def _gen(seed, what):
    return torch.Generator("cuda").manual_seed(1000 * seed + what)


def _activations(case, seed):
    g = _gen(seed, 1)
    A = torch.randint(0, 256, (case["M"], case["K"]), dtype=torch.uint8, device="cuda", generator=g)
    if case.get("relu"):
        A[torch.rand(A.shape, device="cuda", generator=g) < 0.4] = 0
    return A


def _weight(case, seed):
    """N x K, as a torch Linear holds it."""
    return torch.randint(-127, 128, (case["N"], case["K"]), dtype=torch.int8, device="cuda", generator=_gen(seed, 2))


def _requant(case, seed):
    """zA, zC, multipliers and bias of a layer that is requantized."""
    if case["scale"] == "none":
        return None
    g = _gen(seed, 3)
    channel = case["scale"] == "channel"
    u = torch.rand(case["N"] if channel else 1, device="cuda", generator=g)
    mult = torch.exp(math.log(1e-4) + u * math.log(1e2)).float()
    bias = torch.randint(-20000, 20001, (case["N"],), dtype=torch.int32, device="cuda", generator=g) if channel else None
    return (0 if case["relu"] else 128), 128, mult, bias


def _hit(case, seed):
    """(k, j, bit) of the weight element that a soft error has inverted."""
    return (seed * 7919 + 13) % case["K"], (seed * 104729 + 7) % case["N"], seed % 8


def _table(case, seed):
    g = _gen(seed, 4)
    rows, top = case["rows"], (1 << case["bits"]) - 1
    T = torch.randint(0, 256, (rows, case["d"] * case["bits"] // 8), dtype=torch.uint8, device="cuda", generator=g)
    scale = (0.005 + 0.015 * torch.rand(rows, device="cuda", generator=g)) * (255 // top)
    bias = -0.5 * torch.rand(rows, device="cuda", generator=g)
    return T, scale, bias


def _bags(case, seed):
    g = _gen(seed, 5)
    n, pool = case["bags"], case["pool"]
    if case["lengths"] == "fixed":
        sizes = torch.full((n,), pool, dtype=torch.int64, device="cuda")
    elif case["lengths"] == "spread":
        sizes = torch.randint(pool // 2, pool + pool // 2 + 1, (n,), device="cuda", generator=g)
    else:   # geometric, cut at four times the mean; one in ten empty
        u = torch.rand(n, device="cuda", generator=g).clamp_min(1e-9)
        sizes = (-pool * torch.log(u)).to(torch.int64).clamp_max(4 * pool)
        sizes[torch.rand(n, device="cuda", generator=g) < 0.1] = 0
    offsets = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(sizes, 0, out=offsets[1:])
    total = int(offsets[-1])
    indices = torch.randint(0, case["rows"], (total,), device="cuda", generator=g)
    weights = 0.25 + 1.5 * torch.rand(total, device="cuda", generator=g) if case["weighted"] else None
    return indices, offsets, weights


# ---- what a program holds, and its call --------------------------------------------------------

def prepare(case, seed):
    s = {"case": case}
    if case["kind"] == "lookup":
        T, scale, bias = _table(case, seed)
        pack = (b.ABFT_EB_PACK_INT4 if case["bits"] == 4 else 0) | (b.ABFT_EB_PACK_LINE_ALIGNED if case["aligned"] else 0)
        s["table"] = b.abft_eb_pack_rowsum(T, scale, bias, flags=pack)
        torch.cuda.synchronize()    # the codes are dropped once they have been packed
        s["indices"], s["offsets"], s["weights"] = _bags(case, seed)
        s["R"] = torch.empty(case["bags"], case["d"], device="cuda")
        s["flags"] = torch.empty(case["bags"], dtype=torch.int32, device="cuda")
        return s
    M, N, K = case["M"], case["N"], case["K"]
    s["A"] = _activations(case, seed)
    W = _weight(case, seed)
    s["Bp"] = b.abft_pack_b_checksum(W, b_is_transposed=True)
    s["ws"] = b.Workspace(M, s["Bp"]).tensor
    s["row_flags"] = torch.empty(M, dtype=torch.int32, device="cuda")
    s["count"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    s["C"] = s["Cq"] = s["rq"] = None
    if case["kind"] == "refresh":
        s["W"] = _weight(case, seed + 500_000_000)    # the version that replaces the packed one
        s["C"] = torch.empty(M, N, dtype=torch.int32, device="cuda")
        s["S_B"] = torch.empty(K, dtype=torch.int32, device="cuda")
        s["colsum"] = torch.empty(N, dtype=torch.int32, device="cuda")
    else:
        if case["hit"]:
            b.abft_packed_b_flip_bit(s["Bp"], *_hit(case, seed))
        if case["out"] != "q":
            s["C"] = torch.empty(M, N, dtype=torch.int32, device="cuda")
        if case["out"] != "C":
            zA, zC, mult, bias = s["requant"] = _requant(case, seed)
            s["rq"] = b.make_requant(zA, zC, mult, bias)
            s["Cq"] = torch.empty(M, N, dtype=torch.uint8, device="cuda")
        s["how"] = b.ABFT_ERRCOUNT_ACCUMULATE if case["count"] == "accumulate" else b.ABFT_CHECK
    torch.cuda.synchronize()
    return s


def run(state):
    s = state
    kind = s["case"]["kind"]
    if kind == "lookup":
        b.abft_eb_u8_checked(s["table"], s["indices"], s["offsets"], s["R"], s["flags"], weights=s["weights"])
        return {"R": s["R"], "flags": s["flags"]}
    if kind == "refresh":
        s["Bp"] = b.abft_pack_b_checksum(s["W"], b_is_transposed=True)    # the version that it replaces is freed
        b.abft_packed_b_get_checksum(s["Bp"], s["S_B"])
        b.abft_packed_b_get_col_offsets(s["Bp"], s["colsum"])
        b.abft_gemm_u8s8s32_checked(s["A"], s["Bp"], s["C"], s["row_flags"], s["count"], workspace=s["ws"])
        return {"C": s["C"], "flags": s["row_flags"], "count": s["count"], "S_B": s["S_B"], "colsum": s["colsum"]}
    b.abft_gemm_u8s8s32_checked(s["A"], s["Bp"], s["C"], s["row_flags"], s["count"], rq=s["rq"], Cq=s["Cq"], flags=s["how"],
                                workspace=s["ws"])
    return {"C": s["C"], "Cq": s["Cq"], "flags": s["row_flags"], "count": s["count"]}


def work(case):
    if case["kind"] == "lookup":
        pooled = case["bags"] * case["pool"] * (0.9 if case["lengths"] == "ragged" else 1)
        record = case["d"] * case["bits"] // 8 + 16 + 8 + (4 if case["weighted"] else 0)    # codes, parameters, index, weight
        return {"bytes": pooled * record + case["bags"] * (4 * case["d"] + 12), "flops": 2 * pooled * case["d"]}
    M, N, K = case["M"], case["N"], case["K"]
    if case["kind"] == "refresh":
        return {"bytes": 2 * N * K + 4 * (K + N) + M * K + 4 * M * N + 4 * M, "flops": 2 * M * N * K}
    out = {"C": 4, "q": 1, "both": 5}[case["out"]]
    return {"bytes": M * K + N * K + out * M * N + 4 * M, "flops": 2 * M * N * K}


def tolerance(case):
    # The layers are integer arithmetic and the requantization a fixed sequence of binary32 operations: the same values everywhere.
    # A lookup sums `pool` binary32 terms per column: 2.1e-7 (largest 1.0e-6) from the sum in 64 bits on these sizes.
    return {"rel": 1e-6, "max": 5e-6} if case["kind"] == "lookup" else "exact"


def exact(case, seed):
    """What run() returns, in 64 bits."""
    if case["kind"] == "lookup":
        T, scale, bias = _table(case, seed)
        indices, offsets, weights = _bags(case, seed)
        d, n = case["d"], case["bags"]
        R = torch.zeros(n, d, dtype=torch.float64, device="cuda")
        bag = torch.repeat_interleave(torch.arange(n, device="cuda"), offsets[1:] - offsets[:-1])
        for at in range(0, indices.numel(), 1 << 18):
            i = indices[at:at + (1 << 18)]
            codes = T[i]
            if case["bits"] == 4:
                codes = torch.stack((codes & 15, codes >> 4), dim=2).reshape(i.numel(), d)
            rows = scale[i].double()[:, None] * codes.double() + bias[i].double()[:, None]
            if weights is not None:
                rows *= weights[at:at + (1 << 18)].double()[:, None]
            R.index_add_(0, bag[at:at + (1 << 18)], rows)
        return {"R": R, "flags": torch.zeros(n, dtype=torch.int64, device="cuda")}
    A = _activations(case, seed)
    fresh = case["kind"] == "refresh"
    W = _weight(case, seed + 500_000_000 if fresh else seed)
    colsum = W.sum(1, dtype=torch.int64)
    S_B = W.sum(0, dtype=torch.int64)
    flags = torch.zeros(case["M"], dtype=torch.int64, device="cuda")
    if not fresh and case["hit"]:
        k, j, bit = _hit(case, seed)
        hit = W.view(torch.uint8)
        hit[j, k] ^= 1 << bit
        flags = (A[:, k] != 0).long()
    # sums below 2^53 are exact in float64
    C = torch.cat([A.double() @ W[at:at + 4096].double().t().contiguous() for at in range(0, case["N"], 4096)], dim=1).long()
    count = flags.sum().reshape(1)
    if fresh:
        return {"C": C, "flags": flags, "count": count, "S_B": S_B, "colsum": colsum}
    Cq = None
    if case["out"] != "C":
        zA, zC, mult, bias = _requant(case, seed)
        t = C - zA * colsum
        if bias is not None:
            t = t + bias
        Cq = (torch.round(t.double() * mult.double()) + zC).clamp(0, 255).long()
    return {"C": C if case["out"] != "q" else None, "Cq": Cq, "flags": flags, "count": count}
