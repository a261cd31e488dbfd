"""Workloads that a program built on this library runs, for timing it.

Each case is one pass through the public entry points on inputs that already
lie in GPU memory, from the smallest calls (where launches and latency count)
to outputs of several gigabytes: 2-way and 3-way calls on general (some
entries missing) and complete data, threshold-filtered output, a rectangle of
pairs over field chunks with running tallies, a batch of uneven problems, and
multi-allelic markers.  All take the default path (matrix cores); the
popcount path computes the same tables for cross-checks and the int8 operands
serve beyond four million fields, and neither is what a program asks for at
these sizes.

Genotypes follow the repository's generators: per-marker allele frequency
from the Beta(1/2, 1/2) law, Hardy-Weinberg genotypes, missing entries at
random.  Where output is filtered by a threshold the markers come in linked
groups of eight, as neighbouring markers on a chromosome do; unlinked ones
would have nothing to report.
"""
import math

import torch

import paper_1705_08213_amd as ccc

GAMMA = 2.0 / 3.0
GROUP = 8  # linked markers per group
EDGES = 6  # room in an edge list, per marker (a group has 3.5 pairs per marker)


def listed():
    return [
        # a pilot panel: the smallest ordinary call, all launches and latency
        {"name": "pairs_pilot", "kind": "pairs", "n_v": 200, "n_f": 1337, "missing": 0.01},
        # a gene panel against a trial's samples: one wave of tiles or two
        {"name": "pairs_panel", "kind": "pairs", "n_v": 3000, "n_f": 9973, "missing": 0.01},
        # few candidate markers over a biobank's samples: long fields
        {"name": "pairs_cohort", "kind": "pairs", "n_v": 384, "n_f": 250007, "missing": 0.02},
        # a chromosome: throughput, general data
        {"name": "pairs_chromosome", "kind": "pairs", "n_v": 16384, "n_f": 32768, "missing": 0.01},
        # imputed (so complete) data at the same scale, sizes off the tiles
        {"name": "pairs_imputed", "kind": "pairs", "n_v": 16000, "n_f": 40000, "missing": 0.0},
        # network construction: only pairs above a threshold are kept
        {"name": "pairs_filtered", "kind": "pairs_select", "n_v": 12000, "n_f": 8009,
         "missing": 0.01, "threshold": 0.16},
        # triples of a candidate list: the smallest 3-way call
        {"name": "triples_candidates", "kind": "triples", "n_v": 90, "n_f": 2504,
         "missing": 0.005},
        # triples of a panel, general data: 6 GB of output
        {"name": "triples_panel", "kind": "triples", "n_v": 720, "n_f": 16384, "missing": 0.005},
        # triples of an imputed panel, odd sizes
        {"name": "triples_imputed", "kind": "triples", "n_v": 641, "n_f": 5003, "missing": 0.0},
        # one off-diagonal block of a larger matrix, fields arriving in chunks
        {"name": "block_chunks", "kind": "block", "n_a": 6000, "n_b": 5000, "n_f": 65536,
         "chunk": 8192, "missing": 0.02},
        # one problem per gene or region, uneven sizes, run as a batch
        {"name": "batch_regions", "kind": "batch", "n_probs": 64, "v_lo": 64, "v_hi": 2048,
         "f_lo": 1000, "f_hi": 20000, "mix": 5, "missing": 0.01},
        # multi-allelic markers, four states
        {"name": "multi_four", "kind": "multi", "n_v": 4096, "n_f": 16384, "states": 4,
         "missing": 0.01},
    ]


# the most a drawn case may cost: (pair fields, pairs) of the largest calls above
MOST_PAIRS, MOST_PAIR_FIELDS = 16000 * 15999 // 2, 16000 * 15999 // 2 * 32768
MOST_TRIPLES, MOST_TRIPLE_FIELDS = 720 * 719 * 718 // 6, 720 * 719 * 718 // 6 * 16384


def _spread(rng, lo, hi):
    """A whole number, even over the logarithm of [lo, hi]."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["pairs", "pairs", "pairs", "pairs_select", "triples", "triples", "block",
                       "batch", "multi"])
    missing = rng.choice([0.0, 0.002, 0.01, 0.01, 0.02, 0.05])
    while True:
        if kind == "pairs":
            c = {"kind": kind, "n_v": _spread(rng, 40, 16384), "n_f": _spread(rng, 300, 400000)}
            pairs = ccc.n_pairs(c["n_v"])
            fits = pairs <= MOST_PAIRS and pairs * c["n_f"] <= MOST_PAIR_FIELDS
        elif kind == "pairs_select":
            c = {"kind": kind, "n_v": _spread(rng, 500, 14000), "n_f": _spread(rng, 4000, 40000),
                 "threshold": 0.165}
            pairs = ccc.n_pairs(c["n_v"])
            fits = pairs * c["n_f"] <= MOST_PAIR_FIELDS
        elif kind == "triples":
            c = {"kind": kind, "n_v": _spread(rng, 24, 720), "n_f": _spread(rng, 300, 60000)}
            triples = ccc.n_triples(c["n_v"])
            fits = triples <= MOST_TRIPLES and triples * c["n_f"] <= MOST_TRIPLE_FIELDS
        elif kind == "block":
            chunk = 64 * _spread(rng, 16, 512)
            c = {"kind": kind, "n_a": _spread(rng, 200, 8000), "n_b": _spread(rng, 200, 8000),
                 "n_f": rng.randint(chunk // 2, 6 * chunk), "chunk": chunk}
            fits = c["n_a"] * c["n_b"] * c["n_f"] <= 6000 * 5000 * 65536
        elif kind == "batch":
            v_hi, f_hi = _spread(rng, 128, 2048), _spread(rng, 2000, 20000)
            c = {"kind": kind, "n_probs": _spread(rng, 8, 64), "v_lo": rng.randint(33, v_hi // 2),
                 "v_hi": v_hi, "f_lo": rng.randint(500, f_hi // 2), "f_hi": f_hi,
                 "mix": rng.randint(1, 10 ** 6)}
            fits = True
        else:
            c = {"kind": kind, "n_v": _spread(rng, 60, 4096), "n_f": _spread(rng, 300, 50000),
                 "states": rng.choice([2, 3, 4])}
            fits = ccc.n_pairs(c["n_v"]) * c["n_f"] <= ccc.n_pairs(4096) * 16384
        if fits:
            c["missing"] = missing
            return c


def _batch_sizes(case):
    """(n_v, n_f) of every problem of a batch: n_v even over its logarithm."""
    x, sizes = case["mix"], []
    for _ in range(case["n_probs"]):
        u = []
        for _ in range(2):
            x = (x * 6364136223846793005 + 1442695040888963407) % (1 << 64)
            u.append((x >> 11) / float(1 << 53))
        n_v = int(case["v_lo"] * (case["v_hi"] / case["v_lo"]) ** u[0])
        sizes.append((n_v, int(case["f_lo"] + u[1] * (case["f_hi"] - case["f_lo"]))))
    return sizes


def _packed(gen, n_v, n_f, missing, linked=False):
    """Packed rows uint8 [n_v, ld]; what lies past n_f is random too."""
    ld = (n_f + 63) // 64 * 16
    width = 4 * ld
    v = torch.empty((n_v, ld), dtype=torch.uint8, device="cuda")
    rows = max(GROUP, (1 << 27) // width // GROUP * GROUP)
    for r0 in range(0, n_v, rows):
        m = min(rows, n_v - r0)

        def uniform(n=m, w=width):
            return torch.rand((n, w), generator=gen, device="cuda")

        if linked:
            groups = (m + GROUP - 1) // GROUP
            p = torch.rand((groups, 1), generator=gen, device="cuda")
            p = p.repeat_interleave(GROUP, 0)[:m]
        else:
            p = uniform(w=1)
        p = torch.sin(0.5 * math.pi * p) ** 2
        ones = torch.zeros((m, width), dtype=torch.uint8, device="cuda")
        for _ in range(2):  # the two alleles of an entry
            u = uniform()
            if linked:  # most haplotypes carry the group's
                shared = uniform(groups).repeat_interleave(GROUP, 0)[:m]
                u = torch.where(uniform() < 0.9, shared, u)
            ones += u >= p
        code = torch.where(ones == 2, 3, ones)
        if missing > 0:
            code = torch.where(uniform() < missing, 2, code)
        code = code.to(torch.uint8).view(m, ld, 4)
        v[r0:r0 + m] = (code[..., 0] | (code[..., 1] << 2) | (code[..., 2] << 4)
                        | (code[..., 3] << 6))
    return v


def _multi_bytes(gen, n_v, n_f, s, missing):
    """One byte per field, bits 2a and 2a + 1 the copies of state a."""
    ld = (n_f + 15) // 16 * 16
    v = torch.empty((n_v, ld), dtype=torch.uint8, device="cuda")
    rows = max(1, (1 << 27) // ld)
    for r0 in range(0, n_v, rows):
        m = min(rows, n_v - r0)
        w = torch.sin(0.5 * math.pi * torch.rand((m, s), generator=gen, device="cuda")) ** 2 + 1e-3
        edge = torch.cumsum(w, 1) / w.sum(1, keepdim=True)
        out = torch.zeros((m, ld), dtype=torch.int32, device="cuda")
        for _ in range(2):
            u = torch.rand((m, ld), generator=gen, device="cuda")
            state = torch.zeros((m, ld), dtype=torch.int32, device="cuda")
            for a in range(s - 1):
                state += u >= edge[:, a:a + 1]
            out += torch.bitwise_left_shift(torch.ones_like(state), 2 * state)
        if missing > 0:
            out[torch.rand((m, ld), generator=gen, device="cuda") < missing] = 0
        v[r0:r0 + m] = out.to(torch.uint8)
    return v


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind, missing = case["kind"], case["missing"]
    if kind == "multi":
        v = _multi_bytes(gen, case["n_v"], case["n_f"], case["states"], missing)
        return {"case": case, "v": v}
    if kind == "block":
        n_a, n_b = case["n_a"], case["n_b"]

        def buffer(shape, dtype):
            return torch.zeros(shape, dtype=dtype, device="cuda")

        return {"case": case,
                "va": _packed(gen, n_a, case["n_f"], missing),
                "vb": _packed(gen, n_b, case["n_f"], missing),
                # the running state of a chunked block is the program's own
                "tables": buffer((n_a, n_b, 4), torch.int32),
                "ccc": buffer((n_a, n_b, 4), torch.float64),
                "counts_a": buffer((n_a, 4), torch.int32),
                "counts_b": buffer((n_b, 4), torch.int32)}
    if kind == "batch":
        # a program that runs a batch again keeps its buffers: one array of
        # each kind, a stretch of it for every problem
        sizes = _batch_sizes(case)
        pairs, rows = sum(ccc.n_pairs(n) for n, _ in sizes), sum(n for n, _ in sizes)
        tables = torch.zeros((pairs, 4), dtype=torch.int32, device="cuda")
        values = torch.zeros((pairs, 4), dtype=torch.float64, device="cuda")
        counts = torch.zeros((rows, 4), dtype=torch.int32, device="cuda")
        probs, p, r = [], 0, 0
        for n_v, n_f in sizes:
            q = p + ccc.n_pairs(n_v)
            probs.append({"v": _packed(gen, n_v, n_f, missing), "n_f": n_f,
                          "tables": tables[p:q], "ccc": values[p:q], "counts": counts[r:r + n_v]})
            p, r = q, r + n_v
        return {"case": case, "probs": probs, "outs": (tables, values, counts)}
    linked = kind == "pairs_select"
    state = {"case": case, "v": _packed(gen, case["n_v"], case["n_f"], missing, linked)}
    if linked:
        state["edges"] = _edges(case)
    return state


def _edges(case):
    """An empty edge list: pair index (-1: none), values, tables."""
    n = EDGES * case["n_v"]
    return (torch.full((n,), -1, dtype=torch.int64, device="cuda"),
            torch.zeros((n, 4), dtype=torch.float64, device="cuda"),
            torch.zeros((n, 4), dtype=torch.int32, device="cuda"))


def _chunks(case):
    """(first field, fields) of every chunk of a block."""
    return [(f, min(case["chunk"], case["n_f"] - f)) for f in range(0, case["n_f"], case["chunk"])]


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "pairs":
        return ccc.ccc_2way(state["v"], case["n_f"])
    if kind == "pairs_select":
        found, index, values, tables = ccc.ccc_2way_select(
            state["v"], case["n_f"], case["threshold"], cap=EDGES * case["n_v"])
        # records come in no particular order: the program puts them into its
        # edge list in pair order
        index, order = torch.sort(index)
        edges, n = state["edges"], index.shape[0]
        edges[0][:n], edges[0][n:] = index, -1
        edges[1][:n], edges[1][n:] = values[order], 0
        edges[2][:n], edges[2][n:] = tables[order], 0
        return (found,) + edges
    if kind == "triples":
        return ccc.ccc_3way(state["v"], case["n_f"])
    if kind == "block":
        chunks = _chunks(case)
        for f, n in chunks:
            ccc.ccc_2way_block(state["va"], state["vb"], n, state["tables"], state["counts_a"],
                               state["counts_b"], state["ccc"], accumulate=f > 0,
                               finalize=f == chunks[-1][0], field_offset=f // 4)
        return state["tables"], state["ccc"], state["counts_a"], state["counts_b"]
    if kind == "batch":
        ccc.ccc_2way_many(state["probs"])
        return state["outs"]
    return ccc.ccc_2way_multi(state["v"], case["n_f"], case["states"])


def work(case):
    """Bytes read and written once, and 2 operations per multiply-add: four
    (2-way) or eight (3-way) products per comparison on general data, one on
    complete data, s^2 for s states."""
    kind = case["kind"]
    if kind == "multi":
        pairs, s = ccc.n_pairs(case["n_v"]), case["states"]
        return {"bytes": case["n_v"] * case["n_f"] + pairs * 12 * s * s + 32 * case["n_v"],
                "flops": 2.0 * s * s * pairs * case["n_f"]}
    products = 1 if case["missing"] == 0 else 4
    if kind == "block":
        rows, pairs = case["n_a"] + case["n_b"], case["n_a"] * case["n_b"]
        tallies = len(_chunks(case))  # a chunk's tables are updated, and the first one's written
        return {"bytes": rows * case["n_f"] / 4 + pairs * (16 * (2 * tallies - 1) + 32) + 16 * rows,
                "flops": 2.0 * products * pairs * case["n_f"]}
    if kind == "batch":
        total = {"bytes": 0.0, "flops": 0.0}
        for n_v, n_f in _batch_sizes(case):
            pairs = ccc.n_pairs(n_v)
            total["bytes"] += n_v * n_f / 4 + 48 * pairs + 16 * n_v
            total["flops"] += 2.0 * products * pairs * n_f
        return total
    n_v, n_f = case["n_v"], case["n_f"]
    if kind == "triples":
        triples = ccc.n_triples(n_v)
        return {"bytes": n_v * n_f / 4 + 96 * triples + 16 * n_v,
                "flops": 2.0 * (1 if case["missing"] == 0 else 8) * triples * n_f}
    pairs = ccc.n_pairs(n_v)
    out = 48 * pairs if kind == "pairs" else 0
    return {"bytes": n_v * n_f / 4 + out + 16 * n_v, "flops": 2.0 * products * pairs * n_f}


# ---------------------------------------------------------------------------
# The definitions in float64: sums of products of small whole numbers are
# exact there, and the correlation values follow the formula left to right.
# ---------------------------------------------------------------------------

def _planes(v, n_f):
    """Copies of allele 0 and of allele 1 of every entry, float64 [2][n, n_f]."""
    code = torch.stack([(v >> s) & 3 for s in (0, 2, 4, 6)], -1).view(v.shape[0], -1)[:, :n_f]
    table = torch.tensor([[2, 1, 0, 0], [0, 1, 0, 2]], dtype=torch.float64, device=v.device)
    return [table[a][code.to(torch.int32)] for a in (0, 1)]


def _counts(planes):
    n = [p.sum(1) for p in planes]
    m = sum(n) / 2
    w = [1 - GAMMA * torch.where(m > 0, x / (2 * m).clamp(min=1), 0.0) for x in n]
    return n, m, w


def _counts4(planes):
    n, m, _ = _counts(planes)
    return torch.stack([n[0], n[1], m, torch.zeros_like(m)], 1).to(torch.int32)


def _pair_values(C, wa, wb):
    """Values of tables C [..., A * B] with row factors wa and column factors
    wb (lists of tensors that fit C's leading dimensions)."""
    den = C.sum(-1)  # 4 m
    values = torch.empty_like(C)
    for a, x in enumerate(wa):
        for b, y in enumerate(wb):
            e = a * len(wb) + b
            values[..., e] = torch.where(den > 0, C[..., e] / den.clamp(min=1) * x * y, 0.0)
    return values


def _pairs_exact(planes):
    n, s = planes[0].shape[0], len(planes)
    _, _, w = _counts(planes)
    i, j = torch.triu_indices(n, n, 1, device=planes[0].device)
    C = torch.empty((i.shape[0], s * s), dtype=torch.float64, device=i.device)
    for a in range(s):
        for b in range(s):
            C[:, a * s + b] = (planes[a] @ planes[b].t())[i, j]
    return C.to(torch.int32), _pair_values(C, [x[i] for x in w], [x[j] for x in w])


def _triples_exact(planes):
    n = planes[0].shape[0]
    _, _, w = _counts(planes)
    T = ccc.n_triples(n)
    tables = torch.empty((T, 8), dtype=torch.int32, device=planes[0].device)
    values = torch.empty((T, 8), dtype=torch.float64, device=planes[0].device)
    t = 0
    for i in range(n - 2):
        m = n - 1 - i
        J, K = torch.triu_indices(m, m, 1, device=tables.device)
        rest = torch.cat([p[i + 1:] for p in planes])
        C = torch.empty((J.shape[0], 8), dtype=torch.float64, device=tables.device)
        for a in range(2):
            G = (rest * planes[a][i]) @ rest.t()
            for b in range(2):
                for c in range(2):
                    C[:, 4 * a + 2 * b + c] = G[J + m * b, K + m * c]
        den = C.sum(1)
        part = slice(t, t + J.shape[0])
        tables[part] = C.to(torch.int32)
        for a in range(2):
            for b in range(2):
                for c in range(2):
                    e = 4 * a + 2 * b + c
                    values[part, e] = torch.where(
                        den > 0, C[:, e] / den.clamp(min=1) * w[a][i] * w[b][i + 1 + J]
                        * w[c][i + 1 + K], 0.0)
        t += J.shape[0]
    return tables, values


def exact(case, seed):
    kind, state = case["kind"], prepare(case, seed)
    if kind == "batch":
        outs = []
        for p in state["probs"]:
            planes = _planes(p["v"], p["n_f"])
            outs.append(_pairs_exact(planes) + (_counts4(planes),))
        return tuple(torch.cat(x) for x in zip(*outs))
    if kind == "block":
        pa, pb = _planes(state["va"], case["n_f"]), _planes(state["vb"], case["n_f"])
        _, _, wa = _counts(pa)
        _, _, wb = _counts(pb)
        C = torch.stack([x @ y.t() for x in pa for y in pb], -1)
        values = _pair_values(C, [x[:, None] for x in wa], [y[None, :] for y in wb])
        return C.to(torch.int32), values, _counts4(pa), _counts4(pb)
    if kind == "multi":
        s = case["states"]
        v = state["v"][:, :case["n_f"]]
        planes = [((v >> (2 * a)) & 3).to(torch.float64) for a in range(s)]
        n = [p.sum(1) for p in planes]
        counts = torch.zeros((case["n_v"], 8), dtype=torch.int32, device=v.device)
        for a in range(s):
            counts[:, a] = n[a].to(torch.int32)
        counts[:, 4] = (sum(n) / 2).to(torch.int32)
        return _pairs_exact(planes) + (counts,)
    planes = _planes(state["v"], case["n_f"])
    if kind == "triples":
        return _triples_exact(planes) + (_counts4(planes),)
    tables, values = _pairs_exact(planes)
    if kind == "pairs":
        return tables, values, _counts4(planes)
    keep = (values >= case["threshold"]).any(1).nonzero()[:, 0]
    edges, n = _edges(case), keep.shape[0]
    for out, kept in zip(edges, (keep, values[keep], tables[keep])):
        out[:n] = kept
    return (int(n),) + edges
