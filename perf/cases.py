"""What a user of this framework has it do, as cases that can be timed.

A case is one pass through the public entry points on one synthetic input of the workload classes of
`paper_2504_04673_amd/workloads.py`: Erdos-Renyi, R-MAT (power-law) and planted-partition graphs, one rank's row
block of a larger graph, feature widths from 4 to 256.  `listed()` names twelve of them, `draw(rng)` gives more
of the same ranges, `prepare` makes the input on the GPU from a seed together with what a program keeps across
passes (the graph, the weights, the prepared schedule), `run` is the pass.

Kinds of pass:
  step      plan the needed rows, pack them, multiply, dense transform with ReLU: what `bench.py` times
  infer     one layer forward whose intermediate A H is not wanted
  train     two layers forward and backward (the activations whose sign the backward pass takes its ReLU mask
            from are part of the input, so that a result within a rounding of zero decides nothing)
  stages    the 1.5D stage loop of one rank over the column blocks of its row block
  directed  a directed graph is loaded: transpose it, prepare both orientations, first product with each
  reorder   a partitioner's labels become a vertex order: permutation, permuted matrix, rows of H moved
"""
import math

import numpy as np
import torch

import paper_2504_04673_amd as sagnn

DEV = "cuda"
A, B, C = 0.57, 0.19, 0.19                       # R-MAT quadrants of the benchmark configurations
PREC = {"fp32": sagnn.GEMM_FP32, "bf16": sagnn.GEMM_BF16, "fp32x3": sagnn.GEMM_FP32_BF16X3}


def listed():
    return [
        # the smallest call: a few thousand vertices, launches and host work are everything
        {"name": "er_4k_f16_step", "kind": "step", "graph": "er", "n": 4096, "deg": 8, "nb": 4, "f": 16, "f_out": 16,
         "prec": "fp32"},
        # training on a small graph with widths that are no power of two
        {"name": "er_30k_f100_train", "kind": "train", "graph": "er", "n": 30011, "deg": 12, "f": 100, "hidden": 64,
         "f_out": 48, "prec": "fp32"},
        # an ordinary citation-sized power-law graph, 128 features, wide hidden layer
        {"name": "rmat_170k_f128_train", "kind": "train", "graph": "rmat", "n": 170003, "deg": 14, "f": 128,
         "hidden": 256, "f_out": 40, "prec": "fp32"},
        # the paper's own shape of network: 16 hidden units, 24 labels
        {"name": "rmat_1m_f16_train", "kind": "train", "graph": "rmat", "n": 1000000, "deg": 50, "f": 16, "hidden": 16,
         "f_out": 24, "prec": "fp32"},
        # a dense social graph (average degree ~490), one layer forward
        {"name": "rmat_233k_f128_infer", "kind": "infer", "graph": "rmat", "n": 232965, "deg": 489, "f": 128,
         "f_out": 128, "prec": "fp32"},
        # the headline step of the benchmark: 2.45 M vertices, ~124 M stored entries
        {"name": "rmat_2m_f128_step", "kind": "step", "graph": "rmat", "n": 2450000, "deg": 51, "nb": 1, "f": 128,
         "f_out": 128, "prec": "fp32"},
        # one rank's share of a very wide graph: n / 64 rows by n columns in 16 blocks, hardly any row of H used twice
        {"name": "rank_55m_f128_step", "kind": "step", "graph": "rank", "n": 55500000, "deg": 15, "nb": 16, "f": 128,
         "f_out": 128, "prec": "fp32"},
        # the same rank's pass when the blocks arrive one after the other (4 of 16 blocks, two packed buffers)
        {"name": "rank_28m_f128_stages", "kind": "stages", "graph": "rank", "n": 27800000, "deg": 15, "nb": 16,
         "stages": 4, "f": 128},
        # a partitioned graph's first row block with its halo, wide features, bf16 matrix cores
        {"name": "sbm_2m_block_f256_step", "kind": "step", "graph": "sbm_block", "n": 2000000, "deg": 42, "nb": 16,
         "f": 256, "f_out": 256, "prec": "bf16"},
        # the largest: training on the whole partitioned graph
        {"name": "sbm_2m_f256_train", "kind": "train", "graph": "sbm", "n": 2000000, "deg": 42, "f": 256,
         "hidden": 256, "f_out": 256, "prec": "bf16"},
        # set-up of a directed graph
        {"name": "rmat_1m_directed", "kind": "directed", "graph": "rmat_directed", "n": 1000000, "deg": 40, "f": 64},
        # set-up of a vertex order from partition labels
        {"name": "sbm_500k_reorder", "kind": "reorder", "graph": "sbm_random", "n": 500000, "deg": 42, "f": 128},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo=4, hi=256):
    """Half the users have powers of two, the others have what their data gives (a multiple of 4)."""
    common = [w for w in (16, 32, 64, 128, 256) if lo <= w <= hi]
    return rng.choice(common) if rng.random() < 0.5 else 4 * rng.randint((lo + 3) // 4, hi // 4)


def _graph(rng, n_lo, n_hi, nnz_hi):
    n = _log(rng, n_lo, n_hi)
    graph = rng.choice(["er", "rmat", "rmat", "sbm"])
    deg = _log(rng, 4, max(5, min(500 if graph == "rmat" else 64, nnz_hi // n)))
    if graph == "rmat":
        deg = min(deg, max(4, n // 256))          # a small vertex set has no room for a dense power-law tail
    return {"graph": graph, "n": n, "deg": deg}


def draw(rng):
    kind = rng.choice(["step", "step", "step_rank", "step_block", "infer", "train", "train", "stages", "directed", "reorder"])
    prec = rng.choice(["fp32", "fp32", "bf16", "fp32x3"])
    if kind == "step":
        return {"kind": kind, **_graph(rng, 1000, 2450000, 120000000), "nb": rng.choice([1, 4, 16]),
                "f": _width(rng), "f_out": _width(rng), "prec": prec}
    if kind == "step_rank":
        return {"kind": "step", "graph": "rank", "n": _log(rng, 2000000, 55500000), "deg": rng.randint(8, 24), "nb": 16,
                "f": rng.choice([32, 64, 100, 128]), "f_out": _width(rng, 16, 128), "prec": prec}
    if kind == "step_block":
        return {"kind": "step", "graph": "sbm_block", "n": _log(rng, 100000, 2000000), "deg": rng.randint(12, 60), "nb": 16,
                "f": _width(rng, 16), "f_out": _width(rng, 16), "prec": prec}
    if kind == "infer":
        return {"kind": kind, **_graph(rng, 4000, 1000000, 100000000), "f": _width(rng, 16), "f_out": _width(rng, 16), "prec": prec}
    if kind == "train":
        return {"kind": kind, **_graph(rng, 4000, 1000000, 50000000), "f": _width(rng, 8), "hidden": _width(rng, 16),
                "f_out": 4 * rng.randint(2, 32), "prec": prec}
    if kind == "stages":
        return {"kind": kind, "graph": "rank", "n": _log(rng, 1000000, 27800000), "deg": rng.randint(8, 24),
                "nb": rng.choice([8, 16]), "stages": rng.choice([2, 4, 8]), "f": rng.choice([32, 64, 100, 128])}
    if kind == "directed":
        return {"kind": kind, "graph": "rmat_directed", "n": _log(rng, 5000, 1500000), "deg": rng.randint(6, 50),
                "f": rng.choice([16, 32, 64, 100, 128])}
    return {"kind": "reorder", "graph": "sbm_random", "n": _log(rng, 5000, 1000000), "deg": rng.randint(8, 50), "f": _width(rng, 16, 128)}


# ---------------------------------------------------------------------------------------------
# graphs, made on the GPU

def _rmat_ends(count, row_bits, col_bits, gen):
    """Row and column ids of `count` R-MAT draws; with fewer row than column bits the last column bits are drawn
    from the column marginal (a rank's rows are a random subset of the vertices)."""
    r = torch.zeros(count, dtype=torch.int64, device=DEV)
    c = torch.zeros(count, dtype=torch.int64, device=DEV)
    for level in range(col_bits):
        u = torch.rand(count, device=DEV, generator=gen)
        if level < row_bits:
            down = u >= A + B
            r = r * 2 + down
            c = c * 2 + torch.where(down, u >= A + B + C, u >= A)
        else:
            c = c * 2 + (u >= A + C)
    return r, c


def _bits(n):
    return max(1, (n - 1).bit_length())


def _csr(keys, m, n):
    """CSR pattern of sorted distinct keys row * n + col, and the degrees of its rows."""
    row = torch.div(keys, n, rounding_mode="floor")
    deg = torch.bincount(row, minlength=m)
    rp = torch.zeros(m + 1, dtype=torch.int32, device=DEV)
    rp[1:] = torch.cumsum(deg, 0)
    return rp, (keys - row * n).to(torch.int32), row, deg


def _symmetric(und, n):
    """Both directions of undirected edges (keys u * n + v), self loops, values D^-1/2 (A + I) D^-1/2."""
    u = torch.div(und, n, rounding_mode="floor")
    v = und - u * n
    loops = torch.arange(n, device=DEV, dtype=torch.int64) * (n + 1)
    keys = torch.unique(torch.cat([und, v * n + u, loops]))
    rp, ci, row, deg = _csr(keys, n, n)
    s = deg.to(torch.float32).rsqrt()
    return rp, ci, s[row] * s[ci.long()]


def _distinct(want, gen, some):
    """`want` distinct keys out of what `some(count)` draws (it may reject some), a random choice where there are more:
    the number of stored entries is the same for every seed."""
    keys = torch.empty(0, dtype=torch.int64, device=DEV)
    for _ in range(64):
        keys = torch.unique(torch.cat([keys, some(int(1.1 * (want - keys.numel())) + 1024)]))
        if keys.numel() >= want:
            break
    return keys[torch.randperm(keys.numel(), device=DEV, generator=gen)[:want]]


def _graph_of(case, gen):
    """rowptr, colidx, val of the case's matrix, and its number of columns."""
    kind, n, deg = case["graph"], case["n"], case["deg"]
    und = max(1, n * (deg - 1) // 2)              # undirected edges, self loops come on top

    def integers(count, high):
        return torch.randint(high, (count,), device=DEV, generator=gen)

    def undirected(r, c):
        keep = r != c
        return torch.minimum(r, c)[keep] * n + torch.maximum(r, c)[keep]

    if kind in ("rmat", "rmat_directed"):
        bits = _bits(n)
        relabel = torch.randperm(1 << bits, device=DEV, generator=gen)

        def some(count):
            r, c = _rmat_ends(int(count * ((1 << bits) / n) ** 2), bits, bits, gen)
            r, c = relabel[r], relabel[c]
            keep = (r < n) & (c < n) & (r != c)
            return r[keep] * n + c[keep] if kind == "rmat_directed" else undirected(r[keep], c[keep])

        if kind == "rmat":
            return (*_symmetric(_distinct(und, gen, some), n), n)
        rp, ci, row, out = _csr(torch.sort(_distinct(n * deg, gen, some))[0], n, n)
        return rp, ci, (1.0 / out.to(torch.float32))[row], n
    if kind == "er":
        return (*_symmetric(_distinct(und, gen, lambda k: undirected(integers(k, n), integers(k, n))), n), n)
    if kind in ("sbm", "sbm_block", "sbm_random"):
        # 16 equal communities in vertex order; one partner in twenty lies anywhere
        size = n // 16
        perm = torch.randperm(n, device=DEV, generator=gen) if kind == "sbm_random" else None

        def ends(count, rows):
            r = integers(count, rows)
            home = torch.div(r, size, rounding_mode="floor") * size
            away = torch.rand(count, device=DEV, generator=gen) < 0.05
            return r, torch.where(away, integers(count, n), home + integers(count, size))

        if kind == "sbm_block":                   # the first of 16 row blocks, all columns
            def some(count):
                r, c = ends(count, size)
                return (r * n + c)[r != c]

            loops = torch.arange(size, device=DEV, dtype=torch.int64) * (n + 1)
            rp, ci, row, d = _csr(torch.sort(torch.cat([_distinct(size * (deg - 1), gen, some), loops]))[0], size, n)
            return rp, ci, (1.0 / d.to(torch.float32))[row], n

        def some(count):
            r, c = ends(count, size * 16)
            # "sbm_random": the same graph before anybody ordered its vertices
            return undirected(r, c) if perm is None else undirected(perm[r], perm[c])

        return (*_symmetric(_distinct(und, gen, some), n), n)
    # "rank": n / 64 rows of a graph on n vertices, deg entries a row on average, by all n columns
    m = n // 64
    rb, cb = _bits(m), _bits(n)
    rows = torch.randperm(1 << rb, device=DEV, generator=gen)
    cols = torch.randperm(1 << cb, device=DEV, generator=gen)

    def some(count):
        r, c = _rmat_ends(int(count * ((1 << rb) / m) * ((1 << cb) / n)), rb, cb, gen)
        r, c = rows[r], cols[c]
        keep = (r < m) & (c < n) & (r != c)
        return r[keep] * n + c[keep]

    loops = torch.arange(m, device=DEV, dtype=torch.int64) * (n + 1)
    rp, ci, row, d = _csr(torch.sort(torch.cat([_distinct(m * (deg - 1), gen, some), loops]))[0], m, n)
    dc = torch.bincount(ci, minlength=n)
    return rp, ci, (d[row] * dc[ci.long()]).to(torch.float32).rsqrt(), n


# ---------------------------------------------------------------------------------------------

def _normal(gen, *shape):
    return torch.randn(*shape, device=DEV, generator=gen)


def _weight(gen, k, n):
    return torch.randn(k, n, device=DEV, generator=gen) / math.sqrt(k)


def _most_needed(case):
    m, n, nnz, _ = _shape(case)
    if case["graph"] == "rank":
        return min(n, nnz * 7 // 10 + 4096)
    if case["graph"] == "sbm_block":
        return min(n, m + nnz // 16 + 4096)
    return n


def _blocks(n, nb):
    return np.array([q * n // nb for q in range(nb + 1)], dtype=np.int64)


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    kind, f, f_out = case["kind"], case["f"], case.get("f_out")
    rp, ci, va, n = _graph_of(case, gen)
    m, nnz = rp.numel() - 1, ci.numel()
    st = {"kind": kind, "rp": rp, "ci": ci, "va": va, "n": n, "prec": PREC[case.get("prec", "fp32")]}
    st["H"] = H = _normal(gen, n, f)
    if kind == "step":
        # the plan's buffers, the packed buffer and the product's schedule belong to the graph and are kept
        st["blk"] = _blocks(n, case["nb"])
        st["bufs"] = sagnn.plan_buffers(m, n, nnz, case["nb"], rp.device)
        plan = sagnn.spmm_plan_needed_rows(rp, ci, n, st["blk"], bufs=st["bufs"])
        if plan.N > _most_needed(case):
            raise ValueError(f"{plan.N} needed rows do not fit the packed buffer")
        st["W"] = _weight(gen, f, f_out)
        st["ws"] = sagnn.spmm_csr_prepare(rp, plan.colidx_compact, va, plan.N, f)
        # the packed buffer has room for the graphs such a program meets, not for this one alone
        st["bufs"][1].zero_()
        st["Hn"], st["T"] = torch.zeros(_most_needed(case), f, device=DEV), torch.empty(m, f, device=DEV)
    elif kind == "infer":
        st["W"] = _weight(gen, f, f_out)
        st["ws"] = sagnn.spmm_csr_prepare(rp, ci, va, n, f)
        # the library says whether this schedule finishes the layer without storing A H
        st["want_t"] = sagnn.gcn_layer_fwd_form(st["ws"], f, f_out, st["prec"]) != 2
    elif kind == "train":
        h = case["hidden"]
        st["W1"], st["W2"] = _weight(gen, f, h), _weight(gen, h, f_out)
        st["G"], st["Zp"] = _normal(gen, n, f_out), _normal(gen, n, h)
        ws = {w: sagnn.spmm_csr_prepare(rp, ci, va, n, w) for w in {f, h, f_out}}   # one schedule per width in use
        st["ws_in"], st["ws_hid"], st["ws_out"] = ws[f], ws[h], ws[f_out]
    elif kind == "stages":
        blk = _blocks(n, case["nb"])
        plan = sagnn.spmm_plan_needed_rows(rp, ci, n, blk)
        cb = sagnn.spmm_split_colblocks(rp, plan.colidx_compact, va, plan.blk_off)
        stages = []
        for q in range(case["stages"]):
            brp, bci, bva = cb.block(q)
            rows = plan.needed[int(plan.blk_off[q]):int(plan.blk_off[q + 1])]
            stages.append({"rowptr": brp, "colidx": bci, "val": bva, "rows": rows,
                           "ws": sagnn.spmm_csr_prepare(brp, bci, bva, rows.numel(), f)})
        cap = max(s["rows"].numel() for s in stages)
        st["stages"], st["m"] = stages, m
        st["T0"], st["T1"] = torch.empty(cap, f, device=DEV), torch.empty(cap, f, device=DEV)
        st["Z"] = torch.empty(m, f, device=DEV)
    elif kind == "reorder":
        # labels as a partitioner hands them back: sixteen parts of about equal size
        st["labels"] = torch.randint(16, (n,), device=DEV, generator=gen).to(torch.int32)
    del H
    return st


def run(st):
    kind, rp, ci, va, H, prec = st["kind"], st["rp"], st["ci"], st["va"], st["H"], st["prec"]
    if kind == "step":
        p = sagnn.spmm_plan_needed_rows(rp, ci, st["n"], st["blk"], bufs=st["bufs"])
        Hn = sagnn.spmm_pack_rows(H, p.needed, out=st["Hn"][:p.N])
        sagnn.spmm_csr_tallskinny(rp, p.colidx_compact, va, Hn, C=st["T"], ws=st["ws"])
        _, out = sagnn.dense_gemm_act(st["T"], st["W"], prec=prec, act=sagnn.ACT_RELU, want_z=False, want_act=True)
        return {"needed": st["bufs"][1], "blk_off": p.blk_off, "compact": p.colidx_compact, "packed": st["Hn"], "T": st["T"], "H": out}
    if kind == "infer":
        _, _, out = sagnn.gcn_layer_fwd(rp, ci, va, H, st["W"], prec=prec, ws=st["ws"], want_z=False, want_t=st["want_t"])
        return {"H": out}
    if kind == "train":
        _, Z1, H1 = sagnn.gcn_layer_fwd(rp, ci, va, H, st["W1"], prec=prec, ws=st["ws_in"])
        _, Z2, _ = sagnn.gcn_layer_fwd(rp, ci, va, H1, st["W2"], act=sagnn.ACT_IDENTITY, prec=prec, ws=st["ws_hid"], want_h=False)
        S2, G1, Y2 = sagnn.gcn_layer_bwd(rp, ci, va, st["G"], st["W2"], st["Zp"], H1, prec=prec, ws=st["ws_out"])
        S1, _, Y1 = sagnn.gcn_layer_bwd(rp, ci, va, G1, st["W1"], None, H, prec=prec, ws=st["ws_hid"], want_gprev=False)
        return {"Z1": Z1, "Z2": Z2, "S2": S2, "G1": G1, "Y2": Y2, "S1": S1, "Y1": Y1}
    if kind == "stages":
        return {"Z": sagnn.spmm_stage_loop(st["stages"], st["m"], H, st["T0"], st["T1"], st["Z"])}
    if kind == "directed":
        rpt, cit, vat = sagnn.spmm_csr_transpose(rp, ci, va, st["n"])
        fwd = sagnn.spmm_csr_prepare(rpt, cit, vat, st["n"], H.shape[1])
        bwd = sagnn.spmm_csr_prepare(rp, ci, va, st["n"], H.shape[1])
        Z = sagnn.spmm_csr_tallskinny(rpt, cit, vat, H, ws=fwd)
        S = sagnn.spmm_csr_tallskinny(rp, ci, va, H, ws=bwd)
        return {"rowptr": rpt, "colidx": cit, "val": vat, "Z": Z, "S": S}
    perm, inv, off = sagnn.spmm_perm_from_labels(st["labels"], 16)
    prp, pci, pva = sagnn.spmm_csr_permute_symmetric(rp, ci, va, inv)
    return {"perm": perm, "inv": inv, "off": off, "rowptr": prp, "colidx": pci, "val": pva, "H": sagnn.spmm_pack_rows(H, perm)}


# ---------------------------------------------------------------------------------------------

def _shape(case):
    """Rows, columns, stored entries and needed columns of the case's matrix, as expected from its numbers."""
    n, deg = case["n"], case["deg"]
    if case["graph"] == "rank":
        m = n // 64
        return m, n, m * deg, min(n, int(0.30 * m * deg))     # about three entries a needed column
    if case["graph"] == "sbm_block":
        m = n // 16
        return m, n, m * deg, m + min(n - m, int(m * deg * 0.05))
    return n, n, n * deg, n


def work(case):
    m, n, nnz, need = _shape(case)
    f, kind = case["f"], case["kind"]
    f_out = case.get("f_out", f)

    def spmm(w, rows=m, cols=need, e=nnz):
        return e * 8 + rows * 4 + cols * w * 4 + rows * w * 4, 2 * e * w

    def gemm(k, o):
        return m * (k + o) * 4 + k * o * 4, 2 * m * k * o

    if kind == "step":
        parts = [(nnz * 8 + need * 4, 0), (need * f * 8 + need * 4, 0), spmm(f), gemm(f, f_out)]
    elif kind == "infer":
        b, fl = spmm(f)
        parts = [(b - m * f * 4 + m * f_out * 4 + f * f_out * 4, fl + 2 * m * f * f_out)]
    elif kind == "train":
        h = case["hidden"]
        parts = [spmm(f), gemm(f, h), (m * h * 4, 0), spmm(h), gemm(h, f_out), spmm(f_out), gemm(f_out, h), (m * h * 4, 0),
                 (m * (h + f_out) * 4, 2 * m * h * f_out), spmm(h), (m * (f + h) * 4, 2 * m * f * h)]
    elif kind == "stages":
        s = case["stages"] / case["nb"]
        e, rows = int(nnz * s), int(need * s)
        parts = [(rows * f * 4 + rows * 4 + e * 8 + case["stages"] * m * 4 + m * f * 4, 2 * e * f)]
    elif kind == "directed":
        parts = [(nnz * 16 + n * 8, 0), spmm(f), spmm(f)]
    else:
        parts = [(n * 12, 0), (nnz * 16 + n * 12, 0), (n * f * 8 + n * 4, 0)]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    if case["kind"] == "reorder":
        return "exact"
    # bf16: both operands of the dense transform are rounded (2^-9 each); an operand next to a rounding boundary may
    # fall to the other side.  Otherwise 32-bit sums in any order.
    return {"rel": 5e-3} if case.get("prec") == "bf16" else {"rel": 1e-5}
