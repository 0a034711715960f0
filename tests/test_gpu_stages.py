"""GPU parity of the entry points around the 1.5D stage loop: sparsity-oblivious plan,
column-block split, stage loop (one and two streams) and volume statistics, against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2504_04673_amd as sagnn
from paper_2504_04673_amd import synth
from tests.test_oracle_pins import random_csr
from tests.util import assert_close, dev

pytestmark = pytest.mark.gpu

RTOL_SPMM = 1e-5


def row_block(g, i, P=4):
    off = synth.block_offsets(g.n, P)
    return g.row_block(int(off[i]), int(off[i + 1])), off


def test_oblivious_plan_cfg1(cfg1):
    g, H = cfg1
    blk, off = row_block(g, 1)
    rp, ci, v = dev(blk.rowptr), dev(blk.colidx), dev(blk.val)
    plan = sagnn.spmm_plan_needed_rows(rp, ci, g.n, off, oblivious=True, validate=True)
    needed, blk_off, compact = oracle.needed_rows_oblivious(blk.colidx, g.n, off)
    assert np.array_equal(plan.blk_off, blk_off)
    assert np.array_equal(plan.needed.cpu().numpy(), needed)
    assert np.array_equal(plan.colidx_compact.cpu().numpy(), compact)
    # the oblivious path moves every row and computes the same product
    Hd = dev(H)
    T = sagnn.spmm_pack_rows(Hd, plan.needed)
    assert T.cpu().numpy().tobytes() == H.tobytes()
    Z = sagnn.spmm_csr_tallskinny(rp, plan.colidx_compact, v, T)
    ref, zabs = oracle.spmm(blk.rowptr, blk.colidx, blk.val, H, want_abs=True)
    assert_close(Z, ref, zabs, RTOL_SPMM, "oblivious Z")


def check_split(rowptr, colidx, val, bounds):
    got = sagnn.spmm_split_colblocks(dev(rowptr), dev(colidx), dev(val), bounds)
    torch.cuda.synchronize()
    exp = oracle.split_colblocks(rowptr, colidx, val, bounds)
    off = np.concatenate([[0], np.cumsum([b[1].size for b in exp])])
    assert np.array_equal(got.nnz_off, off)
    for q, (rp, ci, va) in enumerate(exp):
        grp, gci, gva = got.block(q)
        assert np.array_equal(grp.cpu().numpy(), rp), q
        assert np.array_equal(gci.cpu().numpy(), ci), q
        assert gva.cpu().numpy().tobytes() == va.tobytes(), q
    return got


@pytest.mark.parametrize("case", ["cfg1_global", "cfg1_compact", "unsorted_dup_ragged", "many_blocks",
                                  "hub_row", "empty"])
def test_split_colblocks(case, cfg1):
    g, _ = cfg1
    rng = np.random.default_rng(3)
    if case == "cfg1_global":
        check_split(g.rowptr, g.colidx, g.val, synth.block_offsets(g.n, 4))
    elif case == "cfg1_compact":
        blk, off = row_block(g, 2)
        needed, blk_off, compact = oracle.needed_rows(blk.rowptr, blk.colidx, g.n, off)
        check_split(blk.rowptr, compact, blk.val, blk_off)
    elif case == "unsorted_dup_ragged":
        rowptr, colidx, val = random_csr(300, 500, 0.1, rng, sort=False, dup=True)
        check_split(rowptr, colidx, val, [7, 7, 100, 101, 333, 480])      # drops both ends
    elif case == "many_blocks":
        rowptr, colidx, val = random_csr(257, 4000, 0.05, rng, sort=False)
        check_split(rowptr, colidx, val, np.linspace(0, 4000, 201).astype(np.int64))   # 200 blocks
    elif case == "hub_row":
        # one row of 5000 entries spanning several 64-entry steps per block, then short rows
        hub = np.sort(rng.choice(20000, size=5000, replace=False))
        rows = [hub] + [np.sort(rng.choice(20000, size=3, replace=False)) for _ in range(40)]
        rowptr = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int32)
        colidx = np.concatenate(rows).astype(np.int32)
        val = rng.standard_normal(colidx.size).astype(np.float32)
        check_split(rowptr, colidx, val, [0, 5000, 10000, 15000, 20000])
    else:
        z = np.zeros(0, dtype=np.int32)
        got = sagnn.spmm_split_colblocks(dev(np.zeros(6, np.int32)), dev(z), dev(z.astype(np.float32)),
                                         [0, 10, 20])
        assert got.nnz_off.tolist() == [0, 0, 0] and int(got.rowptr_blk.abs().sum()) == 0


def stage_inputs(blk, n, colblk, H, stages, prepare):
    rp, ci, v = dev(blk.rowptr), dev(blk.colidx), dev(blk.val)
    plan = sagnn.spmm_plan_needed_rows(rp, ci, n, colblk)
    cb = sagnn.spmm_split_colblocks(rp, plan.colidx_compact, v, plan.blk_off)
    needed, off, compact = oracle.needed_rows(blk.rowptr, blk.colidx, n, colblk)
    assert np.array_equal(plan.blk_off, off)
    oblocks = oracle.split_colblocks(blk.rowptr, compact, blk.val, off)
    glist, olist, orows = [], [], []
    for q in stages:
        brp, bci, bva = cb.block(q)
        rows = plan.needed[int(off[q]):int(off[q + 1])]
        st = {"rowptr": brp, "colidx": bci, "val": bva, "rows": rows}
        if prepare and bci.numel():
            st["ws"] = sagnn.spmm_csr_prepare(brp, bci, bva, rows.numel(), H.shape[1])
        glist.append(st)
        olist.append(oblocks[q])
        orows.append(needed[off[q]:off[q + 1]])
    cap = max(int(np.diff(off).max()), 1)
    return glist, olist, orows, cap


@pytest.mark.parametrize("two_streams", [False, True])
@pytest.mark.parametrize("stages,prepare", [([0, 1, 2, 3], False), ([1, 3], True), ([2], False), ([], False)])
def test_stage_loop_cfg1(cfg1, stages, prepare, two_streams):
    """Row block 0 of configuration 1 (P = 4): partial sums over a rank's stages (Alg. 2)."""
    g, H = cfg1
    blk, off = row_block(g, 0)
    f = H.shape[1]
    glist, olist, orows, cap = stage_inputs(blk, g.n, off, H, stages, prepare)
    Hd = dev(H)
    T0 = torch.empty((cap, f), dtype=torch.float32, device="cuda")
    T1 = torch.empty((cap, f), dtype=torch.float32, device="cuda")
    Z = torch.full((blk.m, f), 7.0, dtype=torch.float32, device="cuda")
    side = torch.cuda.Stream() if two_streams else None
    sagnn.spmm_stage_loop(glist, blk.m, Hd, T0, T1, Z, accumulate_first=False, pack_stream=side)
    torch.cuda.synchronize()
    if not stages:
        assert float(Z.min()) == 7.0 and float(Z.max()) == 7.0      # nothing to do: Z untouched
        return
    ref, zabs = oracle.stage_loop(olist, orows, H, blk.m, want_abs=True)
    assert_close(Z, ref, zabs, RTOL_SPMM, f"stage loop {stages}")
    # accumulate_first = 1 adds to what Z holds
    Z2 = torch.full((blk.m, f), 0.5, dtype=torch.float32, device="cuda")
    sagnn.spmm_stage_loop(glist, blk.m, Hd, T0, T1, Z2, accumulate_first=True, pack_stream=side)
    torch.cuda.synchronize()
    assert_close(Z2, ref.astype(np.float64) + 0.5, zabs + 0.5, RTOL_SPMM, "stage loop accumulate")


def test_stage_loop_with_empty_block_and_capacity_error():
    rng = np.random.default_rng(8)
    m, n, f = 200, 1000, 64
    rowptr, colidx, val = random_csr(m, n, 0.02, rng)
    colidx = np.where((colidx >= 250) & (colidx < 500), colidx + 250, colidx).astype(np.int32)  # block 1 empty
    order = np.argsort(np.repeat(np.arange(m), np.diff(rowptr)) * n + colidx, kind="stable")
    colidx, val = colidx[order], val[order]
    H = rng.standard_normal((n, f)).astype(np.float32)

    class B:  # minimal stand-in for a CSR block
        pass
    blk = B()
    blk.rowptr, blk.colidx, blk.val, blk.m = rowptr, colidx, val, m
    colblk = np.array([0, 250, 500, 750, 1000], dtype=np.int64)
    glist, olist, orows, cap = stage_inputs(blk, n, colblk, H, [0, 1, 2, 3], False)
    assert orows[1].size == 0
    Hd = dev(H)
    T0 = torch.empty((cap, f), dtype=torch.float32, device="cuda")
    T1 = torch.empty((cap, f), dtype=torch.float32, device="cuda")
    Z = torch.empty((m, f), dtype=torch.float32, device="cuda")
    sagnn.spmm_stage_loop(glist, m, Hd, T0, T1, Z, pack_stream=torch.cuda.Stream())
    torch.cuda.synchronize()
    ref, zabs = oracle.stage_loop(olist, orows, H, m, want_abs=True)
    assert_close(Z, ref, zabs, RTOL_SPMM, "stage loop with an empty block")
    with pytest.raises(sagnn.SagnnError) as e:
        sagnn.spmm_stage_loop(glist, m, Hd, T0[:1], T1[:1], Z)
    assert e.value.code == -2


@pytest.mark.parametrize("f", [4, 100, 128, 256])
@pytest.mark.parametrize("sizes", [[33], [32, 31], [1, 0], [0, 1], [0, 0, 65], [64, 7, 32], [5, 1000, 0, 40, 9]])
def test_stage_loop_packs_two_stages_at_a_time(sizes, f):
    """On one stream the rows of an even stage and of the next are packed in one launch: odd numbers of stages, empty lists
    on either side, lists that end inside a workgroup's rows.  Same bits as on two streams, where each has its own, and the
    two buffers hold the last two stages' rows."""
    gen = torch.Generator().manual_seed(f + len(sizes))
    m, n, cap = 300, 1200, max(max(sizes), 1)
    H = torch.randn(n, f, generator=gen).cuda()
    stages = []
    for N in sizes:
        deg = torch.randint(0, 6, (m,), generator=gen) * (N > 0)
        rp = torch.zeros(m + 1, dtype=torch.int32)
        rp[1:] = torch.cumsum(deg, 0)
        nnz = int(rp[-1])
        stages.append({"rowptr": rp.cuda(), "colidx": torch.randint(max(N, 1), (nnz,), generator=gen).to(torch.int32).cuda(),
                       "val": torch.randn(nnz, generator=gen).cuda(),
                       "rows": torch.randperm(n, generator=gen)[:N].sort()[0].to(torch.int32).cuda()})
    out = []
    for side in (None, torch.cuda.Stream()):
        T = [torch.full((cap, f), 3.0, device="cuda") for _ in range(2)]
        Z = torch.full((m, f), 7.0, device="cuda")
        sagnn.spmm_stage_loop(stages, m, H, T[0], T[1], Z, pack_stream=side)
        torch.cuda.synchronize()
        out.append(Z)
        for k in range(max(len(sizes) - 2, 0), len(sizes)):
            assert torch.equal(T[k & 1][:sizes[k]], H[stages[k]["rows"].long()])
    assert torch.equal(out[0], out[1])
    want = torch.zeros(m, f, dtype=torch.float64, device="cuda")
    for st, N in zip(stages, sizes):
        row = torch.repeat_interleave(torch.arange(m, device="cuda"), torch.diff(st["rowptr"]).long())
        want.index_add_(0, row, st["val"][:, None].double() * H[st["rows"].long()][st["colidx"].long()].double())
    # at most 25 terms a row: 32 2^-24 of sums of at most 25 products of two normal numbers
    assert float((out[0].double() - want).abs().max()) <= 32 * 2.0**-24 * 25 * 36


def test_volume_stats_cfg1_all_row_blocks(cfg1):
    """Counts |NnzCols(i,q)| of all P = 4 row blocks from the GPU plan; statistics from the
    library against the oracle's, sparsity-aware and sparsity-oblivious."""
    g, _ = cfg1
    P = 4
    counts = np.zeros((P, P), dtype=np.int64)
    ocounts = np.zeros((P, P), dtype=np.int64)
    for i in range(P):
        blk, off = row_block(g, i)
        plan = sagnn.spmm_plan_needed_rows(dev(blk.rowptr), dev(blk.colidx), g.n, off, want_compact=False)
        counts[i] = np.diff(plan.blk_off)
        ocounts[i] = np.diff(oracle.needed_rows(blk.rowptr, blk.colidx, g.n, off, want_compact=False)[1])
    assert np.array_equal(counts, ocounts)
    for c in (counts, np.tile(np.diff(off), (P, 1))):
        got = sagnn.spmm_volume_stats(c, 16)
        exp = oracle.volume_stats(c, 16)
        for k, v in exp.items():
            assert got[k] == pytest.approx(v, rel=1e-12), k
    aware, obl = sagnn.spmm_volume_stats(counts, 16), sagnn.spmm_volume_stats(np.tile(np.diff(off), (P, 1)), 16)
    assert aware["total_bytes"] < obl["total_bytes"] and aware["cut_rows"] <= 1024


def check_transpose(rowptr, colidx, val, n):
    rpt, cit, vat = sagnn.spmm_csr_transpose(dev(rowptr), dev(colidx), dev(val), n)
    torch.cuda.synchronize()
    erp, eci, eva = oracle.transpose_csr(rowptr, colidx, val, n)
    assert np.array_equal(rpt.cpu().numpy(), erp)
    assert np.array_equal(cit.cpu().numpy(), eci)
    assert vat.cpu().numpy().tobytes() == eva.tobytes()
    return rpt, cit, vat


@pytest.mark.parametrize("case", ["cfg1", "rect_unsorted_dup", "hub_and_empty", "three_passes", "four_passes",
                                  "one_column", "empty"])
def test_csr_transpose(case, cfg1):
    g, _ = cfg1
    rng = np.random.default_rng(12)
    if case == "cfg1":
        rpt, cit, vat = check_transpose(g.rowptr, g.colidx, g.val, g.n)
        # the normalised adjacency matrix is symmetric: its transpose is itself
        assert np.array_equal(rpt.cpu().numpy(), g.rowptr) and np.array_equal(cit.cpu().numpy(), g.colidx)
    elif case == "rect_unsorted_dup":
        rowptr, colidx, val = random_csr(700, 300, 0.05, rng, sort=False, dup=True)
        check_transpose(rowptr, colidx, val, 300)
    elif case == "hub_and_empty":
        hub = np.sort(rng.choice(60000, size=9000, replace=False))
        rows = [np.empty(0, np.int64), hub, np.empty(0, np.int64)] + \
               [np.sort(rng.choice(60000, size=5, replace=False)) for _ in range(3000)]
        rowptr = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int32)
        colidx = np.concatenate(rows).astype(np.int32)
        val = rng.standard_normal(colidx.size).astype(np.float32)
        check_transpose(rowptr, colidx, val, 60000)
    elif case in ("three_passes", "four_passes"):
        n = 5_000_000 if case == "three_passes" else 20_000_000        # 23 and 25 column bits
        nnz = 300_000
        cols = rng.integers(0, n, size=nnz)
        cols[:3] = [0, n - 1, n - 1]
        cuts = np.sort(rng.integers(0, nnz + 1, size=999))
        rowptr = np.array([0, *cuts, nnz], dtype=np.int32)
        check_transpose(rowptr, cols.astype(np.int32), rng.standard_normal(nnz).astype(np.float32), n)
    elif case == "one_column":
        rowptr = np.arange(0, 5001, dtype=np.int32)
        check_transpose(rowptr, np.zeros(5000, np.int32), rng.standard_normal(5000).astype(np.float32), 1)
    else:
        z = np.zeros(0, dtype=np.int32)
        rpt, cit, vat = sagnn.spmm_csr_transpose(dev(np.zeros(8, np.int32)), dev(z), dev(z.astype(np.float32)), 11)
        assert rpt.cpu().numpy().tolist() == [0] * 12
        bad = np.array([0, 5, 11], dtype=np.int32)           # column 11 is outside [0, 11)
        with pytest.raises(sagnn.SagnnError) as e:
            sagnn.spmm_csr_transpose(dev(np.array([0, 3], np.int32)), dev(bad), dev(np.ones(3, np.float32)), 11)
        assert e.value.code == -3


@pytest.mark.parametrize("nnz,m,n", [(1, 1, 1), (1024, 5, 256), (1025, 3000, 257), (262_144, 1000, 1 << 16),
                                     (262_145, 700_000, 1000), (4_194_305, 40_000, 70_001)])
def test_csr_transpose_at_the_edges_of_the_sort_tiles(nnz, m, n):
    """Full and one-over tiles of every tile size, one to three digit passes, and a matrix whose tiles are covered
    by more rows than a tile has entries."""
    rng = np.random.default_rng(nnz)
    rowptr = np.array([0, *np.sort(rng.integers(0, nnz + 1, size=m - 1)), nnz], dtype=np.int32)
    colidx = rng.integers(0, n, size=nnz).astype(np.int32)
    check_transpose(rowptr, colidx, rng.standard_normal(nnz).astype(np.float32), n)


@pytest.mark.parametrize("nnz", [1024 + 63, 131_072, 131_073, 262_145, 4_194_305 + 8191])
def test_csr_transpose_rows_that_begin_at_the_edges_of_tiles(nnz):
    """Rows that begin at, just before and just behind tiles, wavefronts' shares of them and runs of 64 entries, each
    after up to two empty ones, runs of empty rows at both ends, and a row that covers a whole tile.  (Tiles with and
    without a scan of their counts: 128 tiles, one more.)"""
    rng = np.random.default_rng(nnz)
    starts = np.arange(0, min(nnz, 200_000), 64)
    starts = np.concatenate([starts, starts[1:] - 1, starts + 1, np.arange(0, nnz, 8192) + rng.integers(-2, 3)])
    starts = starts[(starts > 0) & (starts < nnz) & ((starts < 20_000) | (starts > 40_000))]
    starts = np.sort(np.repeat(starts, rng.integers(1, 4, size=starts.size)))
    rowptr = np.concatenate([np.zeros(70, np.int64), starts, np.full(70, nnz)]).astype(np.int32)
    n = 3000
    colidx = rng.integers(0, n, size=nnz).astype(np.int32)
    check_transpose(rowptr, colidx, rng.standard_normal(nnz).astype(np.float32), n)


def test_directed_graph_layer_uses_both_orientations():
    """Directed graph: the forward product runs on A^T (Sec. 2.1 forward equation), the backward
    product on A.  A^T comes from the device transpose; both layer calls against the oracle."""
    rng = np.random.default_rng(21)
    n, f_in, f_out = 900, 64, 32
    rowptr, colidx, val = random_csr(n, n, 0.02, rng, sort=True)
    H = rng.standard_normal((n, f_in)).astype(np.float32)
    W = (rng.standard_normal((f_in, f_out)) / 8).astype(np.float32)
    G = rng.standard_normal((n, f_out)).astype(np.float32)
    rp, ci, va = dev(rowptr), dev(colidx), dev(val)
    rpt, cit, vat = sagnn.spmm_csr_transpose(rp, ci, va, n)
    T, Z, Ho = sagnn.gcn_layer_fwd(rpt, cit, vat, dev(H), dev(W), act=sagnn.ACT_RELU)
    ot = oracle.transpose_csr(rowptr, colidx, val, n)
    of = oracle.gcn_layer_fwd(ot[0], ot[1], ot[2], H, W, act=1)
    assert_close(T, of["T"], of["Tabs"], RTOL_SPMM, "directed T")
    assert_close(Z, of["Z"], of["Zabs"], 1e-5, "directed Z")
    assert_close(Ho, of["H"], of["Zabs"], 1e-5, "directed H'")
    Zprev = rng.standard_normal((n, f_in)).astype(np.float32)     # stand-in for Z^{l-1} (mask source)
    S, Gp, Y = sagnn.gcn_layer_bwd(rp, ci, va, dev(G), dev(W), dev(Zprev), dev(H))
    ob = oracle.gcn_layer_bwd(rowptr, colidx, val, G, W, Zprev, H)
    assert_close(S, ob["S"], ob["Sabs"], RTOL_SPMM, "directed S")
    assert_close(Gp, ob["Gprev"], ob["Gabs"], 1e-5, "directed Gprev")
    assert_close(Y, ob["Y"], ob["Yabs"], 1e-5, "directed Y")


# ------------------------------------------------------------------------------------ reordering

@pytest.mark.parametrize("degrees", [[0, 1, 63, 64], [65, 128, 129, 3], [256, 257, 512, 0], [513, 2, 40, 0], [700, 700, 1, 0]])
def test_permute_symmetric_at_the_row_lengths_where_the_method_changes(degrees):
    """Rows around one, two, four and eight columns a lane, and past the longest row that is permuted by itself;
    unsorted columns with repeats."""
    rng = np.random.default_rng(sum(degrees))
    n = 1001
    deg = np.array(degrees)[rng.integers(0, len(degrees), size=n)]
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    colidx = rng.integers(0, n, size=rowptr[-1]).astype(np.int32)
    val = rng.standard_normal(colidx.size).astype(np.float32)
    inv = rng.permutation(n).astype(np.int32)
    rpp, cip, vap = sagnn.spmm_csr_permute_symmetric(dev(rowptr), dev(colidx), dev(val), dev(inv))
    orp, oci, ova = oracle.permute_symmetric(rowptr, colidx, val, inv)
    assert np.array_equal(rpp.cpu().numpy(), orp) and np.array_equal(cip.cpu().numpy(), oci)
    assert vap.cpu().numpy().tobytes() == ova.tobytes()


@pytest.mark.parametrize("case", ["cfg1_random_labels", "sbm_communities", "unsorted_dup", "one_part", "tiny"])
def test_reorder_by_labels_and_permute_symmetric(case, cfg1):
    """Renumbering by partition labels and the symmetric permutation of A (Sec. 5 / 6.1), bit for
    bit against the oracle; then the product in the new numbering, moved back with the inverse
    row gather, against the oracle's product in the old numbering."""
    rng = np.random.default_rng(len(case))
    if case == "cfg1_random_labels":
        g, _ = cfg1
        rowptr, colidx, val, n, parts = g.rowptr, g.colidx, g.val, g.n, 4
        labels = rng.integers(0, parts, size=n).astype(np.int32)
    elif case == "sbm_communities":
        g = synth.sbm_graph(8000, 16, 20, 2, 5, order="random")
        rowptr, colidx, val, n, parts = g.rowptr, g.colidx, g.val, g.n, 16
        labels = synth.sbm_labels(g)
    elif case == "unsorted_dup":
        n, parts = 3001, 7
        rowptr, colidx, val = random_csr(n, n, 0.004, rng, sort=False, dup=True)
        labels = rng.integers(0, parts, size=n).astype(np.int32)
        labels[labels == 3] = 4                       # an empty part
    elif case == "one_part":
        n, parts = 513, 1
        rowptr, colidx, val = random_csr(n, n, 0.02, rng)
        labels = np.zeros(n, np.int32)
    else:
        n, parts = 1, 1
        rowptr, colidx, val = np.array([0, 1], np.int32), np.array([0], np.int32), np.array([2.0], np.float32)
        labels = np.zeros(1, np.int32)
    perm, inv, off = sagnn.spmm_perm_from_labels(dev(labels), parts)
    operm, oinv, ooff = oracle.perm_from_labels(labels, parts)
    assert np.array_equal(perm.cpu().numpy(), operm) and np.array_equal(inv.cpu().numpy(), oinv)
    assert np.array_equal(off, ooff)
    rp, ci, v = dev(rowptr), dev(colidx), dev(val)
    rpp, cip, vap = sagnn.spmm_csr_permute_symmetric(rp, ci, v, inv)
    torch.cuda.synchronize()
    orp, oci, ova = oracle.permute_symmetric(rowptr, colidx, val, oinv)
    assert np.array_equal(rpp.cpu().numpy(), orp)
    assert np.array_equal(cip.cpu().numpy(), oci)
    assert vap.cpu().numpy().tobytes() == ova.tobytes()
    # product in the new numbering, moved back: Z_old = pack(Z_new, inv), H_new = pack(H, perm)
    f = 32
    H = synth.normal((n, f), 3, synth.STREAM_H)
    Hn = sagnn.spmm_pack_rows(dev(H), perm)
    Zn = sagnn.spmm_csr_tallskinny(rpp, cip, vap, Hn)
    Z = sagnn.spmm_pack_rows(Zn, inv)
    torch.cuda.synchronize()
    ref, zabs = oracle.spmm(rowptr, colidx, val, H, want_abs=True)
    assert_close(Z, ref, zabs, RTOL_SPMM, f"reordered product {case}")


@pytest.mark.parametrize("n,parts", [(1, 1), (3, 3), (255, 255), (1024, 256), (1025, 257), (2049, 1024), (131_072, 256), (131_073, 2),
                                     (262_145, 16), (2_100_000, 200)])
def test_order_from_labels_at_the_edges_of_its_tiles(n, parts):
    """One pass for up to 256 parts, sorted pairs beyond; few tiles that add up the counts by themselves, and many; the row
    pointer of the permuted matrix with its tile sums added up by every workgroup (up to 1024 tiles of 2048 rows) or scanned."""
    rng = np.random.default_rng(n)
    labels = np.minimum(rng.integers(0, parts, size=n), rng.integers(0, parts, size=n)).astype(np.int32)
    perm, inv, off = sagnn.spmm_perm_from_labels(dev(labels), parts)
    operm, oinv, ooff = oracle.perm_from_labels(labels, parts)
    assert np.array_equal(perm.cpu().numpy(), operm) and np.array_equal(inv.cpu().numpy(), oinv) and np.array_equal(off, ooff)
    deg = rng.integers(0, 3, size=n)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    colidx = rng.integers(0, n, size=int(rowptr[-1])).astype(np.int32)
    rpp, _, _ = sagnn.spmm_csr_permute_symmetric(dev(rowptr), dev(colidx), dev(np.ones(colidx.size, np.float32)), inv)
    assert np.array_equal(rpp.cpu().numpy(), np.concatenate([[0], np.cumsum(deg[operm])]).astype(np.int32))
    labels[n // 2] = parts
    with pytest.raises(sagnn.SagnnError):
        sagnn.spmm_perm_from_labels(dev(labels), parts)


@pytest.mark.parametrize("over", ["perm", "inv", "both_ends"])
@pytest.mark.parametrize("n,parts", [(5000, 16), (300_001, 3), (4_300_001, 256), (70_000, 300)])
def test_order_from_labels_in_the_labels_own_buffer(n, parts, over):
    """An order written over the labels that it is made from, whole or in part, by the C entry point: one pass writes its tiles
    while others still read theirs."""
    labels = np.random.default_rng(n).integers(0, parts, size=n).astype(np.int32)
    operm, oinv, ooff = oracle.perm_from_labels(labels, parts)
    nbytes = ctypes.c_size_t(0)
    assert sagnn.lib().spmm_permute_workspace_bytes(n, n, ctypes.byref(nbytes)) == 0
    ws = torch.empty(nbytes.value, dtype=torch.uint8, device="cuda")
    room = torch.zeros(3 * n, dtype=torch.int32, device="cuda")       # the labels lie in the middle
    room[n:2 * n] = dev(labels)
    place = {"perm": (n, 2 * n), "inv": (0, n), "both_ends": (1, 2 * n - 1)}[over]
    perm, inv = (room[p:p + n] for p in place)
    off = np.zeros(parts + 1, np.int64)
    rc = sagnn.lib().spmm_perm_from_labels(room[n:].data_ptr(), n, parts, perm.data_ptr(), inv.data_ptr(), off.ctypes.data,
                                           ws.data_ptr(), nbytes.value, torch.cuda.current_stream().cuda_stream)
    assert rc == 0 and np.array_equal(off, ooff)
    assert np.array_equal(perm.cpu().numpy(), operm) and np.array_equal(inv.cpu().numpy(), oinv)


def test_reorder_rejects_bad_labels_and_maps():
    labels = dev(np.array([0, 1, 2, 5, 1], np.int32))
    with pytest.raises(sagnn.SagnnError) as ei:
        sagnn.spmm_perm_from_labels(labels, 3)
    assert ei.value.code == -3
    rowptr, colidx, val = random_csr(6, 6, 0.5, np.random.default_rng(0))
    for bad in ([0, 1, 2, 3, 4, 4], [0, 1, 2, 3, 4, 6], [0, 1, 2, 3, 4, -1]):
        with pytest.raises(sagnn.SagnnError) as ei:
            sagnn.spmm_csr_permute_symmetric(dev(rowptr), dev(colidx), dev(val), dev(np.array(bad, np.int32)))
        assert ei.value.code == -3
    ok = dev(np.array([5, 4, 3, 2, 1, 0], np.int32))
    badcol = colidx.copy()
    badcol[0] = 6
    with pytest.raises(sagnn.SagnnError) as ei:
        sagnn.spmm_csr_permute_symmetric(dev(rowptr), dev(badcol), dev(val), ok)
    assert ei.value.code == -3
    sagnn.spmm_csr_permute_symmetric(dev(rowptr), dev(colidx), dev(val), ok)


@pytest.mark.parametrize("nnz", [1, 300])
def test_permute_symmetric_refuses_entries_without_rows(nnz):
    """A matrix of no rows and columns holds no entries: every column id is out of range."""
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    for last in (0, nnz):
        with pytest.raises(sagnn.SagnnError) as ei:
            sagnn.spmm_csr_permute_symmetric(dev(np.array([last], np.int32)), dev(np.zeros(nnz, np.int32)),
                                             dev(np.ones(nnz, np.float32)), none)
        assert ei.value.code == -3
    rpp, cip, _ = sagnn.spmm_csr_permute_symmetric(dev(np.zeros(1, np.int32)), none, none.float(), none)
    assert rpp.cpu().tolist() == [0] and cip.numel() == 0
