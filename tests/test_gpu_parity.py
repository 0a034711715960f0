"""GPU parity: every step of the hot path, called through the C ABI, element by element against
the CPU oracle on the same seeded inputs.  Integer results bit-exact; fp32 SpMM within
1e-5 * sum|terms|; bf16 GEMM within 1e-2 * sum|terms|."""
import ctypes
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2504_04673_amd as sagnn
from paper_2504_04673_amd import synth
from tests.util import assert_close, csr_dev, dev

pytestmark = pytest.mark.gpu

RTOL_SPMM = 1e-5
RTOL_GEMM_FP32 = 1e-5
RTOL_BF16 = 1e-2


def random_csr(m, n, avg, rng, empty_frac=0.0, hubs=(), dup=False):
    deg = rng.poisson(avg, size=m)
    if empty_frac:
        deg[rng.random(m) < empty_frac] = 0
    for r, d in hubs:
        deg[r] = d
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    nnz = int(rowptr[-1])
    colidx = rng.integers(0, n, size=nnz).astype(np.int32)
    if not dup:
        # sort inside rows (duplicates may remain; both sides sum them)
        for r in range(m):
            colidx[rowptr[r]:rowptr[r + 1]].sort()
    val = rng.standard_normal(nnz).astype(np.float32)
    return rowptr, colidx, val


# ------------------------------------------------------------------------------------ pack

@pytest.mark.parametrize("n,f,N,ld", [(4096, 16, 3700, 16), (1000, 4, 1, 4), (1000, 20, 333, 24),
                                      (5000, 128, 4097, 128), (3000, 256, 1025, 260), (2000, 300, 777, 300),
                                      (10, 64, 0, 64)])
def test_pack_rows(n, f, N, ld):
    rng = np.random.default_rng(n + f)
    Hfull = synth.normal((n, ld), 1, synth.STREAM_H)
    rows = np.sort(rng.choice(n, size=N, replace=False)).astype(np.int32)
    Hd = dev(Hfull)[:, :f]          # strided view: leading dimension ld
    got = torch.empty((N, f), device="cuda")
    L = sagnn.lib()
    import ctypes
    rc = L.spmm_pack_rows(ctypes.c_void_p(Hd.data_ptr()), n, ld, f, ctypes.c_void_p(dev(rows).data_ptr()) if N else None,
                          N, ctypes.c_void_p(got.data_ptr()) if N else None, f,
                          ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    torch.cuda.synchronize()
    ref = oracle.pack_rows(np.ascontiguousarray(Hfull[:, :f]), rows)
    assert got.cpu().numpy().tobytes() == ref.tobytes()


def test_pack_rows_out_of_range_ids_give_zero_rows():
    H = dev(synth.normal((100, 32), 2, synth.STREAM_H))
    rows = dev(np.array([5, -1, 100, 99, 2 ** 31 - 1], np.int32))
    out = sagnn.spmm_pack_rows(H, rows).cpu().numpy()
    Hh = H.cpu().numpy()
    assert np.array_equal(out[0], Hh[5]) and np.array_equal(out[3], Hh[99])
    assert not out[1].any() and not out[2].any() and not out[4].any()


def test_pack_rows_offsets_beyond_4gib():
    """H larger than 2^32 bytes: element offsets must be 64-bit."""
    n, f = 9_000_000, 128                       # 4.6 GB
    H = torch.empty((n, f), device="cuda")
    rows_h = np.array([0, 1, 4_194_304, 8_388_607, 8_388_608, 8_999_999], np.int32)
    vals = synth.normal_rows(rows_h, f, 3, synth.STREAM_H)
    H[torch.from_numpy(rows_h.astype(np.int64)).cuda()] = dev(vals)
    out = sagnn.spmm_pack_rows(H, dev(rows_h)).cpu().numpy()
    assert out.tobytes() == vals.tobytes()
    del H


# ------------------------------------------------------------------------------------ plan

def small_block(m, n, nnz, nb):
    """the shapes the library plans with one workgroup in one launch"""
    return n <= 262144 and m <= 262144 and nnz <= 65536 and nb <= 16


def check_plan(rowptr, colidx, n, colblk):
    """Against the oracle; small blocks through both the one-launch and the general path."""
    needed, blk_off, compact = oracle.needed_rows(rowptr, colidx, n, colblk)
    modes = (False, True) if small_block(rowptr.size - 1, n, colidx.size, len(colblk) - 1) else (False,)
    for multipass in modes:
        plan = sagnn.spmm_plan_needed_rows(dev(rowptr), dev(colidx), n, colblk, multipass=multipass)
        torch.cuda.synchronize()
        assert np.array_equal(plan.blk_off, blk_off), multipass
        assert np.array_equal(plan.needed.cpu().numpy(), needed), multipass
        if colidx.size:
            assert np.array_equal(plan.colidx_compact.cpu().numpy(), compact), multipass
    return plan


@pytest.mark.parametrize("m,n,nnz,nb,seed", [(4096, 262_144, 65_536, 16, 0), (262_144, 262_144, 65_536, 1, 1),
                                             (4096, 262_145, 65_536, 16, 2), (4096, 262_144, 65_537, 16, 3),
                                             (4096, 262_144, 65_536, 17, 4), (300, 129, 5000, 7, 5),
                                             (10, 64, 64, 2, 6), (7, 1, 40, 1, 7), (2000, 200_000, 3, 16, 8)])
def test_plan_small_blocks_one_launch_and_its_limits(m, n, nnz, nb, seed):
    """Shapes at and just beyond the limits of the one-launch path (columns, entries, blocks), tiny
    and nearly empty ones; unsorted columns with duplicates, columns on both sides of every 64-column
    word edge in use and of the last column, block boundaries that coincide and that cut inside a word.
    Capacity: exactly N succeeds; N - 1 is refused with the required size reported and nothing written."""
    rng = np.random.default_rng(seed)
    cols = rng.integers(0, n, size=nnz)
    edge = [0, n - 1, 63, 64, 65, 127, 128, n // 2, (n - 1) // 64 * 64, max((n - 1) // 64 * 64 - 1, 0)]
    k = min(len(edge), nnz)
    cols[:k] = [min(max(c, 0), n - 1) for c in edge[:k]]
    if nnz > 200:
        cols[100:200] = cols[0]                                   # a run of duplicates
    cuts = np.sort(rng.integers(0, nnz + 1, size=m - 1))
    rowptr = np.array([0, *cuts, nnz], dtype=np.int32)
    colidx = cols.astype(np.int32)
    bc = np.sort(rng.integers(0, n + 1, size=nb - 1))
    if nb > 3:
        bc[1] = bc[0]                                             # an empty block
    colblk = np.array([0, *bc, n], dtype=np.int64)
    plan = check_plan(rowptr, colidx, n, colblk)
    N = plan.N
    for multipass in ((False, True) if small_block(m, n, nnz, nb) else (False,)):
        exact = sagnn.spmm_plan_needed_rows(dev(rowptr), dev(colidx), n, colblk, needed_cap=N, multipass=multipass)
        assert exact.N == N and torch.equal(exact.needed, plan.needed)
        if N > 0:
            ws, needed, compact = sagnn.plan_buffers(m, n, nnz, nb, torch.device("cuda"), N - 1, True)
            needed.fill_(-7)
            compact.fill_(-7)
            with pytest.raises(sagnn.SagnnError) as ei:
                sagnn.spmm_plan_needed_rows(dev(rowptr), dev(colidx), n, colblk, needed_cap=N - 1,
                                            bufs=(ws, needed, compact), multipass=multipass)
            assert ei.value.code == -2
            torch.cuda.synchronize()
            assert bool((needed == -7).all()) and bool((compact == -7).all())
        # validation: a negative column, a column equal to n, a row pointer that steps back
        for bad_at, bad_val in ((0, -1), (nnz - 1, n)):
            badc = colidx.copy()
            badc[bad_at] = bad_val
            with pytest.raises(sagnn.SagnnError) as ei:
                sagnn.spmm_plan_needed_rows(dev(rowptr), dev(badc), n, colblk, validate=True, multipass=multipass)
            assert ei.value.code == -3
            lax = sagnn.spmm_plan_needed_rows(dev(rowptr), dev(badc), n, colblk, multipass=multipass)
            assert int(lax.colidx_compact[bad_at]) == -1            # not validated: skipped and flagged
        if m >= 3 and rowptr[1] < nnz:
            badrp = rowptr.copy()
            badrp[1] = badrp[2] + 1
            with pytest.raises(sagnn.SagnnError) as ei:
                sagnn.spmm_plan_needed_rows(dev(badrp), dev(colidx), n, colblk, validate=True, multipass=multipass)
            assert ei.value.code == -3
        sagnn.spmm_plan_needed_rows(dev(rowptr), dev(colidx), n, colblk, validate=True, multipass=multipass)


@pytest.mark.parametrize("n,nnz,nb", [(131_072, 50_000, 3), (131_073, 50_000, 3), (300_000, 70_000, 64),
                                      (300_000, 70_000, 65), (90_000, 800_000, 2044), (90_000, 70_000, 2045)])
def test_plan_at_the_edges_of_its_flags_and_block_lists(n, nnz, nb):
    """Columns that just fit one LDS byte each and one more; block boundaries that travel as kernel
    arguments, through a copy, and more of them than the host record holds.  A column outside [0, n) and too
    small a capacity leave the outputs alone."""
    rng = np.random.default_rng(n + nb)
    m = 700
    cols = rng.integers(0, n, size=nnz).astype(np.int32)
    cols[:4] = [0, n - 1, n // 2, max(n - 64, 0)]
    rowptr = np.array([0, *np.sort(rng.integers(0, nnz + 1, size=m - 1)), nnz], dtype=np.int32)
    colblk = np.array([0, *np.sort(rng.integers(0, n + 1, size=nb - 1)), n], dtype=np.int64)
    plan = check_plan(rowptr, cols, n, colblk)
    bad = cols.copy()
    bad[nnz // 3] = n
    ws, needed, compact = sagnn.plan_buffers(m, n, nnz, nb, torch.device("cuda"), plan.N, True)
    for ci, cap, code in ((bad, plan.N, -3), (cols, plan.N - 1, -2)):
        needed.fill_(-7)
        compact.fill_(-7)
        with pytest.raises(sagnn.SagnnError) as ei:
            sagnn.spmm_plan_needed_rows(dev(rowptr), dev(ci), n, colblk, needed_cap=cap, bufs=(ws, needed, compact),
                                        validate=code == -3)
        assert ei.value.code == code
        torch.cuda.synchronize()
        assert bool((needed == -7).all())
        if nnz < 8 * n:
            assert bool((compact == -7).all())


def test_plan_cfg1_all_blocks(cfg1):
    g, _ = cfg1
    off = synth.block_offsets(g.n, 4)
    for i in range(4):
        blk = g.row_block(int(off[i]), int(off[i + 1]))
        check_plan(blk.rowptr, blk.colidx, g.n, off)
    check_plan(g.rowptr, g.colidx, g.n, np.array([0, g.n]))


@pytest.mark.parametrize("m,n,nb,avg,seed", [(1, 1, 1, 1, 0), (50, 63, 3, 2, 1), (64, 64, 1, 3, 2),
                                             (1000, 65, 5, 1, 3), (3000, 100_003, 16, 9, 4),
                                             (20000, 5_000_001, 7, 4, 5), (10, 1_000_000, 64, 0.3, 6),
                                             (30000, 20_000_003, 9, 6, 7), (5, 33_554_432, 3, 2, 8)])
def test_plan_random_ragged(m, n, nb, avg, seed):
    rng = np.random.default_rng(seed)
    rowptr, colidx, _ = random_csr(m, n, avg, rng, dup=True)
    cuts = np.sort(rng.integers(0, n + 1, size=nb - 1))       # ragged, possibly empty blocks
    colblk = np.array([0, *cuts, n], dtype=np.int64)
    check_plan(rowptr, colidx, n, colblk)


@pytest.mark.parametrize("n,nnz,misalign", [(1_000_000, 4_300_000, 0), (1_245_185, 4_200_003, 1),
                                            (2_700_001, 4_500_001, 3), (4_980_736, 4_194_304, 0),
                                            (500_000, 4_300_000, 0), (100_000, 4_300_003, 0),
                                            (100_001, 4_300_001, 1),
                                            # wider than four LDS ranges: entries partitioned by range first
                                            (4_980_737, 4_200_000, 0), (6_225_921, 4_300_003, 1),
                                            (20_000_003, 4_500_001, 3), (111_059_956, 5_000_000, 0),
                                            (318_767_104, 4_194_304, 0)])
def test_plan_large_entry_counts_lds_marking(n, nnz, misalign):
    """Entry counts above 2^22 with at most ~5 M columns take the LDS-bitmap marking path
    (1 to 4 column ranges); beyond that, up to 2048 ranges of 155,648 columns (318.8 M columns), the
    entries are partitioned by range first and every range is marked from its bucket; the column array is also given at a 4-byte-but-not-16-byte aligned
    address.  Power-law-like columns (squared uniform) plus the last column of every range.
    With eight or more entries per column the marking pass also writes the identity remap in
    advance: the 500 k-column case leaves columns unused (the advance copy must be replaced by
    the real remap), the 100 k-column cases use every column (it is the result)."""
    rng = np.random.default_rng(n % 97)
    m = 5000
    cols = (rng.random(nnz) ** 2 * n).astype(np.int64)
    cols[:8] = [0, n - 1, min(n - 1, 1_245_183), min(n - 1, 1_245_184), min(n - 1, 2_490_367),
                min(n - 1, 2_490_368), min(n - 1, 3_735_552), n // 2]
    if n > 4_980_736:
        # first and last column of the ranges around the middle and at the end; a uniform share so that
        # the far ranges are not empty
        r = 1_245_184
        mid, last = (n // 2) // r, (n - 1) // r
        edge = [mid * r - 1, mid * r, mid * r + r - 1, last * r - 1, last * r, n - 2, 155_647, 155_648,
                (n - 1) // 155_648 * 155_648 - 1, (n - 1) // 155_648 * 155_648]
        cols[8:8 + len(edge)] = [min(max(c, 0), n - 1) for c in edge]
        cols[100:100 + nnz // 4] = rng.integers(0, n, size=nnz // 4)
    cuts = np.sort(rng.integers(0, nnz + 1, size=m - 1))
    rowptr = np.array([0, *cuts, nnz], dtype=np.int32)
    colidx = cols.astype(np.int32)
    colblk = np.array([0, n // 3, n // 3, n - 5, n], dtype=np.int64)
    buf = torch.empty(nnz + 4, dtype=torch.int32, device="cuda")
    ci = buf[misalign:misalign + nnz]
    ci.copy_(torch.from_numpy(colidx))
    plan = sagnn.spmm_plan_needed_rows(dev(rowptr), ci, n, colblk, validate=True)
    torch.cuda.synchronize()
    needed, blk_off, compact = oracle.needed_rows(rowptr, colidx, n, colblk)
    assert np.array_equal(plan.blk_off, blk_off)
    assert np.array_equal(plan.needed.cpu().numpy(), needed)
    assert np.array_equal(plan.colidx_compact.cpu().numpy(), compact)
    if n == 500_000:
        assert plan.N < n
    if n in (100_000, 100_001):
        assert plan.N == n
    ci[12345] = n                                           # out of range: validation must see it
    with pytest.raises(sagnn.SagnnError) as ei:
        sagnn.spmm_plan_needed_rows(dev(rowptr), ci, n, colblk, validate=True)
    assert ei.value.code == -3
    ci[12345] = -2                                          # negative: likewise
    with pytest.raises(sagnn.SagnnError) as ei:
        sagnn.spmm_plan_needed_rows(dev(rowptr), ci, n, colblk, validate=True)
    assert ei.value.code == -3


@pytest.mark.parametrize("n,nnz", [(1_245_185, 10_000_003), (2_500_000, 20_000_000)])
def test_plan_identity_written_by_several_column_ranges(n, nnz):
    """Every column of two and of three ranges is needed: their workgroups take turns at the copy of the columns and at the
    check of their range, in runs of 16384 entries and what is left of a share."""
    rng = np.random.default_rng(n)
    cols = np.concatenate([np.arange(n), rng.integers(0, n, size=nnz - n)]).astype(np.int32)
    rng.shuffle(cols)
    rowptr = np.linspace(0, nnz, 4001).astype(np.int32)
    ci, rp = dev(cols), dev(rowptr)
    plan = sagnn.spmm_plan_needed_rows(rp, ci, n, np.array([0, n], dtype=np.int64), validate=True)
    assert plan.N == n and torch.equal(plan.colidx_compact[:nnz], ci)
    per = -(-(nnz // 4) // (256 // -(-n // 1_245_184))) * 4      # entries of a share
    for at in (0, 16_384, 2 * 16_384 + 1, per - 1, per, per + 40_000, nnz // 4 * 4 - 1, nnz - 1):
        for bad in (n, -1):
            keep = int(ci[at])
            ci[at] = bad
            with pytest.raises(sagnn.SagnnError) as ei:
                sagnn.spmm_plan_needed_rows(rp, ci, n, np.array([0, n], dtype=np.int64), validate=True)
            assert ei.value.code == -3, (at, bad)
            ci[at] = keep


def test_step_calls_take_numbers_of_numpy():
    """Sizes and options as they come out of a host array, the block boundaries that the plan itself takes among them."""
    g = synth.er_graph(4096, 8, 0)
    blk = synth.block_offsets(g.n, 4)
    rp, ci, v = dev(g.rowptr), dev(g.colidx), dev(g.val)
    plan, same = (sagnn.spmm_plan_needed_rows(rp, ci, n, blk) for n in (blk[-1], g.n))
    assert isinstance(blk[-1], np.int64) and plan.N == same.N and torch.equal(plan.needed, same.needed)
    X, W = dev(synth.normal((g.n, 32), 0, synth.STREAM_H)), dev(synth.normal((32, 16), 0, synth.STREAM_W))
    options = np.array([0, sagnn.GEMM_BF16, sagnn.ACT_RELU], dtype=np.int32)
    for a, b in zip(sagnn.dense_gemm_act(X, W, transW=options[0], prec=options[1], act=options[2]),
                    sagnn.dense_gemm_act(X, W, prec=sagnn.GEMM_BF16, act=sagnn.ACT_RELU)):
        assert a is b or torch.equal(a, b)


def test_plan_empty_matrix_and_capacity_and_validate():
    rp = np.zeros(6, np.int32)
    plan = sagnn.spmm_plan_needed_rows(dev(rp), torch.empty(0, dtype=torch.int32, device="cuda"), 100,
                                       np.array([0, 50, 100]))
    assert plan.N == 0 and list(plan.blk_off) == [0, 0, 0]
    rng = np.random.default_rng(0)
    rowptr, colidx, _ = random_csr(100, 1000, 5, rng)
    with pytest.raises(sagnn.SagnnError) as ei:
        sagnn.spmm_plan_needed_rows(dev(rowptr), dev(colidx), 1000, np.array([0, 1000]), needed_cap=3)
    assert ei.value.code == -2
    bad = colidx.copy()
    bad[7] = 1000
    with pytest.raises(sagnn.SagnnError) as ei:
        sagnn.spmm_plan_needed_rows(dev(rowptr), dev(bad), 1000, np.array([0, 1000]), validate=True)
    assert ei.value.code == -3
    badrp = rowptr.copy()
    badrp[10] = badrp[11] + 1
    with pytest.raises(sagnn.SagnnError) as ei:
        sagnn.spmm_plan_needed_rows(dev(badrp), dev(colidx), 1000, np.array([0, 1000]), validate=True)
    assert ei.value.code == -3
    # without validation the bad column is skipped and flagged -1 in the remap
    plan = sagnn.spmm_plan_needed_rows(dev(rowptr), dev(bad), 1000, np.array([0, 1000]))
    assert int(plan.colidx_compact[7]) == -1
    sagnn.spmm_plan_needed_rows(dev(rowptr), dev(colidx), 1000, np.array([0, 1000]), validate=True)
    # every column needed (the remap is then the identity) and one column out of range
    n = 777
    rp2 = np.arange(0, n + 2, dtype=np.int32)
    ci2 = np.concatenate([rng.permutation(n), [n + 3]]).astype(np.int32)
    plan = sagnn.spmm_plan_needed_rows(dev(rp2), dev(ci2), n, np.array([0, 100, n]))
    assert plan.N == n and np.array_equal(plan.needed.cpu().numpy(), np.arange(n))
    assert np.array_equal(plan.colidx_compact.cpu().numpy(), np.concatenate([ci2[:-1], [-1]]))


# ------------------------------------------------------------------------------------ SpMM

def run_spmm(rowptr, colidx, val, B, use_ws, C0=None, expect_mode=None):
    rp, ci, v = dev(rowptr), dev(colidx), dev(val)
    ws = sagnn.spmm_csr_prepare(rp, ci, v, B.shape[0], B.shape[1]) if use_ws else None
    if expect_mode is not None:
        assert ws.info()["mode"] == expect_mode, ws.info()
    C = None if C0 is None else dev(C0)
    out = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(B), C=C, accumulate=C0 is not None, ws=ws)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("f", [4, 16, 20, 32, 48, 64, 100, 128, 192, 256, 320])
@pytest.mark.parametrize("use_ws", [True, False])
def test_spmm_random_widths(f, use_ws):
    rng = np.random.default_rng(f)
    m, n = 3001, 2500
    rowptr, colidx, val = random_csr(m, n, 12, rng, empty_frac=0.15, hubs=[(7, 3000), (1500, 777), (3000, 300)],
                                     dup=True)
    B = synth.normal((n, f), f, synth.STREAM_H)
    ref, zabs = oracle.spmm(rowptr, colidx, val, B, want_abs=True)
    got = run_spmm(rowptr, colidx, val, B, use_ws)
    assert_close(got, ref, zabs, RTOL_SPMM, f"spmm f={f} ws={use_ws}")
    C0 = synth.normal((m, f), f + 1, synth.STREAM_G)
    ref2, zabs2 = oracle.spmm(rowptr, colidx, val, B, C=C0, want_abs=True)
    got2 = run_spmm(rowptr, colidx, val, B, use_ws, C0=C0)
    assert_close(got2, ref2, zabs2, RTOL_SPMM, f"spmm accumulate f={f} ws={use_ws}")


@pytest.fixture(params=["short_rows_by_nonzero_splitting", "short_rows_swept_whole"])
def force_sweep(request, monkeypatch):
    """Force the slab-sweep schedule on small matrices (the heuristic reserves it for big ones)
    with tiny pieces and many slabs, so that split rows, staggered starts and the short-row
    path are all exercised -- the short rows once through the nonzero-splitting kernel on their
    compacted CSR, once as whole-row wavefronts of the sweep (where the width has that form)."""
    monkeypatch.setenv("SAGNN_SWEEP_SHORT_ROWS", "-1" if request.param == "short_rows_by_nonzero_splitting" else "1")
    monkeypatch.setenv("SAGNN_SWEEP", "1")
    monkeypatch.setenv("SAGNN_SWEEP_MINDEG", "16")
    monkeypatch.setenv("SAGNN_SWEEP_PIECE", "1024")
    monkeypatch.setenv("SAGNN_SWEEP_SLAB_MB", "0")
    monkeypatch.setenv("SAGNN_SWEEP_GROUPS", "2")      # lane-group kernels at f = 128 / 64 even with little reuse


@pytest.mark.parametrize("m,n,f", [(1, 50, 64), (700, 300, 16), (30_001, 30_001, 64), (300_000, 1000, 256), (300_000, 9000, 256)])
def test_spmm_chunks_in_runs_for_each_xcd(m, n, f, monkeypatch):
    """Nonzero splitting with the chunks dealt to the XCDs in runs: fewer workgroups than XCDs, all in one run each, and
    several windows of runs (more rows than the memory-side cache holds), also with the columns in parts; rows that neighbouring
    chunks share."""
    monkeypatch.setenv("SAGNN_SWEEP", "0")
    rng = np.random.default_rng(m)
    rowptr, colidx, val = random_csr(m, n, 2, rng, empty_frac=0.1, hubs=[(m // 2, 200), (m - 1, 40)])
    B = synth.normal((n, f), 3, synth.STREAM_H)
    ref, zabs = oracle.spmm(rowptr, colidx, val, B, want_abs=True)
    assert_close(run_spmm(rowptr, colidx, val, B, True, expect_mode=0), ref, zabs, RTOL_SPMM, f"{m} rows, f={f}")


@pytest.mark.parametrize("f,target", [(4, 3_000), (16, 8_500_000), (20, 400_000), (32, 4_300_000), (36, 40_000), (64, 600_000),
                                      (100, 300_000), (132, 140_000), (256, 270_000), (260, 1_100_000)])
def test_spmm_chunks_at_their_edges(f, target, monkeypatch):
    """Nonzero splitting with chunks of every length (16 entries up to 128): rows that end on, just before and just
    behind a chunk boundary, rows shared by two, some and many chunks (both carry fix-ups), empty rows, every lane-group
    width with a full and a ragged operand."""
    monkeypatch.setenv("SAGNN_SWEEP", "0")
    rng = np.random.default_rng(f)
    kinds = np.array([0, 1, 7, 8, 9, 15, 16, 17, 31, 33, 100, 129, 300])
    deg = kinds[rng.integers(0, kinds.size, size=max(8, target // 55))]
    deg[deg.size // 2] = min(20_000, target)
    deg[-1] = 3000
    n = 5000
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    colidx = rng.integers(0, n, size=rowptr[-1]).astype(np.int32)
    val = rng.standard_normal(colidx.size).astype(np.float32)
    B = synth.normal((n, f), f, synth.STREAM_H)
    ref, zabs = oracle.spmm(rowptr, colidx, val, B, want_abs=True)
    assert_close(run_spmm(rowptr, colidx, val, B, True, expect_mode=0), ref, zabs, RTOL_SPMM, f"chunks f={f}")
    C0 = synth.normal((deg.size, f), f + 1, synth.STREAM_G)
    ref2, zabs2 = oracle.spmm(rowptr, colidx, val, B, C=C0, want_abs=True)
    assert_close(run_spmm(rowptr, colidx, val, B, True, C0=C0), ref2, zabs2, RTOL_SPMM, f"chunks accumulate f={f}")


@pytest.mark.parametrize("f,n,deg,hubs", [(128, 16_411, 12, 0), (192, 16_411, 17, 0), (256, 9_001, 11, 0), (256, 33_001, 20, 3), (320, 9_001, 13, 0),
                                          (128, 100_003, 11, 2), (256, 13_001, 11, 0), (256, 50_003, 12, 2), (192, 38_503, 30, 2),
                                          (192, 48_001, 12, 0), (192, 48_001, 12, 2)])
def test_spmm_chunks_in_column_parts(f, n, deg, hubs, monkeypatch):
    """Nonzero splitting of operands that are larger than two L2s takes columns in two and four parts: bit for bit
    what the same workspace gives of 64 columns at a time, which are not cut.  Counts of workgroups that the XCDs of a part do not share evenly,
    rows shared by chunks, empty rows, hubs, accumulation, an operand with gaps and one that begins inside a line."""
    monkeypatch.setenv("SAGNN_SWEEP", "0")
    gen = torch.Generator(device="cuda").manual_seed(f + n)
    count = torch.randint(0, 2 * deg + 2, (n,), device="cuda", generator=gen)
    count[5::499] = 0
    count[:hubs] = 4000
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(count, 0)
    nnz = int(rp[-1])
    assert nnz >= 10 * n
    ci = torch.randint(n, (nnz,), device="cuda", generator=gen, dtype=torch.int32)
    v = torch.randn(nnz, device="cuda", generator=gen)
    wide = torch.randn(n, f + 64, device="cuda", generator=gen)
    C0 = torch.randn(n, f, device="cuda", generator=gen)
    ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
    assert ws.info()["mode"] == 0
    A, Aabs = (torch.sparse_csr_tensor(rp.long(), ci.long(), x.double(), (n, n)) for x in (v, v.abs()))
    for B in (wide[:, :f].contiguous(), wide[:, :f], wide[:, 4:f + 4]):
        got = sagnn.spmm_csr_tallskinny(rp, ci, v, B, ws=ws)
        for c in range(0, f, 64):
            assert torch.equal(got[:, c:c + 64], sagnn.spmm_csr_tallskinny(rp, ci, v, B[:, c:c + 64], ws=ws)), c
        assert float(((got.double() - A @ B.double()).abs() - RTOL_SPMM * (Aabs @ B.double().abs())).max()) <= 1e-30
        acc = sagnn.spmm_csr_tallskinny(rp, ci, v, B, C=C0.clone(), accumulate=True, ws=ws)
        bound = RTOL_SPMM * (Aabs @ B.double().abs() + C0.double().abs())
        assert float(((acc.double() - A @ B.double() - C0.double()).abs() - bound).max()) <= 1e-30


@pytest.mark.parametrize("f,target", [(4, 3_000), (16, 8_500_000), (32, 400_000), (64, 600_000), (100, 300_000), (128, 300_000),
                                      (256, 270_000), (320, 60_000)])
def test_spmm_infinities_in_rows_that_chunks_cut(f, target, monkeypatch):
    """Nonzero splitting: entries and operand are positive, some rows of B infinite, so every row of C that uses one of them
    is +inf and no other is.  A chunk that is done before its neighbours goes on with weight 0 on its last column; a row
    that the chunk's end cuts is open until then."""
    monkeypatch.setenv("SAGNN_SWEEP", "0")
    rng = np.random.default_rng(f)
    kinds = np.array([0, 1, 7, 9, 17, 33, 40, 50, 70, 100, 129, 300])
    deg = kinds[rng.integers(0, kinds.size, size=max(8, target // 63))]
    deg[deg.size // 2] = min(20_000, target)
    n = 5000
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    colidx = rng.integers(0, n, size=rowptr[-1]).astype(np.int32)
    val = rng.uniform(0.5, 1.5, size=colidx.size).astype(np.float32)
    B = np.abs(synth.normal((n, f), f, synth.STREAM_H)) + np.float32(0.1)
    infinite = rng.random(n) < 0.02
    rows = np.repeat(np.arange(deg.size), deg)
    hit = np.bincount(rows[infinite[colidx]], minlength=deg.size) > 0
    ref, zabs = oracle.spmm(rowptr, colidx, val, B, want_abs=True)
    B[infinite] = np.inf
    for C0 in (None, np.ones((deg.size, f), np.float32)):
        got = run_spmm(rowptr, colidx, val, B, True, C0=C0, expect_mode=0).cpu().numpy()
        assert np.isposinf(got[hit]).all(), f"{np.isnan(got[hit]).any(axis=1).sum()} of {hit.sum()} rows hold NaN"
        assert_close(got[~hit], ref[~hit] + (0 if C0 is None else 1), zabs[~hit] + 1, RTOL_SPMM, f"f={f}")


@pytest.mark.parametrize("f", [4, 12, 16, 20, 32, 36, 60, 68, 100, 124])
def test_spmm_narrow_products_are_closer_than_one_sum_in_stored_order(f, monkeypatch):
    """Nonzero splitting below full width adds batches of eight entries, then the batches: on rows of 60 entries the error
    against 64 bits is well below that of one fused multiply-add after the other (root mean squares of the partial sums:
    sqrt(525) against sqrt(1830), 0.54; up to 0.6 for rows that begin inside a batch)."""
    monkeypatch.setenv("SAGNN_SWEEP", "0")
    m, n, d = 30_011, 20_000, 60
    gen = torch.Generator(device="cuda").manual_seed(f)
    ci = torch.randint(n, (m, d), device="cuda", generator=gen, dtype=torch.int32)
    v = torch.full((m, d), 1.0 / d, device="cuda")
    B = torch.randn(n, f, device="cuda", generator=gen)
    exact, serial = torch.zeros(m, f, device="cuda", dtype=torch.double), torch.zeros(m, f, device="cuda")
    for j in range(d):
        term = v[:, j:j + 1].double() * B[ci[:, j].long()].double()
        exact += term
        serial = (serial.double() + term).float()
    rp = torch.arange(m + 1, device="cuda", dtype=torch.int32) * d
    args = rp, ci.reshape(-1), v.reshape(-1)
    ws = sagnn.spmm_csr_prepare(*args, n, f)
    assert ws.info()["mode"] == 0
    got = sagnn.spmm_csr_tallskinny(*args, B, ws=ws)
    assert float((got.double() - exact).norm()) < 0.75 * float((serial.double() - exact).norm())


@pytest.mark.parametrize("f", [16, 32, 64, 128, 192, 256, 320])
def test_spmm_slab_sweep_schedule(f, force_sweep):
    rng = np.random.default_rng(100 + f)
    m, n = 5003, 40_000
    rowptr, colidx, val = random_csr(m, n, 20, rng, empty_frac=0.1,
                                     hubs=[(3, 9000), (7, 3000), (2500, 1024), (2501, 1025), (5002, 17), (11, 16)])
    B = synth.normal((n, f), f, synth.STREAM_H)
    ref, zabs = oracle.spmm(rowptr, colidx, val, B, want_abs=True)
    got = run_spmm(rowptr, colidx, val, B, True, expect_mode=1)
    assert_close(got, ref, zabs, RTOL_SPMM, f"sweep f={f}")
    got_again = run_spmm(rowptr, colidx, val, B, True)
    assert torch.equal(got, got_again)                       # reproducible across preparations
    C0 = synth.normal((m, f), f + 1, synth.STREAM_G)
    ref2, zabs2 = oracle.spmm(rowptr, colidx, val, B, C=C0, want_abs=True)
    got2 = run_spmm(rowptr, colidx, val, B, True, C0=C0)
    assert_close(got2, ref2, zabs2, RTOL_SPMM, f"sweep accumulate f={f}")


@pytest.mark.parametrize("groups", [0, 1, 2])
@pytest.mark.parametrize("f", [4, 12, 20, 28, 36, 60, 68, 100, 124, 132, 252, 260, 300, 516])
def test_spmm_sweep_widths_between_the_kernels(f, groups, force_sweep, monkeypatch):
    """Widths that no sweep kernel has exactly, in every lane-group form; also a narrower operand on the same
    workspace, and a row stride wider than the operand."""
    monkeypatch.setenv("SAGNN_SWEEP_GROUPS", str(groups))
    rng = np.random.default_rng(f)
    m, n = 3001, 9000
    rowptr, colidx, val = random_csr(m, n, 25, rng, empty_frac=0.1, hubs=[(3, 5000), (1500, 1024), (3000, 17), (11, 16)])
    B = synth.normal((n, f), f, synth.STREAM_H)
    C0 = synth.normal((m, f), f + 1, synth.STREAM_G)
    rp, ci, v = dev(rowptr), dev(colidx), dev(val)
    ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
    if groups == 2 or f > 32:
        assert ws.info()["mode"] == 1
    for w in sorted({f, max(4, f - 4), max(4, f // 2 // 4 * 4)}):
        wide = torch.full((n, f + 8), float("nan"), device="cuda")
        wide[:, :w] = dev(B)[:, :w]
        ref, zabs = oracle.spmm(rowptr, colidx, val, B[:, :w], want_abs=True)
        got = sagnn.spmm_csr_tallskinny(rp, ci, v, wide[:, :w], C=torch.full((m, w), float("nan"), device="cuda"), ws=ws)
        assert_close(got, ref, zabs, RTOL_SPMM, f"f={f} w={w}")
        ref, zabs = oracle.spmm(rowptr, colidx, val, B[:, :w], C=C0[:, :w], want_abs=True)
        got = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(B[:, :w].copy()), C=dev(C0[:, :w].copy()), accumulate=True, ws=ws)
        assert_close(got, ref, zabs, RTOL_SPMM, f"accumulate f={f} w={w}")


@pytest.mark.parametrize("f,sync", [(4, 0), (8, 0), (12, 0), (16, 0), (20, 0), (32, 0), (64, 0), (100, 0), (128, 0), (256, 0),
                                    (48, 96), (64, 96), (128, 96)])
def test_spmm_sweep_keeps_a_non_finite_row_of_b_to_the_rows_that_use_it(f, sync, monkeypatch):
    """The steps that pad a stream, or an interval of `sync` slabs, multiply row 0 of B by 0: where that row holds NaN and
    infinities, a row of C has them if and only if one of its entries lies in column 0."""
    for name, value in (("", 1), ("_MINDEG", 16), ("_PIECE", 1024), ("_SLAB_MB", 0), ("_GROUPS", 2), ("_SYNC", sync)):
        monkeypatch.setenv("SAGNN_SWEEP" + name, str(value))
    rng = np.random.default_rng(f)
    m, n = 3001, 9000
    rowptr, colidx, val = random_csr(m, n, 25, rng, empty_frac=0.1, hubs=[(3, 5000), (40, 20), (1500, 1024), (3000, 17)])
    colidx = np.maximum(colidx, 1)
    users = np.array([3, 40, 1500])
    colidx[rowptr[users]] = 0
    B = synth.normal((n, f), f, synth.STREAM_H)
    B[0, 0::2], B[0, 1::2] = np.nan, np.inf
    finite = B.copy()
    finite[0] = 0.0
    rp, ci, v = dev(rowptr), dev(colidx), dev(val)
    ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
    assert ws.info()["mode"] == 1 and (ws.info()["intervals"] > 1) == (sync > 0)
    others = np.setdiff1d(np.arange(m), users)
    infinity = np.broadcast_to(np.copysign(np.inf, val[rowptr[users]])[:, None], (users.size, f // 2))
    for C0 in (None, synth.normal((m, f), f + 1, synth.STREAM_G)):
        ref, zabs = oracle.spmm(rowptr, colidx, val, finite, C=C0, want_abs=True)
        got = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(B), C=None if C0 is None else dev(C0), accumulate=C0 is not None,
                                        ws=ws).cpu().numpy()
        assert np.isfinite(got[others]).all(), f"{(~np.isfinite(got[others])).any(axis=1).sum()} rows that do not use row 0"
        assert_close(got[others], ref[others], zabs[others], RTOL_SPMM, f"f={f}")
        assert np.isnan(got[users, 0::2]).all() and np.array_equal(got[users, 1::2], infinity)


@pytest.mark.parametrize("f,n", [(12, 200_000), (24, 90_000), (28, 90_001), (60, 40_000), (124, 20_000)])
@pytest.mark.parametrize("sweep", [False, True])
def test_spmm_rows_moved_to_cache_lines(f, n, sweep, monkeypatch):
    """Widths and entry counts at which B is copied to aligned rows first, by both schedules: rows of B with gaps between
    them, fewer rows of B than the workspace has room for, more of them (no copy then)."""
    monkeypatch.setenv("SAGNN_SWEEP", "1" if sweep else "0")
    rng = np.random.default_rng(f)
    deg = 30 if f < 60 else 60
    for m, k in ((n, n), (n, n - 777), (n // 2, n)):
        nnz = deg * n
        rowptr = np.concatenate([[0], np.cumsum(rng.multinomial(nnz, np.full(m, 1.0 / m)))]).astype(np.int32)
        rows = np.repeat(np.arange(m), np.diff(rowptr))
        colidx = rng.integers(0, k, size=nnz)
        colidx = colidx[np.lexsort((colidx, rows))].astype(np.int32)
        val = rng.standard_normal(nnz).astype(np.float32)
        B = synth.normal((k, f), f, synth.STREAM_H)
        rp, ci, v = dev(rowptr), dev(colidx), dev(val)
        ws = sagnn.spmm_csr_prepare(rp, ci, v, k, f)
        wide = torch.full((k, f + 4), float("nan"), device="cuda")
        wide[:, :f] = dev(B)
        ref = torch.sparse_csr_tensor(rp.long(), ci.long(), v.double(), (m, k)) @ dev(B).double()
        zabs = torch.sparse_csr_tensor(rp.long(), ci.long(), v.double().abs(), (m, k)) @ dev(B).double().abs()
        for operand in (dev(B), wide[:, :f]):
            got = sagnn.spmm_csr_tallskinny(rp, ci, v, operand, C=torch.full((m, f), float("nan"), device="cuda"), ws=ws)
            assert_close(got, ref.cpu().numpy(), zabs.cpu().numpy(), RTOL_SPMM, f"f={f} m={m} k={k}")


@pytest.mark.parametrize("f,n,deg,parts", [(64, 300_000, 20, 1), (128, 150_000, 24, 1), (192, 60_000, 60, 1), (256, 60_000, 60, 1),
                                           (64, 300_000, 20, 4), (256, 260_000, 20, 4)])
def test_spmm_sweep_in_groups_of_64_columns(f, n, deg, parts):
    """Matrices without hubs whose rows of B are wanted several times by rows that are resident together: 64 columns a
    launch, several launches for many rows.  Rows of B with gaps, an operand narrower than the workspace was prepared for
    (one that is a multiple of 64 and one that is not), accumulation, and the layer that needs whole rows of A H."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(f + n)
    count = torch.randint(deg - 6, deg + 7, (n,), device="cuda", generator=gen)
    count[::977] = 0
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(count, 0)
    nnz, part = int(rp[-1]), n // parts
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), count)
    col = row // part * part + torch.randint(part, (nnz,), device="cuda", generator=gen)
    col = torch.where(torch.rand(nnz, device="cuda", generator=gen) < 0.05, torch.randint(n, (nnz,), device="cuda", generator=gen), col)
    ci = (torch.sort(row * n + col.clamp(max=n - 1))[0] - row * n).to(torch.int32)
    v = torch.randn(nnz, device="cuda", generator=gen)
    wide = torch.randn(n, f + 12, device="cuda", generator=gen)
    B = wide[:, :f]
    ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
    assert ws.info()["mode"] == 1 and ws.info()["groups"] == 1 and ws.launch_info()["columns"] == 64
    A, Aabs = (torch.sparse_csr_tensor(rp.long(), ci.long(), x.double(), (n, n)) for x in (v, v.abs()))
    C0 = torch.randn(n, f, device="cuda", generator=gen)
    for w in {f, 64, 52}:
        ref, zabs = A @ B[:, :w].double(), Aabs @ B[:, :w].double().abs()
        for C in (None, C0[:, :w].contiguous()):
            want, scale = (ref, zabs) if C is None else (ref + C.double(), zabs + C.double().abs())
            got = sagnn.spmm_csr_tallskinny(rp, ci, v, B[:, :w], C=C, accumulate=C is not None, ws=ws)
            err = (got.double() - want).abs() - RTOL_SPMM * scale
            assert float(err.max()) <= 1e-30, f"f={f} w={w} accumulate={C is not None}"
    if f == 192:
        return
    W = torch.randn(f, 40, device="cuda", generator=gen) / f ** 0.5
    T, Z, H = sagnn.gcn_layer_fwd(rp, ci, v, B, W, ws=ws)
    assert sagnn.gcn_layer_fwd_form(ws, f, 40) == 2
    _, Z2, H2 = sagnn.gcn_layer_fwd(rp, ci, v, B, W, ws=ws, want_t=False)
    scale = (Aabs @ B.double().abs()) @ W.double().abs()
    want = (A @ B.double()) @ W.double()
    for z, h in ((Z, H), (Z2, H2)):
        # the rows of A H, then f products and sums in 32 bits: both within the forward error of their sums
        assert float(((z.double() - want).abs() - (RTOL_SPMM + f * 2.0 ** -24) * scale).max()) <= 1e-30
        assert torch.equal(h, torch.relu(z))


@pytest.mark.parametrize("f", [64, 128, 192])
@pytest.mark.parametrize("n,deg,half", [(700_000, 20, 35_000), (500_000, 24, 60_000)])
def test_spmm_no_column_groups_along_the_diagonal(n, deg, half, f):
    """Entries within a distance of the diagonal: resident rows do not choose from the same columns, as they do in
    communities, and the product keeps the whole width in a launch where it can."""
    gen = torch.Generator(device="cuda").manual_seed(n + f)
    cols = torch.arange(n, device="cuda")[:, None] + torch.randint(-half, half + 1, (n, deg), device="cuda", generator=gen)
    cols = torch.sort(cols.clamp_(0, n - 1), dim=1)[0]
    rp = torch.arange(0, n * deg + 1, deg, dtype=torch.int32, device="cuda")
    ci = cols.to(torch.int32).reshape(-1)
    v, B = torch.randn(n * deg, device="cuda", generator=gen), torch.randn(n, f, device="cuda", generator=gen)
    ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
    assert ws.info()["mode"] == 1 and ws.launch_info()["columns"] == 0
    C = sagnn.spmm_csr_tallskinny(rp, ci, v, B, ws=ws)
    rows = torch.cat([torch.arange(0, n, 101, device="cuda"), torch.tensor([n - 1], device="cuda")])
    t = v.reshape(n, deg)[rows].double()[:, :, None] * B[cols[rows]].double()
    assert bool(((C[rows].double() - t.sum(1)).abs() <= (deg + 2) * 2.0 ** -24 * t.abs().sum(1)).all())


@pytest.mark.parametrize("f,k", [(64, 4_505_600), (64, 4_505_601), (96, 3_003_733), (96, 3_003_734), (128, 2_252_800), (128, 2_252_801)])
def test_spmm_one_row_per_load_on_both_sides_of_turns(f, k):
    """Rows of B that are hardly used twice, one row per load, with B just under and just over 1100 MB: whether the
    wavefronts take turns changes nothing in the result, which is compared with 64-bit sums of the same rows."""
    gen = torch.Generator(device="cuda").manual_seed(f)
    m, deg = 170_000, 20
    rp = torch.arange(0, m * deg + 1, deg, dtype=torch.int32, device="cuda")
    ci = torch.sort(torch.randint(k, (m, deg), device="cuda", generator=gen), dim=1)[0].to(torch.int32).reshape(-1)
    ci[-1] = k - 1
    v, B = torch.randn(m * deg, device="cuda", generator=gen), torch.randn(k, f, device="cuda", generator=gen)
    ws = sagnn.spmm_csr_prepare(rp, ci, v, k, f)
    info = ws.info()
    assert info["mode"] == 1 and info["groups"] == 1 and ws.launch_info()["columns"] == 0
    C = sagnn.spmm_csr_tallskinny(rp, ci, v, B, ws=ws)
    rows = torch.cat([torch.arange(0, m, 37, device="cuda"), torch.tensor([m - 1], device="cuda")])
    t = v.reshape(m, deg)[rows].double()[:, :, None] * B[ci.reshape(m, deg)[rows].long()].double()
    assert bool(((C[rows].double() - t.sum(1)).abs() <= (deg + 2) * 2.0 ** -24 * t.abs().sum(1)).all())


@pytest.mark.parametrize("n,deg,slabs", [(60_000, 120, 8), (60_000, 200, 16), (60_000, 489, 16), (45_000, 60, 8)])
def test_spmm_column_groups_keep_segments_short(n, deg, slabs):
    """Random columns, 256 of B, 64 a launch: slabs of 8192 rows of B while a row has at most 16 entries in one, else slabs of
    4 MB.  The error against 64 bits is no larger than in slabs of 4 MB (1 % for what a sample of rows leaves open)."""
    gen = torch.Generator(device="cuda").manual_seed(deg)
    f = 256
    rp = torch.arange(0, n * deg + 1, deg, dtype=torch.int32, device="cuda")
    ci = torch.sort(torch.randint(n, (n, deg), device="cuda", generator=gen), dim=1)[0].to(torch.int32).reshape(-1)
    v, B = torch.randn(n * deg, device="cuda", generator=gen), torch.randn(n, f, device="cuda", generator=gen)
    rows = torch.arange(0, n, 7, device="cuda")
    At = torch.sparse_csr_tensor(torch.arange(0, rows.numel() * deg + 1, deg, device="cuda"), ci.reshape(n, deg)[rows].reshape(-1).long(),
                                 v.reshape(n, deg)[rows].reshape(-1).double(), (rows.numel(), n))
    ref = At @ B.double()

    def error(options):
        ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f, options=options)
        assert ws.launch_info()["columns"] == 64
        C = sagnn.spmm_csr_tallskinny(rp, ci, v, B, ws=ws)
        return ws.launch_info()["slabs"], float((C[rows].double() - ref).norm() / ref.norm())

    got, err = error(None)
    assert got == slabs
    assert err <= 1.01 * error(sagnn.SpmmOptions(slab_kb=4096))[1]


@pytest.mark.parametrize("f,k,ld", [(96, 436_906, 96), (96, 436_907, 96), (128, 1_228_800, 128), (128, 1_228_801, 128), (128, 1_228_801, 1024), (100, 671_088, 100), (100, 671_089, 100),
                                    (100, 671_089, 1700)])
def test_spmm_two_rows_per_load_on_both_sides_of_words_ahead(f, k, ld):
    """Two lane groups with B on either side of the sizes up to which the stream's words are requested ahead, also with rows
    of B so far apart that buffer loads do not reach them; at 128 columns the layer in its three precisions too."""
    gen = torch.Generator(device="cuda").manual_seed(f)
    m, deg = 106_000, 30
    rp = torch.arange(0, m * deg + 1, deg, dtype=torch.int32, device="cuda")
    ci = torch.sort(torch.randint(k, (m, deg), device="cuda", generator=gen), dim=1)[0].to(torch.int32).reshape(-1)
    ci[-1] = k - 1
    v, B = torch.randn(m * deg, device="cuda", generator=gen), torch.randn(k, ld, device="cuda", generator=gen)[:, :f]
    ws = sagnn.spmm_csr_prepare(rp, ci, v, k, f, options=sagnn.SpmmOptions(groups=2))
    assert ws.info()["mode"] == 1 and ws.info()["groups"] == 2
    C = sagnn.spmm_csr_tallskinny(rp, ci, v, B, ws=ws)
    rows = torch.cat([torch.arange(0, m, 23, device="cuda"), torch.tensor([m - 1], device="cuda")])
    t = v.reshape(m, deg)[rows].double()[:, :, None] * B[ci.reshape(m, deg)[rows].long()].double()
    T, unit = t.sum(1), (deg + 2) * 2.0 ** -24 * t.abs().sum(1)
    assert bool(((C[rows].double() - T).abs() <= unit).all())
    if f != 128:
        return
    W = torch.randn(f, 64, device="cuda", generator=gen) / f ** 0.5
    Wd = W.double()
    for prec in (sagnn.GEMM_FP32, sagnn.GEMM_BF16, sagnn.GEMM_FP32_BF16X3):
        assert sagnn.gcn_layer_fwd_form(ws, f, 64, prec) == 2
        _, Z, _ = sagnn.gcn_layer_fwd(rp, ci, v, B, W, prec=prec, ws=ws, want_t=False)
        bound = unit @ Wd.abs() + (f + 4) * 2.0 ** -24 * (T.abs() @ Wd.abs())
        if prec == sagnn.GEMM_BF16:   # both operands rounded to 8 bits, the sums on top
            bound = (unit * 1.01 + 2.0 ** -8 * T.abs()) @ Wd.abs() * 1.01 + bound
        assert bool(((Z[rows].double() - T @ Wd).abs() <= bound).all())


@pytest.mark.parametrize("f,f_out,prec", [(128, 40, sagnn.GEMM_FP32), (128, 128, sagnn.GEMM_BF16), (128, 64, sagnn.GEMM_FP32_BF16X3),
                                          (128, 128, sagnn.GEMM_FP32), (64, 64, sagnn.GEMM_FP32), (256, 256, sagnn.GEMM_BF16)])
def test_layer_on_a_schedule_in_groups_of_64_columns(f, f_out, prec):
    """The layer whose A H is not wanted, on communities that are multiplied 64 columns at a time: at 128 columns with a
    short dense part its wavefronts come in several launches.  Bounds as for the product, then f products and sums."""
    gen = torch.Generator(device="cuda").manual_seed(f + f_out)
    n, part = 300_000, 75_000
    count = torch.randint(20, 34, (n,), device="cuda", generator=gen)
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(count, 0)
    nnz = int(rp[-1])
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), count)
    col = row // part * part + torch.randint(part, (nnz,), device="cuda", generator=gen)
    col = torch.where(torch.rand(nnz, device="cuda", generator=gen) < 0.05, torch.randint(n, (nnz,), device="cuda", generator=gen), col)
    ci = (torch.sort(row * n + col)[0] - row * n).to(torch.int32)
    v, H = torch.randn(nnz, device="cuda", generator=gen), torch.randn(n, f, device="cuda", generator=gen)
    W = torch.randn(f, f_out, device="cuda", generator=gen) / f ** 0.5
    ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
    launch = ws.launch_info()
    assert launch["columns"] == 64 and launch["layer_waves"] * 2 == launch["waves"] and ws.info()["sweep_waves"] > 2 * launch["layer_waves"]
    assert sagnn.gcn_layer_fwd_form(ws, f, f_out, prec) == 2
    _, Z, Hout = sagnn.gcn_layer_fwd(rp, ci, v, H, W, prec=prec, ws=ws, want_t=False)
    A, Aabs = (torch.sparse_csr_tensor(rp.long(), ci.long(), x.double(), (n, n)) for x in (v, v.abs()))
    T, Tabs = A @ H.double(), Aabs @ H.double().abs()
    unit = 2.0 ** -24 * (count.double() + 2)[:, None] * Tabs       # of a row of A H, any order of its sums
    Wd = W.double()
    if prec == sagnn.GEMM_BF16:
        # both operands are rounded to 8 bits: 2^-9 of each, an element of A H after its own error
        bound = (unit * (1 + 2.0 ** -8) + 2.0 ** -9 * T.abs()) @ Wd.abs() + (T.abs() * (1 + 2.0 ** -8)) @ (Wd.abs() * 2.0 ** -9)
    else:
        bound = unit @ Wd.abs()
    bound += (f + 4) * 2.0 ** -24 * ((T.abs() * (1 + 2.0 ** -7)) @ Wd.abs())
    assert bool(((Z.double() - T @ Wd).abs() <= bound).all())
    assert torch.equal(Hout, torch.relu(Z))


@pytest.mark.parametrize("n,lo,hi,parts", [(30_000, 55, 65, 1), (30_000, 64, 64, 1), (30_000, 55, 65, 16), (25_600, 100, 120, 16), (80_000, 28, 34, 16)])
@pytest.mark.parametrize("f", [20, 32, 48, 100])
def test_spmm_small_matrices_swept_are_no_further_from_exact(f, n, lo, hi, parts):
    """Small matrices whose sweep takes the place of nonzero splitting, which adds as a tree at these widths: the error
    against 64 bits is no larger (1 %: rows in communities at 48 columns measure 0.7 % at most, the others less than by the
    tree).  One entry in twenty lies outside its row's community."""
    gen = torch.Generator(device="cuda").manual_seed(n + lo)
    deg = torch.randint(lo, hi + 1, (n,), device="cuda", generator=gen)
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(deg, 0)
    nnz, part = int(rp[-1]), n // parts
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), deg)
    col = row // part * part + torch.randint(part, (nnz,), device="cuda", generator=gen)
    col = torch.where(torch.rand(nnz, device="cuda", generator=gen) < 0.05, torch.randint(n, (nnz,), device="cuda", generator=gen), col)
    ci = (torch.sort(row * n + col)[0] - row * n).to(torch.int32)
    v, B = torch.randn(nnz, device="cuda", generator=gen), torch.randn(n, f, device="cuda", generator=gen)
    ref = torch.sparse_csr_tensor(rp.long(), ci.long(), v.double(), (n, n)) @ B.double()

    def error(mode, options):
        ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f, options=options)
        assert ws.info()["mode"] == mode
        return float((sagnn.spmm_csr_tallskinny(rp, ci, v, B, ws=ws).double() - ref).norm())

    assert error(0 if lo == 100 and f == 48 else 1, None) <= 1.01 * error(0, sagnn.SpmmOptions(schedule=1))


@pytest.mark.parametrize("f", [20, 32])
@pytest.mark.parametrize("n,deg,parts", [(300_000, 20, 1), (200_000, 60, 1), (240_000, 20, 16), (240_000, 42, 16)])
def test_spmm_eight_groups_sum_by_the_length_of_segments(n, deg, parts, f):
    """Eight lane groups: plain sums of short segments at 32 columns, two sums of longer ones and at 20, folded every 32
    entries in rows of 42 that lie in one slab.  The error against 64 bits is no larger than that of plain sums, slab by slab,
    of the same rows in 32 bits (half a percent for what a sample of rows leaves open)."""
    gen = torch.Generator(device="cuda").manual_seed(n + deg)
    part = n // parts
    home = (torch.arange(n, device="cuda") // part * part)[:, None]
    cols = torch.sort(home + torch.randint(part, (n, deg), device="cuda", generator=gen), dim=1)[0]
    rp = torch.arange(0, n * deg + 1, deg, dtype=torch.int32, device="cuda")
    ci = cols.to(torch.int32).reshape(-1)
    v, B = torch.randn(n * deg, device="cuda", generator=gen), torch.randn(n, f, device="cuda", generator=gen)
    ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
    assert ws.info()["mode"] == 1 and ws.info()["groups"] == 8
    C = sagnn.spmm_csr_tallskinny(rp, ci, v, B, ws=ws)
    rows = torch.arange(0, n, 3, device="cuda")
    cols, vals = cols[rows], v.reshape(n, deg)[rows]
    slab = cols // -(-n // ws.launch_info()["slabs"])
    total = torch.zeros(rows.numel(), f, device="cuda")
    run, ref, size = torch.zeros_like(total), total.double(), total.double()
    for e in range(deg):
        t = vals[:, e].double()[:, None] * B[cols[:, e]].double()
        ref += t
        size += t.abs()
        run = (run.double() + t).float()   # one fused multiply-add
        last = ((slab[:, e] != slab[:, e + 1]) if e + 1 < deg else torch.ones_like(rows, dtype=torch.bool))[:, None]
        total = torch.where(last, total + run, total)
        run = torch.where(last, torch.zeros_like(run), run)
    assert bool(((C[rows].double() - ref).abs() <= (deg + 2) * 2.0 ** -24 * size).all())
    # (at 20 columns two sums also of short segments: nonzero splitting adds these widths as a tree)
    if f == 32 or deg > 40:
        assert float((C[rows].double() - ref).norm()) <= 1.005 * float((total.double() - ref).norm())


@pytest.mark.parametrize("f", [20, 32, 36, 48, 64, 72, 96, 128, 160, 192, 200])
@pytest.mark.parametrize("n,deg,parts", [(120_000, 40, 16), (640_000, 21, 16), (40_000, 90, 1)])
def test_spmm_with_and_without_turns(n, deg, parts, f):
    """Communities of few and of many columns, and random ones: whether the wavefronts take turns changes nothing in the
    product, nor in the layer where it ends the sweep."""
    gen = torch.Generator(device="cuda").manual_seed(n + f)
    part = n // parts
    home = (torch.arange(n, device="cuda") // part * part)[:, None]
    cols = torch.sort(home + torch.randint(part, (n, deg), device="cuda", generator=gen), dim=1)[0]
    rp = torch.arange(0, n * deg + 1, deg, dtype=torch.int32, device="cuda")
    ci = cols.to(torch.int32).reshape(-1)
    v, B = torch.randn(n * deg, device="cuda", generator=gen), torch.randn(n, f, device="cuda", generator=gen)
    ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
    assert ws.info()["mode"] == 1
    C = sagnn.spmm_csr_tallskinny(rp, ci, v, B, ws=ws)
    rows = torch.arange(0, n, 29, device="cuda")
    t = v.reshape(n, deg)[rows].double()[:, :, None] * B[cols[rows]].double()
    T, unit = t.sum(1), (deg + 2) * 2.0 ** -24 * t.abs().sum(1)
    assert bool(((C[rows].double() - T).abs() <= unit).all())
    if f in (64, 128) and sagnn.gcn_layer_fwd_form(ws, f, 64) == 2:
        W = torch.randn(f, 64, device="cuda", generator=gen) / f ** 0.5
        Wd = W.double()
        _, Z, _ = sagnn.gcn_layer_fwd(rp, ci, v, B, W, ws=ws, want_t=False)
        bound = unit @ Wd.abs() + (f + 4) * 2.0 ** -24 * (T.abs() @ Wd.abs())
        assert bool(((Z[rows].double() - T @ Wd).abs() <= bound).all())


@pytest.mark.parametrize("n,deg,parts,f,mode", [(10_000, 160, 1, 16, 1), (10_000, 228, 1, 16, 0), (10_000, 228, 1, 32, 0), (10_000, 228, 1, 48, 0), (10_000, 228, 1, 64, 0),
                                                (10_000, 228, 1, 256, 1), (5_000, 220, 4, 128, 0), (14_400, 180, 16, 64, 0), (14_400, 180, 16, 256, 1)])
def test_spmm_few_long_rows_without_hubs(n, deg, parts, f, mode):
    """Few long rows make few, long streams: such small matrices are swept only where that is faster."""
    gen = torch.Generator(device="cuda").manual_seed(f)
    part = n // parts
    home = (torch.arange(n, device="cuda") // part * part)[:, None]
    ci = torch.sort(home + torch.randint(part, (n, deg), device="cuda", generator=gen), dim=1)[0].to(torch.int32)
    rp = torch.arange(0, n * deg + 1, deg, dtype=torch.int32, device="cuda")
    v, B = torch.randn(n * deg, device="cuda", generator=gen), torch.randn(n, f, device="cuda", generator=gen)
    ws = sagnn.spmm_csr_prepare(rp, ci.reshape(-1), v, n, f)
    assert ws.info()["mode"] == mode
    C = sagnn.spmm_csr_tallskinny(rp, ci.reshape(-1), v, B, ws=ws)
    rows = torch.arange(0, n, 13, device="cuda")
    t = v.reshape(n, deg)[rows].double()[:, :, None] * B[ci[rows].long()].double()
    assert bool(((C[rows].double() - t.sum(1)).abs() <= (deg + 2) * 2.0 ** -24 * t.abs().sum(1)).all())


@pytest.mark.parametrize("f", [4, 16, 20, 32, 36, 64, 72, 100, 128, 192, 256])
@pytest.mark.parametrize("kind", ["even", "local", "empty rows", "long", "cut", "around 64", "hub", "few"])
def test_spmm_small_matrices_without_hubs(kind, f):
    """From 1 M entries on a matrix whose rows are all of a size is swept; one row of many entries, or fewer entries, and it
    is not.  Rows of 20 to 52 entries, some empty, some of exactly a piece's 256, some cut into two pieces, or of 60 to 92;
    products, sums and the layer."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(f)
    m, k = (28_000 if kind == "few" else 31_003), 30_011
    deg = torch.randint(20, 53, (m,), device="cuda", generator=gen)
    if kind == "empty rows":
        deg[::7] = 0
        deg[1::7] += 24
    if kind == "long":
        deg[::500] = 256
    if kind == "cut":
        deg[::200] = torch.randint(257, 501, (deg[::200].numel(),), device="cuda", generator=gen)
    if kind == "around 64":
        deg += 40
    if kind == "hub":
        deg[17] = 12_000
    rp = torch.zeros(m + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(deg, 0)
    nnz = int(rp[-1])
    assert (nnz < 1 << 20) == (kind == "few")
    row = torch.repeat_interleave(torch.arange(m, device="cuda"), deg)
    ci = torch.randint(k, (nnz,), device="cuda", generator=gen)
    if kind == "local":
        ci = (row * k // m // 2000 * 2000 + ci % 2000).clamp(max=k - 1)
    ci = torch.sort(row * k + ci)[0] % k
    v = torch.randn(nnz, device="cuda", generator=gen)
    B = torch.randn(k, f, device="cuda", generator=gen)
    ci32 = ci.to(torch.int32)
    ws = sagnn.spmm_csr_prepare(rp, ci32, v, k, f)
    assert ws.info()["mode"] == (0 if kind in ("hub", "few") else 1)
    assert kind != "cut" or ws.info()["split_rows"] > 0
    ref = torch.zeros(m, f, dtype=torch.float64, device="cuda")
    size = torch.zeros_like(ref)
    for at in range(0, nnz, 1 << 18):
        s = slice(at, min(nnz, at + (1 << 18)))
        t = v[s, None].double() * B[ci[s]].double()
        ref.index_add_(0, row[s], t)
        size.index_add_(0, row[s], t.abs())
    # any order of a row's additions: at most its number of entries 2^-24 of the sum of the terms' sizes
    bound = (deg.double() + 2)[:, None] * 2.0**-24 * size
    C = sagnn.spmm_csr_tallskinny(rp, ci32, v, B, ws=ws)
    assert bool(((C.double() - ref).abs() <= bound).all())
    C0 = torch.randn(m, f, device="cuda", generator=gen)
    C2 = sagnn.spmm_csr_tallskinny(rp, ci32, v, B, C=C0.clone(), accumulate=True, ws=ws)
    assert bool(((C2.double() - ref - C0.double()).abs() <= bound + 2.0**-22 * (size + C0.abs().double())).all())
    W = torch.randn(f, 32, device="cuda", generator=gen)
    T, Z, _ = sagnn.gcn_layer_fwd(rp, ci32, v, B, W, act=sagnn.ACT_IDENTITY, ws=ws, want_h=False)
    assert torch.equal(T, C)
    Zn = Z
    if sagnn.gcn_layer_fwd_form(ws, f, 32, sagnn.GEMM_FP32) != 0:
        _, Zn, _ = sagnn.gcn_layer_fwd(rp, ci32, v, B, W, act=sagnn.ACT_IDENTITY, ws=ws, want_h=False, want_t=False)
    want, wsize = ref @ W.double(), size @ W.abs().double()
    for z in (Z, Zn):
        assert bool(((z.double() - want).abs() <= (deg.double()[:, None] + f + 4) * 2.0**-24 * wsize).all())


@pytest.mark.parametrize("f,n,more", [(24, 270_000, 280_000), (60, 180_000, 190_000)])
def test_spmm_workspace_of_a_matrix_with_more_rows_serves_one_with_fewer(f, n, more):
    """With more rows the copy of B to aligned rows does not pay and the workspace has no room for it; the matrix with
    fewer rows, which would be given a copy, goes without one in that room."""
    nnz = 6_000_000
    L = sagnn.lib()

    def size(m):
        b = ctypes.c_size_t(0)
        assert L.spmm_csr_workspace_bytes(m, nnz, f, ctypes.byref(b)) == 0
        return b.value

    assert size(more) < size(n)
    rng = np.random.default_rng(f)
    rowptr = np.concatenate([[0], np.cumsum(rng.multinomial(nnz, np.full(n, 1.0 / n)))]).astype(np.int32)
    rows = np.repeat(np.arange(n), np.diff(rowptr))
    colidx = rng.integers(0, n, size=nnz)
    colidx = colidx[np.lexsort((colidx, rows))].astype(np.int32)
    rp, ci, v, B = dev(rowptr), dev(colidx), dev(rng.standard_normal(nnz).astype(np.float32)), dev(synth.normal((n, f), f, synth.STREAM_H))
    ref = torch.sparse_csr_tensor(rp.long(), ci.long(), v.double(), (n, n)) @ B.double()
    zabs = torch.sparse_csr_tensor(rp.long(), ci.long(), v.double().abs(), (n, n)) @ B.double().abs()
    C, guard = torch.empty((n, f), device="cuda"), 4096
    stream = torch.cuda.current_stream().cuda_stream
    for schedule in (1, 2):
        opt = sagnn.SpmmOptions()
        opt.schedule = schedule
        buf = torch.full((size(more) + guard,), 0xA5, dtype=torch.uint8, device="cuda")
        args = (rp.data_ptr(), ci.data_ptr(), v.data_ptr(), n, n, nnz)
        assert L.spmm_csr_prepare_opt(*args, f, buf.data_ptr(), size(more), ctypes.byref(opt), stream) == 0
        C.fill_(float("nan"))
        assert L.spmm_csr_tallskinny(*args, B.data_ptr(), f, f, C.data_ptr(), f, 0, buf.data_ptr(), size(more), stream) == 0
        assert_close(C, ref.cpu().numpy(), zabs.cpu().numpy(), RTOL_SPMM, f"f={f} schedule {schedule}")
        assert bool((buf[size(more):] == 0xA5).all())
        assert L.spmm_csr_release(buf.data_ptr()) == 0


@pytest.mark.parametrize("f,labels", [(16, "order"), (100, "order"), (256, "order"), (64, "random"), (256, "random"), (64, "hubs")])
def test_spmm_sweep_with_and_without_locality_of_the_rows(f, labels):
    """The sweep of a matrix whose row order carries locality is dealt in many small windows, of others in few: communities
    in row order, the same degrees with columns that lie anywhere, or at the same few places for all rows.  Each with a
    hub row, empty rows and rows at the long-row threshold."""
    rng = np.random.default_rng(f)
    n, size = 150_000, 10_000
    deg = 16 + rng.exponential(14.0, size=n).astype(np.int64)
    deg[::1000] = 0
    deg[7] = 20_000
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    rows = np.repeat(np.arange(n), deg)
    if labels == "order":
        colidx = rows // size * size + rng.integers(0, size, size=rows.size)
    else:
        colidx = rng.integers(0, n if labels == "random" else n // 16, size=rows.size)
    colidx = colidx[np.lexsort((colidx, rows))].astype(np.int32)
    val = rng.standard_normal(colidx.size).astype(np.float32)
    B = synth.normal((n, f), f, synth.STREAM_H)
    rp, ci, v = dev(rowptr), dev(colidx), dev(val)

    ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
    assert ws.info()["mode"] == 1
    got = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(B), ws=ws)
    ref = torch.sparse_csr_tensor(rp.long(), ci.long(), v.double(), (n, n)) @ dev(B).double()
    zabs = torch.sparse_csr_tensor(rp.long(), ci.long(), v.double().abs(), (n, n)) @ dev(B).double().abs()
    assert_close(got, ref.cpu().numpy(), zabs.cpu().numpy(), RTOL_SPMM, f"f={f} {labels}")


@pytest.mark.parametrize("f,n,deg,parts", [(16, 300_011, 18, 50), (24, 300_011, 18, 50), (64, 300_011, 18, 50), (100, 150_001, 24, 40),
                                           (128, 150_001, 24, 40), (256, 100_003, 24, 64), (256, 70_001, 40, 1000)])
def test_spmm_runs_of_workgroups_for_each_xcd(f, n, deg, parts):
    """Small communities in row order: the workgroups of two generations are shared out among the XCDs in runs.  More rows
    than two generations hold and counts of workgroups that are no multiple of eight; product, accumulation, layer."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(f + n)
    count = torch.randint(deg - 2, deg + 9, (n,), device="cuda", generator=gen)
    count[::977] = 0
    count[5::1234] = 3
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(count, 0)
    nnz, part = int(rp[-1]), n // parts
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), count)
    col = (row // part * part + torch.randint(part, (nnz,), device="cuda", generator=gen)).clamp(max=n - 1)
    ci = (torch.sort(row * n + col)[0] - row * n).to(torch.int32)
    v = torch.randn(nnz, device="cuda", generator=gen)
    B = torch.randn(n, f, device="cuda", generator=gen)
    ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
    assert ws.info()["mode"] == 1
    A, Aabs = (torch.sparse_csr_tensor(rp.long(), ci.long(), x.double(), (n, n)) for x in (v, v.abs()))
    ref, zabs = A @ B.double(), Aabs @ B.double().abs()
    C0 = torch.randn(n, f, device="cuda", generator=gen)
    for C in (None, C0.clone()):
        want, scale = (ref, zabs) if C is None else (ref + C.double(), zabs + C.double().abs())
        got = sagnn.spmm_csr_tallskinny(rp, ci, v, B, C=C, accumulate=C is not None, ws=ws)
        assert float(((got.double() - want).abs() - RTOL_SPMM * scale).max()) <= 1e-30, f"f={f} accumulate={C is not None}"
    W = torch.randn(f, 40, device="cuda", generator=gen) / f ** 0.5
    _, Z, _ = sagnn.gcn_layer_fwd(rp, ci, v, B, W, ws=ws, want_t=sagnn.gcn_layer_fwd_form(ws, f, 40) != 2)
    # (the rows of A H, then f products and sums in 32 bits)
    bound = (RTOL_SPMM + f * 2.0 ** -24) * (zabs @ W.double().abs())
    assert float(((Z.double() - ref @ W.double()).abs() - bound).max()) <= 1e-30


@pytest.mark.parametrize("f", [4, 8, 12, 20, 28, 36, 60])
def test_spmm_sweep_of_narrow_widths_between_the_kernels_is_closer_than_one_sum(f, monkeypatch):
    """Rows whose 120 entries lie in one slab of B and are one segment: at the widths below 64 that no kernel has exactly,
    the error against 64 bits is well below that of one fused multiply-add after the other (root mean squares of the
    partial sums: sqrt(1400) against sqrt(7260), 0.44)."""
    for name, value in (("", 1), ("_MINDEG", 16), ("_GROUPS", 2)):
        monkeypatch.setenv("SAGNN_SWEEP" + name, str(value))
    m, n, d = 20_011, 4_000, 120
    gen = torch.Generator(device="cuda").manual_seed(f)
    ci = torch.randint(n // 8, (m, d), device="cuda", generator=gen, dtype=torch.int32).sort(1).values
    ci += torch.arange(m, device="cuda", dtype=torch.int32)[:, None] % 8 * (n // 8)
    v = torch.full((m, d), 1.0 / d, device="cuda")
    B = torch.randn(n, f, device="cuda", generator=gen)
    exact, serial = torch.zeros(m, f, device="cuda", dtype=torch.double), torch.zeros(m, f, device="cuda")
    for j in range(d):
        term = v[:, j:j + 1].double() * B[ci[:, j].long()].double()
        exact += term
        serial = (serial.double() + term).float()
    rp = torch.arange(m + 1, device="cuda", dtype=torch.int32) * d
    args = rp, ci.reshape(-1), v.reshape(-1)
    ws = sagnn.spmm_csr_prepare(*args, n, f)
    assert ws.info()["mode"] == 1
    got = sagnn.spmm_csr_tallskinny(*args, B, ws=ws)
    assert float((got.double() - exact).norm()) < 0.6 * float((serial.double() - exact).norm())


@pytest.mark.parametrize("f", [4, 12, 16, 20, 28, 32])
def test_spmm_narrow_sweep_short_rows_as_whole_rows(f, monkeypatch):
    """Eight and sixteen lane groups sweep short rows as whole rows too: rows of 1 to 63 entries and around the steps of a
    batch, unsorted and repeated columns in them, hubs, empty rows; plain, accumulating, and with infinite rows of B, which
    reach the rows that use them and no other (streams of a wavefront end at different steps)."""
    monkeypatch.setenv("SAGNN_SWEEP", "1")
    monkeypatch.setenv("SAGNN_SWEEP_PIECE", "1024")
    monkeypatch.setenv("SAGNN_SWEEP_SLAB_MB", "0")
    monkeypatch.setenv("SAGNN_SWEEP_MINDEG", "64")
    monkeypatch.setenv("SAGNN_SWEEP_GROUPS", "2")     # (whatever the uses of a row of B)
    rng = np.random.default_rng(700 + f)
    n = 30_000
    deg = rng.choice([0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 33, 62, 63, 64, 65, 200], size=7001)
    deg[[3, 7, 2500]] = 9000, 3000, 1025
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    colidx = rng.integers(0, n, size=rowptr[-1]).astype(np.int32)
    for r in np.flatnonzero(deg >= 64):
        colidx[rowptr[r]:rowptr[r + 1]].sort()
    val = rng.uniform(0.5, 1.5, size=colidx.size).astype(np.float32)
    B = np.abs(synth.normal((n, f), f, synth.STREAM_H)) + np.float32(0.1)
    rp, ci, v = dev(rowptr), dev(colidx), dev(val)
    ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
    info = ws.info()
    assert info["mode"] == 1 and info["groups"] in (8, 16) and info["chunk_rows"] == 0 and info["split_rows"] >= 3, info
    infinite = rng.random(n) < 0.02
    infinite[0] = True                                # what padding multiplies by 0
    hit = np.bincount(np.repeat(np.arange(deg.size), deg)[infinite[colidx]], minlength=deg.size) > 0
    for C0 in (None, synth.normal((deg.size, f), f + 1, synth.STREAM_G)):
        ref, zabs = oracle.spmm(rowptr, colidx, val, B, C=C0, want_abs=True)
        C = None if C0 is None else dev(C0)
        got = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(B), C=C, accumulate=C0 is not None, ws=ws)
        assert_close(got, ref, zabs, RTOL_SPMM, f"f={f}")
        Binf = B.copy()
        Binf[infinite] = np.inf
        C = None if C0 is None else dev(C0)
        got = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(Binf), C=C, accumulate=C0 is not None, ws=ws).cpu().numpy()
        assert np.isposinf(got[hit]).all()
        assert_close(got[~hit], ref[~hit], zabs[~hit], RTOL_SPMM, f"f={f} beside infinite rows")


@pytest.mark.parametrize("f,longest", [(16, range(600, 1800, 40)), (24, range(1600, 3600, 60)), (32, range(1600, 3600, 60))])
def test_spmm_narrow_sweep_where_padded_short_rows_do_not_fit(f, longest, monkeypatch):
    """The streams of eight and sixteen lane groups are padded to the longest of a wavefront, here by one long row more and
    more.  Short rows are swept whole, then, where their padding is what no longer fits, the preparation is made again with
    them beside the sweep, then nothing is swept.  The second preparation is the one without whole short rows, bit for bit."""
    monkeypatch.setenv("SAGNN_SWEEP", "1")
    monkeypatch.setenv("SAGNN_SWEEP_MINDEG", "64")
    monkeypatch.setenv("SAGNN_SWEEP_GROUPS", "2")
    rng = np.random.default_rng(f)
    n, short = 5000, 300
    B = synth.normal((n, f), f, synth.STREAM_H)
    met = []
    for x in longest:
        deg = rng.permutation(np.concatenate([[x], np.full(159, 64), np.ones(short)])).astype(np.int64)
        rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
        colidx = np.concatenate([np.sort(rng.choice(n, size=d, replace=False)) for d in deg]).astype(np.int32)
        val = rng.standard_normal(colidx.size).astype(np.float32)
        rp, ci, v = dev(rowptr), dev(colidx), dev(val)
        ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
        got = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(B), ws=ws)
        ref, zabs = oracle.spmm(rowptr, colidx, val, B, want_abs=True)
        assert_close(got, ref, zabs, RTOL_SPMM, f"f={f}, longest row {x}")
        info = ws.info()
        met.append("plain" if info["mode"] == 0 else ("beside" if info["chunk_rows"] else "whole"))
        if met[-1] == "beside":
            assert info["chunk_rows"] == short and info["groups"] == (16 if f == 16 else 8)
            with monkeypatch.context() as apart:
                apart.setenv("SAGNN_SWEEP_SHORT_ROWS", "-1")
                ws2 = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
            assert ws2.info() == info
            assert torch.equal(sagnn.spmm_csr_tallskinny(rp, ci, v, dev(B), ws=ws2), got)
    assert met == sorted(met, key=["whole", "beside", "plain"].index) and set(met) == {"whole", "beside", "plain"}, met


@pytest.mark.parametrize("f", [64, 128, 192, 256])
@pytest.mark.parametrize("groups", [1, 2])
def test_spmm_sweep_short_rows_as_whole_rows(f, groups, monkeypatch):
    """Option short_rows: the rows below the long-row threshold are swept as whole rows, 16 per
    wavefront, instead of going through the nonzero-splitting kernel (no compacted short-row CSR is
    left).  Most rows of this matrix are short, their columns are not sorted and may repeat; long
    rows are ascending as the sweep requires; hubs are cut into pieces; some rows are empty."""
    monkeypatch.setenv("SAGNN_SWEEP", "1")
    monkeypatch.setenv("SAGNN_SWEEP_PIECE", "1024")
    monkeypatch.setenv("SAGNN_SWEEP_SLAB_MB", "0")
    monkeypatch.setenv("SAGNN_SWEEP_MINDEG", "64")
    monkeypatch.setenv("SAGNN_SWEEP_GROUPS", str(groups))
    rng = np.random.default_rng(300 + f + groups)
    m, n = 7001, 30_000
    rowptr, colidx, val = random_csr(m, n, 22, rng, empty_frac=0.1, dup=True,
                                     hubs=[(3, 9000), (7, 3000), (2500, 1025), (5002, 64), (11, 63), (12, 1),
                                           (7000, 200)])
    for r in range(m):
        a, b = rowptr[r], rowptr[r + 1]
        if b - a >= 64:
            o = np.argsort(colidx[a:b], kind="stable")
            colidx[a:b], val[a:b] = colidx[a:b][o], val[a:b][o]
    B = synth.normal((n, f), f, synth.STREAM_H)
    ref, zabs = oracle.spmm(rowptr, colidx, val, B, want_abs=True)
    rp, ci, v = dev(rowptr), dev(colidx), dev(val)
    ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
    info = ws.info()
    assert info["mode"] == 1 and info["chunk_rows"] == 0 and info["chunk_entries"] == 0, info
    assert info["split_rows"] >= 3 and info["has_empty_rows"] == 1
    C0 = torch.full((m, f), float("nan"), device="cuda")
    got = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(B), C=C0, ws=ws)
    torch.cuda.synchronize()
    assert_close(got, ref, zabs, RTOL_SPMM, f"whole-row sweep f={f} groups={groups}")
    Cacc = synth.normal((m, f), f + 1, synth.STREAM_G)
    ref2, zabs2 = oracle.spmm(rowptr, colidx, val, B, C=Cacc, want_abs=True)
    got2 = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(B), C=dev(Cacc), accumulate=True, ws=ws)
    torch.cuda.synchronize()
    assert_close(got2, ref2, zabs2, RTOL_SPMM, f"whole-row sweep accumulate f={f} groups={groups}")
    if f in (64, 128, 256):
        # every row ends in a wavefront of the sweep: the layer takes the sweep-epilogue form
        fout = 96
        W = synth.normal((f, fout), 5, synth.STREAM_W, scale=1 / np.sqrt(f))
        for prec in (0, 1, 2):
            assert sagnn.gcn_layer_fwd_form(ws, f, fout, prec) == 2
            o = oracle.gcn_layer_fwd(rowptr, colidx, val, B, W, act=1, bf16=(prec == 1))
            Z0 = torch.full((m, fout), float("nan"), device="cuda")
            H0 = torch.full((m, fout), float("nan"), device="cuda")
            _, Z, Ho = sagnn.gcn_layer_fwd(rp, ci, v, dev(B), dev(W), act=sagnn.ACT_RELU, prec=prec, ws=ws,
                                           want_t=False, out=(None, Z0, H0))
            torch.cuda.synchronize()
            rtol = RTOL_BF16 if prec == 1 else RTOL_GEMM_FP32
            assert_close(Z, o["Z"], o["Zabs"], rtol, f"whole-row sweep layer Z f={f} prec={prec}")
            assert_close(Ho, o["H"], o["Zabs"], rtol, f"whole-row sweep layer H' f={f} prec={prec}")


@pytest.mark.parametrize("variant", ["sixteen_pieces_per_wavefront", "many_small_windows", "snake_dealing",
                                     "one_window_long_threshold_64", "one_row_per_instruction"])
def test_spmm_slab_sweep_planner_variants(variant, force_sweep, monkeypatch):
    """The planner's alternatives (pieces per wavefront, dealing windows, dealing order,
    thresholds) all have to give the same product; small inputs take them through the
    environment overrides the experiments use."""
    if variant == "sixteen_pieces_per_wavefront":
        monkeypatch.setenv("SAGNN_SWEEP_MIN_WAVES", "1")
    elif variant == "many_small_windows":
        monkeypatch.setenv("SAGNN_SWEEP_MIN_WAVES", "64")
        monkeypatch.setenv("SAGNN_SWEEP_WINDOW_PCT", "1")
    elif variant == "snake_dealing":
        monkeypatch.setenv("SAGNN_SWEEP_MIN_WAVES", "1")
        monkeypatch.setenv("SAGNN_SWEEP_LPT", "0")
        monkeypatch.setenv("SAGNN_SWEEP_GROUPS", "1")   # snake dealing exists for one stream per wavefront
    elif variant == "one_row_per_instruction":
        monkeypatch.setenv("SAGNN_SWEEP_GROUPS", "1")
    else:
        monkeypatch.setenv("SAGNN_SWEEP_MINDEG", "64")
        monkeypatch.setenv("SAGNN_SWEEP_WINDOW_PCT", "0")
        monkeypatch.setenv("SAGNN_SWEEP_SLAB_MB", "1")
    f = 128
    rng = np.random.default_rng(77)
    m, n = 9001, 50_000
    rowptr, colidx, val = random_csr(m, n, 30, rng, empty_frac=0.05,
                                     hubs=[(0, 20000), (1, 4097), (4500, 2048), (9000, 700), (17, 64), (18, 63)])
    B = synth.normal((n, f), 3, synth.STREAM_H)
    ref, zabs = oracle.spmm(rowptr, colidx, val, B, want_abs=True)
    got = run_spmm(rowptr, colidx, val, B, True, expect_mode=1)
    assert_close(got, ref, zabs, RTOL_SPMM, f"sweep planner variant {variant}")
    C0 = synth.normal((m, f), 4, synth.STREAM_G)
    ref2, zabs2 = oracle.spmm(rowptr, colidx, val, B, C=C0, want_abs=True)
    assert_close(run_spmm(rowptr, colidx, val, B, True, C0=C0), ref2, zabs2, RTOL_SPMM, f"{variant} accumulate")


@pytest.mark.parametrize("f", [128, 64, 256])
def test_spmm_sweep_planner_balances_streams(f, monkeypatch):
    """The device planner deals pieces longest-first to the shortest stream in batches; its longest
    stream must be as short as the one of the sequential piece-by-piece rule, computed here with a
    heap on the sizes the planner cuts (rows of >= 64 entries in pieces of <= 4096, strided).
    Heavy-tailed degrees make the rule matter: dealing in whole rounds would leave the streams
    that got the largest pieces first ~30 % longer than the average."""
    import heapq
    monkeypatch.setenv("SAGNN_SWEEP", "1")
    monkeypatch.setenv("SAGNN_SWEEP_MINDEG", "64")
    monkeypatch.setenv("SAGNN_SWEEP_MIN_WAVES", "1")          # all 16 slots of a wavefront
    monkeypatch.setenv("SAGNN_SWEEP_SHORT_ROWS", "-1")        # the streams of the long rows only
    rng = np.random.default_rng(9)
    m, n = 30_000, 200_000
    deg = np.minimum((64 / rng.random(m) ** 0.8).astype(np.int64), 30_000)   # heavy tail from 64 up
    deg[rng.random(m) < 0.3] = 5                                              # some short rows
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    nnz = int(rowptr[-1])
    colidx = np.empty(nnz, np.int32)
    for r in range(m):
        colidx[rowptr[r]:rowptr[r + 1]] = np.sort(rng.integers(0, n, size=deg[r]))
    val = np.ones(nnz, np.float32)
    ws = sagnn.spmm_csr_prepare(dev(rowptr), dev(colidx), dev(val), n, f)
    info = ws.info()
    assert info["mode"] == 1 and info["sweep_entries"] + info["chunk_entries"] == nnz
    R = info["groups"]
    sizes = []
    for d in deg[deg >= 64]:
        p = -(-int(d) // 4096)
        sizes += [(int(d) - j + p - 1) // p for j in range(p)]
    sizes.sort(reverse=True)
    assert info["sweep_entries"] == sum(sizes)
    n_waves = -(-len(sizes) // 16)        # as few wavefronts as the 16 slots allow (the launch rounds up to 4)
    assert n_waves <= info["sweep_waves"] < n_waves + 4
    units, per_unit = n_waves * R, 16 // R
    heap = [(0, u) for u in range(units)]
    used = [0] * units
    longest = 0
    for sz in sizes:
        load, u = heapq.heappop(heap)
        load += sz
        used[u] += 1
        longest = max(longest, load)
        if used[u] < per_unit:
            heapq.heappush(heap, (load, u))
    # the library counts steps of wavefronts (the longer of a wavefront's group streams, in whole
    # batches of 8): allow that rounding and 3 % on top
    assert info["longest_stream_steps"] <= 1.03 * longest + 8, (info, longest, sum(sizes) / units)
    # and the product is right
    B = synth.normal((n, f), 5, synth.STREAM_H)
    rows = rng.choice(m, size=200, replace=False)
    got = sagnn.spmm_csr_tallskinny(dev(rowptr), dev(colidx), dev(val), dev(B), ws=ws)
    torch.cuda.synchronize()
    rows.sort()
    sub_deg = deg[rows]
    sub_rowptr = np.concatenate([[0], np.cumsum(sub_deg)]).astype(np.int32)
    sub_idx = np.concatenate([np.arange(rowptr[r], rowptr[r + 1]) for r in rows])
    ref, zabs = oracle.spmm(sub_rowptr, colidx[sub_idx], val[sub_idx], B, want_abs=True)
    assert_close(got[torch.from_numpy(rows).cuda()], ref, zabs, RTOL_SPMM, f"balanced planner f={f}")


@pytest.mark.parametrize("groups", [1, 2])
@pytest.mark.parametrize("min_waves", [1, 16])
def test_spmm_sweep_planner_deals_few_pieces(groups, min_waves, force_sweep, monkeypatch):
    """The batches that meet empty streams are dealt without a sort: two and three wavefronts' streams with about as many
    pieces as they have slots, one or four streams a wavefront."""
    monkeypatch.setenv("SAGNN_SWEEP_GROUPS", str(groups))
    monkeypatch.setenv("SAGNN_SWEEP_MIN_WAVES", str(min_waves))
    monkeypatch.setenv("SAGNN_SWEEP_SHORT_ROWS", "-1")
    f, n = 64, 5000
    B = synth.normal((n, f), 3, synth.STREAM_H)
    for rows in (31, 32, 33, 47, 48, 49, 64, 65, 513):
        rng = np.random.default_rng(rows)
        rowptr, colidx, val = random_csr(rows, n, 0, rng, hubs=[(r, 64 + int(rng.integers(0, 200))) for r in range(rows)])
        ref, zabs = oracle.spmm(rowptr, colidx, val, B, want_abs=True)
        got = run_spmm(rowptr, colidx, val, B, True, expect_mode=1)
        assert_close(got, ref, zabs, RTOL_SPMM, f"{rows} long rows, {groups}")


@pytest.mark.parametrize("slab_mb", ["0", "1"])
@pytest.mark.parametrize("at", [-1, 0, 999, 1000, 2500, 4998])
def test_spmm_sweep_reads_every_pair_of_a_row(slab_mb, at, force_sweep, monkeypatch):
    """Rows whose ends lie around the 63 entries that a wavefront looks at at a time, and rows cut into five pieces whose shares
    are looked at apart: one descending pair anywhere is found, and without one the streams are right, with tables of many slabs
    (found again for the layout) and of few (left by the counting pass)."""
    monkeypatch.setenv("SAGNN_SWEEP_SLAB_MB", slab_mb)
    rng = np.random.default_rng(13)
    m, n, f = 600, 20_000, 64
    ends = [62, 63, 64, 125, 126, 127, 128, 189, 251, 252, 253]
    rowptr, colidx, val = random_csr(m, n, 20, rng, hubs=[(5, 5000), (300, 5000)] + [(20 + r, ends[r % 11]) for r in range(200)])
    for r in (5, 300):                                        # distinct columns
        colidx[rowptr[r]:rowptr[r] + 5000] = np.sort(rng.choice(n, 5000, replace=False))
    if at >= 0:
        e = rowptr[300] + at
        colidx[[e, e + 1]] = colidx[[e + 1, e]]
    B = synth.normal((n, f), 1, synth.STREAM_H)
    ref, zabs = oracle.spmm(rowptr, colidx, val, B, want_abs=True)
    got = run_spmm(rowptr, colidx, val, B, True, expect_mode=1 if at < 0 else 0)
    assert_close(got, ref, zabs, RTOL_SPMM, f"descending pair at {at}")


@pytest.mark.parametrize("f", [192, 256, 320])
def test_spmm_sweep_wide_operand_as_128_wide_slabs(f, force_sweep, monkeypatch):
    """Operands wider than 128 taken as 128-wide column slabs (plus a 64-wide rest) by the kernels
    that fetch two rows of B per load: same product."""
    monkeypatch.setenv("SAGNN_SWEEP_SLAB_WIDTH", "128")
    rng = np.random.default_rng(f + 1)
    m, n = 6001, 40_000
    rowptr, colidx, val = random_csr(m, n, 25, rng, empty_frac=0.1,
                                     hubs=[(4, 7000), (9, 2049), (3000, 1024), (6000, 33)])
    B = synth.normal((n, f), f, synth.STREAM_H)
    ref, zabs = oracle.spmm(rowptr, colidx, val, B, want_abs=True)
    rp, ci, v = dev(rowptr), dev(colidx), dev(val)
    ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
    info = ws.info()
    assert info["mode"] == 1 and info["groups"] == 2
    got = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(B), ws=ws)
    torch.cuda.synchronize()
    assert_close(got, ref, zabs, RTOL_SPMM, f"128-wide slabs f={f}")
    C0 = synth.normal((m, f), f + 2, synth.STREAM_G)
    ref2, zabs2 = oracle.spmm(rowptr, colidx, val, B, C=C0, want_abs=True)
    got2 = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(B), C=dev(C0), accumulate=True, ws=ws)
    torch.cuda.synchronize()
    assert_close(got2, ref2, zabs2, RTOL_SPMM, f"128-wide slabs accumulate f={f}")
    # a narrower call on the same workspace (the streams serve 128- and 64-wide launches)
    B64 = synth.normal((n, 64), 3, synth.STREAM_H)
    ref3, zabs3 = oracle.spmm(rowptr, colidx, val, B64, want_abs=True)
    got3 = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(B64), ws=ws)
    torch.cuda.synchronize()
    assert_close(got3, ref3, zabs3, RTOL_SPMM, f"128-wide slabs prepared {f}, called 64")


def test_spmm_sweep_workspace_prepared_for_wider_f(force_sweep):
    """A workspace prepared for f = 128 (two lane groups) or 256 also serves narrower calls."""
    rng = np.random.default_rng(31)
    m, n = 3000, 30_000
    rowptr, colidx, val = random_csr(m, n, 25, rng, hubs=[(2, 6000), (1500, 1500)])
    rp, ci, v = dev(rowptr), dev(colidx), dev(val)
    for f_prep, f_call in ((128, 64), (256, 128), (256, 64), (192, 128)):
        ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f_prep)
        assert ws.info()["mode"] == 1
        B = synth.normal((n, f_call), f_prep + f_call, synth.STREAM_H)
        ref, zabs = oracle.spmm(rowptr, colidx, val, B, want_abs=True)
        got = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(B), ws=ws)
        torch.cuda.synchronize()
        assert_close(got, ref, zabs, RTOL_SPMM, f"prepared {f_prep}, called {f_call}")


def test_spmm_slab_sweep_falls_back_on_unsorted_rows(force_sweep):
    rng = np.random.default_rng(5)
    m, n, f = 2000, 30_000, 128
    rowptr, colidx, val = random_csr(m, n, 40, rng, hubs=[(5, 5000)], dup=True)   # unsorted rows
    B = synth.normal((n, f), 1, synth.STREAM_H)
    ref, zabs = oracle.spmm(rowptr, colidx, val, B, want_abs=True)
    assert_close(run_spmm(rowptr, colidx, val, B, True, expect_mode=0), ref, zabs, RTOL_SPMM, "unsorted fallback")
    bad = colidx.copy()
    rowptr2, colidx2, val2 = random_csr(m, n, 40, rng, hubs=[(5, 5000)])
    colidx2[rowptr2[5] + 4999] = n + 7                        # out-of-range column in a long row
    ref, zabs = oracle.spmm(rowptr2, np.minimum(colidx2, n - 1), val2, B, want_abs=True)
    assert_close(run_spmm(rowptr2, colidx2, val2, B, True, expect_mode=0), ref, zabs, RTOL_SPMM, "clamped column")
    _ = bad


def _strided(a, pad, fill):
    """Device matrix whose rows are `pad` floats apart wider than a's: returns (view, whole)."""
    m, f = a.shape
    whole = torch.full((m, f + pad), fill, dtype=torch.float32, device="cuda")
    whole[:, :f] = dev(a)
    return whole[:, :f], whole


@pytest.mark.parametrize("schedule", ["no_workspace", "nonzero_splitting", "sweep", "sweep_one_row_per_load"])
@pytest.mark.parametrize("f", [16, 32, 48, 64, 100, 128, 192, 256, 320])
def test_spmm_leading_dimensions_wider_than_f(f, schedule, monkeypatch):
    """B and C as column slices of wider matrices (ldb = f + 4, ldc = f + 8), overwrite and
    accumulate; the padding columns of C must come back untouched."""
    if schedule.startswith("sweep"):
        if f not in (16, 32, 64, 128, 192, 256, 320) or (schedule == "sweep_one_row_per_load" and f < 64):
            pytest.skip("no such kernel at this width")
        monkeypatch.setenv("SAGNN_SWEEP", "1")
        monkeypatch.setenv("SAGNN_SWEEP_MINDEG", "16")
        monkeypatch.setenv("SAGNN_SWEEP_PIECE", "1024")
        monkeypatch.setenv("SAGNN_SWEEP_SLAB_MB", "0")
        monkeypatch.setenv("SAGNN_SWEEP_GROUPS", "1" if schedule == "sweep_one_row_per_load" else "2")
    else:
        monkeypatch.setenv("SAGNN_SWEEP", "0")
    rng = np.random.default_rng(1000 + f)
    m, n = 4001, 30_000
    rowptr, colidx, val = random_csr(m, n, 18, rng, empty_frac=0.1,
                                     hubs=[(3, 7000), (9, 2049), (2000, 1024), (4000, 100), (17, 16)])
    B = synth.normal((n, f), f, synth.STREAM_H)
    C0 = synth.normal((m, f), f + 1, synth.STREAM_G)
    rp, ci, v = dev(rowptr), dev(colidx), dev(val)
    Bv, _ = _strided(B, 4, 123.0)
    ws = None
    if schedule != "no_workspace":
        ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
        assert ws.info()["mode"] == (1 if schedule.startswith("sweep") else 0), ws.info()
    for acc in (False, True):
        ref, zabs = oracle.spmm(rowptr, colidx, val, B, C=C0 if acc else None, want_abs=True)
        Cv, Cw = _strided(C0, 8, -77.0)
        sagnn.spmm_csr_tallskinny(rp, ci, v, Bv, C=Cv, accumulate=acc, ws=ws)
        torch.cuda.synchronize()
        assert_close(Cv, ref, zabs, RTOL_SPMM, f"strided f={f} {schedule} accumulate={acc}")
        assert torch.all(Cw[:, f:] == -77.0)


@pytest.mark.parametrize("case", ["f128_lane_groups", "f128_one_row_per_load", "f256_one_row_per_load", "f64_quarter_groups",
                                  "f32_perm", "f16_perm", "f128_nonzero_splitting", "f128_no_workspace",
                                  "f100_slabs_and_remainder"])
def test_spmm_operand_larger_than_4gib(case, monkeypatch):
    """Rows of B beyond byte offset 2^32 (k * ldb * 4 > 2^32): the kernels cannot use 32-bit
    buffer offsets and switch to 64-bit addressing; every schedule has such a variant.  B is a
    4.6 GB allocation in which only the referenced rows are filled; the oracle multiplies by
    those rows alone (columns renumbered), which is the same product."""
    f = int(case[1:case.index("_")])
    ld = 256 if f > 128 else 128
    k = (9_000_000 * 128) // ld
    sweep = not ("nonzero" in case or "no_workspace" in case or "slabs" in case)
    monkeypatch.setenv("SAGNN_SWEEP", "1" if sweep else "0")
    if sweep:
        monkeypatch.setenv("SAGNN_SWEEP_MINDEG", "16")
        monkeypatch.setenv("SAGNN_SWEEP_PIECE", "1024")
        monkeypatch.setenv("SAGNN_SWEEP_SLAB_MB", "64")
        monkeypatch.setenv("SAGNN_SWEEP_GROUPS", "1" if "one_row" in case else "2")
    rng = np.random.default_rng(len(case) + f)
    m = 3000
    rowptr, colidx, val = random_csr(m, k, 14, rng, empty_frac=0.05, hubs=[(5, 6000), (70, 1500), (2999, 64)])
    # make sure both sides of the 2^32-byte line and the very last row are referenced
    line = (1 << 32) // (ld * 4)
    colidx[rowptr[5]:rowptr[5] + 6] = np.sort(np.array([0, line - 1, line, line + 1, k - 2, k - 1], np.int32))
    colidx[rowptr[5]:rowptr[6]].sort()
    ucols, inv = np.unique(colidx, return_inverse=True)
    assert ucols[-1] == k - 1 and (ucols.astype(np.int64) * ld * 4 >= (1 << 32)).sum() > 1000
    Bsmall = synth.normal((ucols.size, f), f, synth.STREAM_H)
    buf = torch.empty(9_000_000 * 128, dtype=torch.float32, device="cuda")
    Bfull = buf.view(k, ld)
    Bfull[torch.from_numpy(ucols.astype(np.int64)).cuda(), :f] = dev(Bsmall)
    Bv = Bfull[:, :f]
    rp, ci, v = dev(rowptr), dev(colidx), dev(val)
    ws = None if "no_workspace" in case else sagnn.spmm_csr_prepare(rp, ci, v, k, f)
    if ws is not None:
        assert ws.info()["mode"] == (1 if sweep else 0), ws.info()
    C0 = synth.normal((m, f), 5, synth.STREAM_G)
    for acc in (False, True):
        ref, zabs = oracle.spmm(rowptr, inv.astype(np.int32), val, Bsmall, C=C0 if acc else None, want_abs=True)
        Cv, Cw = _strided(C0, 8, -77.0)
        sagnn.spmm_csr_tallskinny(rp, ci, v, Bv, C=Cv, accumulate=acc, ws=ws)
        torch.cuda.synchronize()
        assert_close(Cv, ref, zabs, RTOL_SPMM, f"{case} accumulate={acc}")
        assert torch.all(Cw[:, f:] == -77.0)
    del buf, Bfull, Bv


def test_spmm_workspace_rejects_a_shorter_operand_and_release_forgets_it(monkeypatch):
    """A schedule prepared for k rows of B holds column ids up to k-1: a call with fewer rows is
    refused on the host (nothing launched).  After spmm_csr_release the address is unknown."""
    import ctypes
    monkeypatch.setenv("SAGNN_SWEEP", "1")
    rng = np.random.default_rng(8)
    m, n, f = 2000, 20_000, 128
    rowptr, colidx, val = random_csr(m, n, 30, rng, hubs=[(1, 4000)])
    rp, ci, v = dev(rowptr), dev(colidx), dev(val)
    B = dev(synth.normal((n, f), 1, synth.STREAM_H))
    for sweep in ("1", "0"):
        monkeypatch.setenv("SAGNN_SWEEP", sweep)
        ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
        with pytest.raises(ValueError):
            sagnn.spmm_csr_tallskinny(rp, ci, v, B[: n - 1], ws=ws)
        C = torch.zeros((m, f), device="cuda")
        L = sagnn.lib()
        args = lambda kk: (ctypes.c_void_p(rp.data_ptr()), ctypes.c_void_p(ci.data_ptr()), ctypes.c_void_p(v.data_ptr()),
                           m, kk, ci.numel(), ctypes.c_void_p(B.data_ptr()), f, f, ctypes.c_void_p(C.data_ptr()), f, 0,
                           ctypes.c_void_p(ws.buf.data_ptr()), ws.buf.numel(), None)
        assert L.spmm_csr_tallskinny(*args(n - 1)) == -1
        assert L.spmm_csr_tallskinny(*args(n)) == 0
        torch.cuda.synchronize()
        ptr = ctypes.c_void_p(ws.buf.data_ptr())
        keep = ws.buf
        assert L.spmm_csr_release(ptr) == 0
        assert L.spmm_csr_tallskinny(*args(n)) == -1           # unknown workspace now
        assert L.spmm_csr_release(ptr) == 0                    # releasing twice is harmless
        ws.buf = None
        del keep


@pytest.mark.parametrize("sweep", ["0", "1"])
@pytest.mark.parametrize("f", [16, 32, 64, 128, 256])
def test_spmm_long_rows_of_equal_terms_stay_within_tolerance(f, sweep, monkeypatch):
    """Rows whose products are all the same positive number are the worst case for fp32 rounding:
    every addition of a long serial sum rounds the same way, so the error grows with the length of
    the sum instead of its square root.  The kernels keep every serial run short; the result must
    stay within the SpMM tolerance of the exact value (here known in closed form)."""
    monkeypatch.setenv("SAGNN_SWEEP", sweep)
    rng = np.random.default_rng(f)
    n = 65_536
    # enough entries in long rows for the planner to keep the sweep at every width
    degs = np.concatenate([[60_000] * 8, [33_333] * 4, [4096, 4097, 9000], rng.integers(1, 40, size=3000)])
    rowptr = np.zeros(degs.size + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum(degs)
    colidx = np.concatenate([np.sort(rng.choice(n, size=int(d), replace=False)) for d in degs]).astype(np.int32)
    val = np.concatenate([np.full(int(d), np.float32(1.0 / math.sqrt(d))) for d in degs]).astype(np.float32)
    B = np.full((n, f), np.float32(math.sqrt(3.0)), dtype=np.float32)
    exact = degs.astype(np.float64) * val[rowptr[:-1]].astype(np.float64) * float(B[0, 0])
    got = run_spmm(rowptr, colidx, val, B, True, expect_mode=int(sweep)).cpu().numpy().astype(np.float64)
    rel = np.abs(got - exact[:, None]) / exact[:, None]
    assert rel.max() <= RTOL_SPMM, (rel.max(), int(rel.max(axis=1).argmax()))
    if sweep == "0":                                          # the kernel for calls without a workspace
        got = run_spmm(rowptr, colidx, val, B, False).cpu().numpy().astype(np.float64)
        rel = np.abs(got - exact[:, None]) / exact[:, None]
        assert rel.max() <= RTOL_SPMM, (rel.max(), int(rel.max(axis=1).argmax()))


def test_spmm_prepare_tuned_keeps_a_correct_plan(monkeypatch):
    """The tuned preparation tries several plan variants on the caller's operand; whichever it
    keeps has to give the product, in the buffer it wrote during tuning and in later calls.  A
    matrix too small for the sweep has nothing to vary and behaves like the plain preparation."""
    g = synth.rmat_graph(60_000, 4_000_000, 11)
    H = synth.normal((g.n, 128), 11, synth.STREAM_H)
    ref, zabs = oracle.spmm(g.rowptr, g.colidx, g.val, H, want_abs=True)
    rp, ci, v = dev(g.rowptr), dev(g.colidx), dev(g.val)
    monkeypatch.setenv("SAGNN_SWEEP", "1")
    C = torch.full((g.m, 128), float("nan"), device="cuda")
    ws = sagnn.spmm_csr_prepare_tuned(rp, ci, v, dev(H), C=C)
    torch.cuda.synchronize()
    assert ws.info()["mode"] == 1 and 0 <= ws.choice["variant"] < 5 and ws.choice["best_us"] > 0
    assert_close(C, ref, zabs, RTOL_SPMM, "product left by the tuning runs")
    got = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(H), ws=ws)
    torch.cuda.synchronize()
    assert_close(got, ref, zabs, RTOL_SPMM, f"tuned plan {ws.choice}")
    monkeypatch.setenv("SAGNN_SWEEP", "0")
    ws0 = sagnn.spmm_csr_prepare_tuned(rp, ci, v, dev(H))
    assert ws0.info()["mode"] == 0 and ws0.choice["variant"] == 0
    got0 = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(H), ws=ws0)
    torch.cuda.synchronize()
    assert_close(got0, ref, zabs, RTOL_SPMM, "plain schedule through the tuned entry point")


@pytest.mark.parametrize("f,n", [(16, 20_000), (32, 20_000), (64, 20_000), (64, 60_000)])
def test_spmm_prepare_tuned_goes_on_behind_a_variant_that_cannot_be_swept(f, n):
    """Rows of 60 to 92 entries: the default plan is swept, the variants whose threshold is 96 entries would leave no
    row to the sweep.  The tuned preparation keeps a plan that it has timed, on a small matrix and on one of 4.5 M entries."""
    gen = torch.Generator(device="cuda").manual_seed(f)
    deg = torch.randint(60, 93, (n,), device="cuda", generator=gen)
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(deg, 0)
    nnz = int(rp[-1])
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), deg)
    ci = (torch.sort(row * n + torch.randint(n, (nnz,), device="cuda", generator=gen))[0] % n).to(torch.int32)
    v, B = torch.randn(nnz, device="cuda", generator=gen), torch.randn(n, f, device="cuda", generator=gen)
    assert nnz >= 1 << 20 and sagnn.spmm_csr_prepare(rp, ci, v, n, f).info()["mode"] == 1
    ws = sagnn.spmm_csr_prepare_tuned(rp, ci, v, B)
    assert ws.info()["mode"] == 1 and ws.choice["best_us"] > 0
    C = sagnn.spmm_csr_tallskinny(rp, ci, v, B, ws=ws)
    ref = torch.sparse_csr_tensor(rp.long(), ci.long(), v.double(), (n, n)) @ B.double()
    size = torch.sparse_csr_tensor(rp.long(), ci.long(), v.double().abs(), (n, n)) @ B.double().abs()
    assert bool(((C.double() - ref).abs() <= (deg.double() + 2)[:, None] * 2.0**-24 * size).all())


def test_spmm_rmat_with_and_without_sweep(monkeypatch):
    g = synth.rmat_graph(60_000, 4_000_000, 9)
    H = synth.normal((g.n, 128), 9, synth.STREAM_H)
    ref, zabs = oracle.spmm(g.rowptr, g.colidx, g.val, H, want_abs=True)
    for mode in ("0", "1"):
        monkeypatch.setenv("SAGNN_SWEEP", mode)
        got = run_spmm(g.rowptr, g.colidx, g.val, H, True, expect_mode=int(mode))
        assert_close(got, ref, zabs, RTOL_SPMM, f"rmat sweep={mode}")


@pytest.mark.parametrize("case", ["all_empty", "single_entry", "one_long_row", "exact_chunk", "tail_empty"])
def test_spmm_degenerate(case):
    f, n = 128, 700
    rng = np.random.default_rng(1)
    if case == "all_empty":
        rowptr = np.zeros(11, np.int32); colidx = np.empty(0, np.int32); val = np.empty(0, np.float32)
    elif case == "single_entry":
        rowptr = np.array([0, 0, 1, 1], np.int32); colidx = np.array([699], np.int32); val = np.array([2.5], np.float32)
    elif case == "one_long_row":
        rowptr = np.array([0, 2000], np.int32); colidx = rng.integers(0, n, 2000).astype(np.int32)
        val = rng.standard_normal(2000).astype(np.float32)
    elif case == "exact_chunk":     # rows end exactly on chunk boundaries
        rowptr = np.array([0, 256, 512, 512, 1024], np.int32); colidx = rng.integers(0, n, 1024).astype(np.int32)
        val = rng.standard_normal(1024).astype(np.float32)
    else:
        rowptr = np.array([0, 300, 300, 300], np.int32); colidx = rng.integers(0, n, 300).astype(np.int32)
        val = rng.standard_normal(300).astype(np.float32)
    B = synth.normal((n, f), 9, synth.STREAM_H)
    ref, zabs = oracle.spmm(rowptr, colidx, val, B, want_abs=True)
    for use_ws in (True, False):
        got = torch.full((rowptr.size - 1, f), 7.0, device="cuda")     # stale contents must be overwritten
        rp = dev(rowptr)
        ci = dev(colidx) if colidx.size else torch.empty(0, dtype=torch.int32, device="cuda")
        va = dev(val) if val.size else torch.empty(0, device="cuda")
        ws = sagnn.spmm_csr_prepare(rp, ci, va, n, f) if use_ws else None
        sagnn.spmm_csr_tallskinny(rp, ci, va, dev(B), C=got, ws=ws)
        torch.cuda.synchronize()
        assert_close(got, ref, zabs, RTOL_SPMM, f"{case} ws={use_ws}")


def test_spmm_identity_and_ring_closed_forms():
    n, f = 1000, 128
    H = synth.normal((n, f), 4, synth.STREAM_H)
    rp = np.arange(n + 1, dtype=np.int32); ci = np.arange(n, dtype=np.int32); v = np.ones(n, np.float32)
    got = run_spmm(rp, ci, v, H, True)
    assert got.cpu().numpy().tobytes() == H.tobytes()
    g = synth.ring_graph(4096, 8)
    ones = np.ones((4096, 64), np.float32)
    got = run_spmm(g.rowptr, g.colidx, g.val, ones, True).cpu().numpy()
    assert np.all(got == 8.0)


def test_spmm_cfg1_blocks_through_packed_buffer(cfg1):
    """Configuration 1 end to end: plan -> pack -> SpMM with compact indices, per row block,
    equals the oracle's A_i * H; also the whole matrix as one block."""
    g, H = cfg1
    off = synth.block_offsets(g.n, 4)
    Hd = dev(H)
    for i in range(4):
        blk = g.row_block(int(off[i]), int(off[i + 1]))
        rp, ci, v = csr_dev(blk)
        plan = sagnn.spmm_plan_needed_rows(rp, ci, g.n, off)
        Hn = sagnn.spmm_pack_rows(Hd, plan.needed)
        ws = sagnn.spmm_csr_prepare(rp, plan.colidx_compact, v, plan.N, 16)
        Z = sagnn.spmm_csr_tallskinny(rp, plan.colidx_compact, v, Hn, ws=ws)
        torch.cuda.synchronize()
        ref, zabs = oracle.spmm(blk.rowptr, blk.colidx, blk.val, H, want_abs=True)
        assert_close(Z, ref, zabs, RTOL_SPMM, f"cfg1 block {i}")
        # block-by-block accumulation (Alg. 1 inner loop): Z += A_iq * H[NnzCols(i,q)]
        Zacc = torch.zeros_like(Z)
        comp = plan.colidx_compact.cpu().numpy()
        for q in range(4):
            keep = (blk.colidx >= off[q]) & (blk.colidx < off[q + 1])
            cnt = np.add.reduceat(keep.astype(np.int64), blk.rowptr[:-1]) * (np.diff(blk.rowptr) > 0)
            rpq = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32)
            ciq = (comp[keep] - plan.blk_off[q]).astype(np.int32)
            Hq = Hn[int(plan.blk_off[q]):int(plan.blk_off[q + 1])].contiguous()
            drp, dci, dva = dev(rpq), dev(ciq), dev(blk.val[keep])
            wsq = sagnn.spmm_csr_prepare(drp, dci, dva, Hq.shape[0], 16)
            sagnn.spmm_csr_tallskinny(drp, dci, dva, Hq, C=Zacc, accumulate=True, ws=wsq)
        torch.cuda.synchronize()
        assert_close(Zacc, ref, zabs, RTOL_SPMM, f"cfg1 block {i} accumulated")
    rp, ci, v = csr_dev(g)
    ws = sagnn.spmm_csr_prepare(rp, ci, v, g.n, 16)
    Z = sagnn.spmm_csr_tallskinny(rp, ci, v, Hd, ws=ws)
    ref, zabs = oracle.spmm(g.rowptr, g.colidx, g.val, H, want_abs=True)
    assert_close(Z, ref, zabs, RTOL_SPMM, "cfg1 whole")


@pytest.mark.parametrize("f", [16, 64, 128, 256])
def test_spmm_small_rmat(f):
    g = synth.rmat_graph(40_000, 2_000_000, 5)
    H = synth.normal((g.n, f), 5, synth.STREAM_H)
    ref, zabs = oracle.spmm(g.rowptr, g.colidx, g.val, H, want_abs=True)
    got = run_spmm(g.rowptr, g.colidx, g.val, H, True)
    assert_close(got, ref, zabs, RTOL_SPMM, f"rmat f={f}")
    # sqrt(d) is an eigenvector of the normalised adjacency matrix (closed form at any size)
    x = np.sqrt(np.diff(g.rowptr).astype(np.float64)).astype(np.float32)
    X = np.repeat(x[:, None], f, axis=1).copy()
    got = run_spmm(g.rowptr, g.colidx, g.val, X, True).cpu().numpy()
    assert np.allclose(got, X, rtol=2e-5, atol=0)


# ------------------------------------------------------------------------------------ GEMM / layer

@pytest.mark.parametrize("m,k,n", [(1, 32, 32), (31, 64, 96), (33, 128, 128), (1000, 160, 256), (4097, 256, 64),
                                   (77, 16, 16), (500, 20, 100), (129, 100, 44), (64, 4, 4)])
@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("transW", [False, True])
def test_dense_gemm(m, k, n, prec, transW):
    X = synth.normal((m, k), m, synth.STREAM_H)
    W = synth.normal((n, k) if transW else (k, n), k, synth.STREAM_W, scale=1 / np.sqrt(k))
    if prec == 1:
        X.reshape(-1)[:4] = [1.0 + 2.0 ** -8, 1.0 + 3 * 2.0 ** -8, -(1.0 + 2.0 ** -8), 1.0 + 2.0 ** -8 + 2.0 ** -20][:min(4, X.size)]
    mask = synth.normal((m, n), n, synth.STREAM_G)
    ref, zabs = oracle.gemm(X, W, bf16=(prec == 1), transW=transW, want_abs=True)
    rtol = RTOL_BF16 if prec == 1 else RTOL_GEMM_FP32
    Z, A = sagnn.dense_gemm_act(dev(X), dev(W), transW=transW, prec=prec, act=sagnn.ACT_RELU, want_z=True, want_act=True)
    torch.cuda.synchronize()
    assert_close(Z, ref, zabs, rtol, "gemm Z")
    assert torch.equal(A, torch.clamp_min(Z, 0))
    Zm, _ = sagnn.dense_gemm_act(dev(X), dev(W), transW=transW, prec=prec, mask=dev(mask))
    torch.cuda.synchronize()
    assert_close(Zm, np.where(mask > 0, ref, 0), zabs, rtol, "gemm masked")
    assert torch.equal(Zm == 0, (dev(mask) <= 0) | (Z == 0))


@pytest.mark.parametrize("prec", [sagnn.GEMM_FP32, sagnn.GEMM_BF16, sagnn.GEMM_FP32_BF16X3])
@pytest.mark.parametrize("m,k,n", [(31, 4, 4), (32, 32, 32), (33, 36, 36), (95, 64, 100), (64, 68, 132), (97, 96, 128), (70, 100, 20),
                                   (65, 124, 256), (64, 128, 200), (40, 132, 64), (96, 160, 256), (33, 252, 12), (64, 256, 252)])
def test_dense_gemm_at_the_edges_of_its_groups_and_slabs(m, k, n, prec):
    """Every number of 32-wide k groups, full and ragged; full and ragged column slabs; rows that fill their last tile
    and rows that do not.  What lies beyond X's and W's columns is NaN, W begins anywhere and has an odd leading
    dimension; with and without mask, both outputs."""
    gen = torch.Generator().manual_seed(1000 * k + n)
    X = torch.randn(m, k, generator=gen)
    W = torch.randn(k, n, generator=gen)
    mask = torch.randint(-1, 2, (m, n), generator=gen).float()
    ref = X.double() @ W.double()
    # any order of k fp32 additions: k 2^-24 of the sum of the terms' sizes; both operands rounded to bfloat16: 2 2^-9
    tol = (2 * 2.0**-9 if prec == sagnn.GEMM_BF16 else 2 * 2.0**-23) + (k + 2) * 2.0**-24
    bound = tol * (X.abs().double() @ W.abs().double())

    def inside(t, wide, off):
        out = torch.full((t.shape[0], wide), float("nan"), device="cuda")
        out[:, off:off + t.shape[1]] = t.cuda()
        return out[:, off:off + t.shape[1]]

    for trans in (False, True):
        Wt = W.t().contiguous() if trans else W
        for Wd in (Wt.cuda(), inside(Wt, Wt.shape[1] + 5, 1), inside(Wt, Wt.shape[1] + 8, 4)):
            for mk in (None, mask.cuda()):
                Z, A = sagnn.dense_gemm_act(inside(X, k + 8, 0), Wd, transW=trans, prec=prec, act=sagnn.ACT_RELU, mask=mk,
                                            want_z=True, want_act=True)
                want = ref if mk is None else torch.where(mask > 0, ref, torch.zeros(()).double())
                assert bool(((Z.cpu().double() - want).abs() <= bound).all())
                assert torch.equal(A, Z.clamp(min=0))


@pytest.mark.parametrize("prec", [sagnn.GEMM_FP32, sagnn.GEMM_BF16, sagnn.GEMM_FP32_BF16X3])
@pytest.mark.parametrize("m,k,n", [(49_152, 100, 64), (49_153, 132, 40), (38_400, 132, 132), (38_401, 132, 132), (65_537, 132, 128), (81_921, 128, 128),
                                   (65_537, 36, 64), (98_305, 64, 132), (98_306, 100, 256), (49_130, 128, 256), (131_073, 132, 96),
                                   (131_041, 256, 256), (16_380, 160, 200), (32_770, 40, 40), (200_001, 28, 20),
                                   (40_000, 64, 64)])
def test_dense_gemm_with_wide_and_narrow_slabs(m, k, n, prec):
    """Row counts on both sides of the lines between one launch of narrow slabs side by side and slabs as wide as W; with
    mask, W as it lies and transposed, and the product written over X."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + k)
    X = torch.randn(m, k, device="cuda", generator=gen)
    W = torch.randn(k, n, device="cuda", generator=gen)
    mask = torch.randn(m, n, device="cuda", generator=gen)
    ref, size = X.double() @ W.double(), X.abs().double() @ W.abs().double()
    # any order of k fp32 additions: k 2^-24 of the sum of the terms' sizes; an operand rounded to the 8 bits of bfloat16
    # is off by half of its last, 2^-8 of its size at most: (1 + 2^-8)^2 - 1 for the product of two
    tol = (2 * 2.0**-8 + 2.0**-16 if prec == sagnn.GEMM_BF16 else 2 * 2.0**-23) + (k + 2) * 2.0**-24
    for trans in (False, True):
        Wd = W.t().contiguous() if trans else W
        Z, A = sagnn.dense_gemm_act(X, Wd, transW=trans, prec=prec, act=sagnn.ACT_RELU, want_z=True, want_act=True)
        assert bool(((Z.double() - ref).abs() <= tol * size).all()) and torch.equal(A, Z.clamp(min=0))
        Zm, _ = sagnn.dense_gemm_act(X, Wd, transW=trans, prec=prec, mask=mask)
        assert torch.equal(Zm, torch.where(mask > 0, Z, torch.zeros_like(Z)))
    if n == k and n <= 64:   # one slab
        over = X.clone()
        sagnn.dense_gemm_act(over, W, prec=prec, want_z=True, out=(over, None))
        assert torch.equal(over, Z)


@pytest.mark.parametrize("prec", [sagnn.GEMM_FP32, sagnn.GEMM_FP32_BF16X3])
@pytest.mark.parametrize("m,k,n", [(31, 32, 64), (64, 32, 32), (97, 64, 64), (128, 64, 192), (65, 96, 64), (4100, 96, 32), (160, 128, 64)])
def test_dense_gemm_of_whole_k_groups_and_64_columns(m, k, n, prec):
    """One to four whole groups of k by slabs of 32 and 64 columns, each output alone and both, masked and not."""
    gen = torch.Generator().manual_seed(100 * k + n)
    X, W = torch.randn(m, k, generator=gen), torch.randn(k, n, generator=gen)
    mask = torch.randint(-1, 2, (m, n), generator=gen).float()
    ref = X.double() @ W.double()
    # any order of k fp32 additions: k 2^-24 of the sum of the terms' sizes
    bound = (2 * 2.0**-23 + (k + 2) * 2.0**-24) * (X.abs().double() @ W.abs().double())
    for mk in (None, mask.cuda()):
        want = ref if mk is None else torch.where(mask > 0, ref, torch.zeros(()).double())
        for z, a in ((True, False), (False, True), (True, True)):
            Z, A = sagnn.dense_gemm_act(X.cuda(), W.cuda(), prec=prec, act=sagnn.ACT_RELU, mask=mk, want_z=z, want_act=a)
            assert (Z is not None) == z and (A is not None) == a
            if z:
                assert bool(((Z.cpu().double() - want).abs() <= bound).all())
            if a:
                assert bool(((A.cpu().double() - want.clamp(min=0)).abs() <= bound).all())


@pytest.mark.parametrize("k,n", [(128, 128), (256, 256), (100, 44)])
def test_bf16x3_gemm_has_the_accuracy_of_the_fp32_gemm(k, n):
    """fp32 operands as three bfloat16 terms, six products: every operand bit takes part, so the
    result must be as close to the fp64 oracle as the fp32 matrix-core product is (both accumulate
    in fp32), and far inside the fp32 tolerance.  Operands with all 24 significant bits set, of both
    signs, very small and very large magnitudes, and zeros: a term lost in the split, a wrong pairing
    of the terms or a rounding that does not sum back to the operand shows at 2^-9 .. 2^-17."""
    m = 777
    X = synth.normal((m, k), 5, synth.STREAM_H)
    W = synth.normal((k, n), 5, synth.STREAM_W, scale=1 / np.sqrt(k))
    X[0, :] = np.float32(1.0) + np.float32(2.0 ** -23) * np.arange(1, 2 * k, 2, dtype=np.float32)   # dense low bits
    X[1, :] = -(np.float32(2.0) - np.float32(2.0 ** -23))                                              # all ones
    X[2, :] = X[2, :] * np.float32(1e-30)
    X[3, :] = X[3, :] * np.float32(1e30)
    X[4, :] = 0
    X[5, ::2] = np.float32(1.0 + 2.0 ** -8 + 2.0 ** -16)      # a tie at the first rounding, low bits behind it
    W[:, 0] = np.float32(1.0) - np.float32(2.0 ** -24)
    W[:, 1] = np.float32(-3.0) * (np.float32(1.0) + np.float32(2.0 ** -23))
    ref, zabs = oracle.gemm(X, W, want_abs=True)
    Z32, _ = sagnn.dense_gemm_act(dev(X), dev(W), prec=0)
    Zs, _ = sagnn.dense_gemm_act(dev(X), dev(W), prec=2)
    torch.cuda.synchronize()
    assert_close(Zs, ref, zabs, RTOL_GEMM_FP32, "bf16x3 gemm")
    scale = np.where(zabs > 0, zabs, 1.0)
    e32 = float(np.max(np.abs(Z32.cpu().numpy().astype(np.float64) - ref) / scale))
    es = float(np.max(np.abs(Zs.cpu().numpy().astype(np.float64) - ref) / scale))
    assert es <= max(2 * e32, 2e-7), (es, e32)
    assert es < 2e-6
    assert bool((Zs[4] == 0).all())


@pytest.mark.parametrize("m,k,n,transW", [(51_203, 64, 64, False), (51_203, 100, 68, True), (53_001, 256, 132, False), (70_001, 160, 40, False),
                                          (90_001, 128, 128, True), (170_003, 128, 40, False), (70_001, 40, 256, False), (307_203, 8, 36, True)])
def test_fp32_gemm_of_many_rows_with_values_that_three_terms_do_not_hold(m, k, n, transW):
    """Products of many rows are no further from 64 bits than those of few; a tile with an infinity, a tiny or a huge value, or
    all tiles of its columns if it is in W, gives bit for bit what a call of few rows gives; a row with a NaN is NaN, and no
    other."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + k)
    X = torch.randn(m, k, device="cuda", generator=gen)
    W = torch.randn(k, n, device="cuda", generator=gen) / k ** 0.5
    M = torch.randn(m, n, device="cuda", generator=gen)
    few = 640                                       # whole tiles
    odd = {3: float("inf"), 40: 1e-31, 100: 3e38, 140: -1e-42, m - 1: 2.0 ** 61}
    run = lambda x, w, mask: sagnn.dense_gemm_act(x, w.t().contiguous() if transW else w, transW=transW, mask=mask, want_z=True)[0]
    for mask in (None, M):
        Z, Z0 = run(X, W, mask), run(X[:few], W, None if mask is None else M[:few])
        ref = X.double() @ W.double()
        if mask is not None:
            ref = torch.where(M > 0, ref, 0.0)
        bound = k * 2.0 ** -24 * (X.double().abs() @ W.double().abs())
        assert float(((Z.double() - ref).abs() - bound).max()) <= 0
        assert float((Z.double() - ref)[:few].norm()) <= 1.02 * float((Z0.double() - ref[:few]).norm())
        Y = X.clone()
        for r, x in odd.items():
            Y[r, r % k] = x
        Y[75, 75 % k] = float("nan")
        last = (m - 1) // 32 * 32
        Z = run(Y, W, mask)
        tail = run(Y[last:], W, None if mask is None else M[last:])
        Z0 = run(Y[:few], W, None if mask is None else M[:few])
        for t in {r // 32 for r in odd if r < few}:
            a, b = Z[32 * t:32 * t + 32], Z0[32 * t:32 * t + 32]
            assert bool(((a == b) | (torch.isnan(a) & torch.isnan(b))).all()), t
        assert torch.equal(Z[last:], tail)
        want = torch.zeros(32, n, dtype=torch.bool, device="cuda")
        want[75 - 64] = True if mask is None else mask[75] > 0
        assert torch.equal(torch.isnan(Z[64:96]), want)
    for x in (float("inf"), 1e-38):
        V = W.clone()
        V[k - 1, n - 1] = x
        a, b = (z[:, (n - 1) // 32 * 32:] for z in (run(X, V, None)[:few], run(X[:few], V, None)))
        assert bool(((a == b) | (torch.isnan(a) & torch.isnan(b))).all()), x


@pytest.mark.parametrize("m,k,n,transW", [(51_203, 64, 64, False), (53_001, 256, 132, False), (70_001, 160, 40, False),
                                          (90_001, 128, 128, True), (70_001, 40, 256, False), (307_203, 8, 36, True)])
def test_fp32_gemm_rounds_once_a_term_and_row_by_row(m, k, n, transW):
    """One value a row of X: an output is one product, which fp32 instructions round once.  And a row's result is its own:
    bit for bit the same in a call of other rows, of few or many, and beside a row with an infinity, an underflowed and a
    huge value."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + n)
    X = torch.randn(m, k, device="cuda", generator=gen)
    W = torch.randn(k, n, device="cuda", generator=gen) / k ** 0.5
    run = lambda x: sagnn.dense_gemm_act(x, W.t().contiguous() if transW else W, transW=transW, want_z=True)[0]
    one = torch.zeros_like(X)
    at = torch.randint(k, (m, 1), device="cuda", generator=gen)
    one.scatter_(1, at, X.gather(1, at))
    assert torch.equal(run(one), (X.gather(1, at).double() * W.double()[at[:, 0]]).float())   # (24 bits by 24 in 53)
    Z = run(X)
    for a, b in ((0, 1), (17, 700), (700, 51_100), (51_100, m)):
        assert torch.equal(run(X[a:b]), Z[a:b]), (a, b)
    Y = X.clone()
    odd = [5, 640, m - 2]
    for r, x in zip(odd, (float("inf"), 1e-41, 3e38)):
        Y[r, r % k] = x
    rest = torch.ones(m, dtype=torch.bool, device="cuda")
    rest[odd] = False
    assert torch.equal(run(Y)[rest], Z[rest])


def test_bf16_gemm_is_tight_against_bf16_rounded_oracle():
    """With operands rounded the same way the only difference left is fp32 vs fp64 accumulation,
    so the result must sit far inside the 1e-2 budget; a wrong rounding mode would not."""
    X = synth.normal((512, 256), 1, synth.STREAM_H)
    W = synth.normal((256, 256), 1, synth.STREAM_W, scale=1 / 16)
    ref, zabs = oracle.gemm(X, W, bf16=True, want_abs=True)
    Z, _ = sagnn.dense_gemm_act(dev(X), dev(W), prec=1)
    torch.cuda.synchronize()
    assert_close(Z, ref, zabs, 2e-5, "bf16 gemm vs bf16-rounded oracle")


@pytest.mark.parametrize("fin,fout", [(4, 4), (16, 20), (20, 16), (32, 36), (36, 32), (64, 68), (132, 64), (160, 160), (256, 132), (256, 256)])
@pytest.mark.parametrize("m", [1, 31, 129, 4100])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_weight_gradient_at_the_edges_of_its_blocks(prec, m, fin, fout):
    """Y = H^T S with S = G (identity matrix): one, two and four columns a lane, several blocks of 64 columns with
    ragged ends, fewer rows than one matrix instruction takes, a slice's partial last step."""
    rp = dev(np.arange(m + 1, dtype=np.int32))
    ci, v = dev(np.arange(m, dtype=np.int32)), dev(np.ones(m, np.float32))
    H = synth.normal((m, fin), 1, synth.STREAM_H)
    G = synth.normal((m, fout), 1, synth.STREAM_G)
    W = synth.normal((fin, fout), 1, synth.STREAM_W)
    _, _, Y = sagnn.gcn_layer_bwd(rp, ci, v, dev(G), dev(W), None, dev(H), prec=prec, want_gprev=False)
    torch.cuda.synchronize()
    ref, yabs = oracle.gemm(H, G, bf16=(prec == 1), transX=True, want_abs=True)
    assert_close(Y, ref, yabs, RTOL_GEMM_FP32, "weight gradient")


@pytest.mark.parametrize("fin,fout", [(36, 16), (48, 48), (16, 40), (68, 64), (96, 92), (36, 100), (132, 44), (140, 144), (256, 72)])
@pytest.mark.parametrize("m", [1, 17, 64, 131, 5003, 40_003])
def test_weight_gradient_with_three_columns_a_lane(m, fin, fout):
    """Widths that blocks of 48 columns cover, whole and ragged; with NaN in the first two columns of H, which is what a
    lane of three columns reads past a row's end and must not use."""
    gen = torch.Generator().manual_seed(m + fin)
    rp = torch.arange(m + 1, dtype=torch.int32, device="cuda")
    ci, v = torch.arange(m, dtype=torch.int32, device="cuda"), torch.ones(m, device="cuda")
    H, G, W = torch.randn(m, fin, generator=gen), torch.randn(m, fout, generator=gen), torch.zeros(fin, fout, device="cuda")
    ref, size = H.double().T @ G.double(), H.abs().double().T @ G.abs().double()
    for first in (0, 2):
        H[:, :first] = float("nan")
        _, _, Y = sagnn.gcn_layer_bwd(rp, ci, v, G.cuda(), W, None, H.cuda(), prec=sagnn.GEMM_FP32, want_gprev=False)
        # any order of m additions: at most m 2^-24 of the sum of the terms' sizes
        assert bool(((Y.cpu().double() - ref).abs() <= (m + 2) * 2.0**-24 * size)[first:].all())


@pytest.mark.parametrize("fin,fout", [(256, 256), (200, 160), (144, 256)])
@pytest.mark.parametrize("m", [1, 129, 1000, 16_384, 16_385, 40_003])
def test_weight_gradient_of_more_than_eight_blocks(m, fin, fout):
    """Nine to sixteen blocks of Y: eight a workgroup up to 128 slices of 128 rows, sixteen beyond."""
    gen = torch.Generator().manual_seed(m + fin)
    rp = torch.arange(m + 1, dtype=torch.int32, device="cuda")
    ci, v = torch.arange(m, dtype=torch.int32, device="cuda"), torch.ones(m, device="cuda")
    H, G, W = torch.randn(m, fin, generator=gen), torch.randn(m, fout, generator=gen), torch.zeros(fin, fout, device="cuda")
    ref, size = H.double().T @ G.double(), H.abs().double().T @ G.abs().double()
    _, _, Y = sagnn.gcn_layer_bwd(rp, ci, v, G.cuda(), W, None, H.cuda(), prec=sagnn.GEMM_FP32, want_gprev=False)
    # any order of m additions: at most m 2^-24 of the sum of the terms' sizes
    assert bool(((Y.cpu().double() - ref).abs() <= (m + 2) * 2.0**-24 * size).all())


@pytest.mark.parametrize("prec,fin,fout", [(0, 128, 128), (1, 256, 256), (0, 64, 32), (0, 16, 16), (1, 48, 20),
                                           (2, 128, 128), (2, 256, 256), (2, 48, 20)])
def test_gcn_layer_fwd_bwd_small(prec, fin, fout):
    g = synth.sbm_graph(6000, 16, 40, 2, 3)
    H = synth.normal((g.n, fin), 1, synth.STREAM_H)
    W = synth.normal((fin, fout), 1, synth.STREAM_W, scale=1 / np.sqrt(fin))
    G = synth.normal((g.n, fout), 1, synth.STREAM_G)
    rp, ci, v = csr_dev(g)
    ws_in = sagnn.spmm_csr_prepare(rp, ci, v, g.n, fin)
    ws_out = sagnn.spmm_csr_prepare(rp, ci, v, g.n, fout)
    rtol = RTOL_BF16 if prec == 1 else RTOL_GEMM_FP32
    o = oracle.gcn_layer_fwd(g.rowptr, g.colidx, g.val, H, W, act=1, bf16=(prec == 1))
    T, Z, Ho = sagnn.gcn_layer_fwd(rp, ci, v, dev(H), dev(W), act=sagnn.ACT_RELU, prec=prec, ws=ws_in)
    torch.cuda.synchronize()
    assert_close(T, o["T"], o["Tabs"], RTOL_SPMM, "layer T")
    assert_close(Z, o["Z"], o["Zabs"], rtol, "layer Z")
    assert_close(Ho, o["H"], o["Zabs"], rtol, "layer H")
    # the dense stage by itself, on the very T the library produced: scale |T| |W| (no slack
    # inherited from the sparse product's sum of magnitudes)
    Tg = T.cpu().numpy()
    zt, ztabs = oracle.gemm(Tg, W, bf16=(prec == 1), want_abs=True)
    assert_close(Z, zt, ztabs, rtol, "layer Z vs oracle GEMM of the library's T")
    # backward of this layer with the oracle's own Z / inputs as given data
    Zprev = synth.normal((g.n, fin), 2, synth.STREAM_G)
    ob = oracle.gcn_layer_bwd(g.rowptr, g.colidx, g.val, G, W, Zprev, H, bf16=(prec == 1))
    S, Gp, Y = sagnn.gcn_layer_bwd(rp, ci, v, dev(G), dev(W), dev(Zprev), dev(H), prec=prec, ws=ws_out)
    torch.cuda.synchronize()
    assert_close(S, ob["S"], ob["Sabs"], RTOL_SPMM, "bwd S")
    assert_close(Gp, ob["Gprev"], ob["Gabs"], rtol, "bwd Gprev")
    assert_close(Y, ob["Y"], ob["Yabs"], rtol, "bwd Y")
    Sg = S.cpu().numpy()
    gt, gtabs = oracle.gemm(Sg, W, bf16=(prec == 1), transW=True, want_abs=True)
    assert_close(Gp, np.where(Zprev > 0, gt, 0), gtabs, rtol, "bwd Gprev vs oracle GEMM of the library's S")
    yt, ytabs = oracle.gemm(H, Sg, bf16=(prec == 1), transX=True, want_abs=True)
    assert_close(Y, yt, ytabs, rtol, "bwd Y vs oracle GEMM of the library's S")


@pytest.mark.parametrize("f", [64, 128])
def test_spmm_sweep_interval_barrier_gives_up_and_still_computes(f, force_sweep, monkeypatch):
    """Barrier mode: the workgroups of the sweep wait for each other at interval boundaries, for a
    bounded time.  Here every barrier is then told to expect more arrivals than there are
    workgroups (a host-side test hook), so the first wait runs into its 20-microsecond limit, the
    launch gives all barriers up and free-runs: every kernel still ends and the product is unchanged."""
    rng = np.random.default_rng(9 + f)
    m, n = 6000, 60_000
    rowptr, colidx, val = random_csr(m, n, 25, rng, hubs=[(3, 9000), (7, 3000), (2500, 1024)])
    B = synth.normal((n, f), f, synth.STREAM_H)
    ref, zabs = oracle.spmm(rowptr, colidx, val, B, want_abs=True)
    rp, ci, v = dev(rowptr), dev(colidx), dev(val)

    def run():
        ws = sagnn.spmm_csr_prepare(rp, ci, v, n, f)
        assert ws.info()["mode"] == 1
        out = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(B), ws=ws)
        torch.cuda.synchronize()
        return out, ws

    monkeypatch.setenv("SAGNN_SWEEP_SYNC", "48")             # 384 slabs: 8 intervals
    monkeypatch.setenv("SAGNN_SWEEP_BARRIERS", "1")
    normal, ws = run()
    assert ws.info()["barriers"] == 1 and ws.info()["intervals"] > 1 and not ws.barriers_gave_up()
    assert_close(normal, ref, zabs, RTOL_SPMM, "with interval barriers")
    monkeypatch.setenv("SAGNN_SWEEP_SYNC_TEST_EXTRA", "1000")
    monkeypatch.setenv("SAGNN_SWEEP_SYNC_US", "20")
    gave_up, ws = run()
    assert ws.barriers_gave_up()
    assert torch.equal(gave_up, normal)                       # same summation order either way
    monkeypatch.delenv("SAGNN_SWEEP_SYNC_TEST_EXTRA")
    monkeypatch.delenv("SAGNN_SWEEP_BARRIERS")
    # pacing: every wavefront holds itself to a time schedule (here far slower than it could run,
    # so every boundary really waits); same bits again
    monkeypatch.setenv("SAGNN_SWEEP_PACE_PS", "2000000")
    paced, ws = run()
    assert ws.info()["pace_ps_per_step"] == 2000000 and ws.info()["barriers"] == 0
    assert torch.equal(paced, normal)
    monkeypatch.delenv("SAGNN_SWEEP_PACE_PS")                 # and without intervals at all (the default)
    monkeypatch.delenv("SAGNN_SWEEP_SYNC")
    plain, ws = run()
    assert ws.info()["intervals"] == 1
    assert_close(plain, ref, zabs, RTOL_SPMM, "without intervals")


# ------------------------------------------------------------------------------------ fused layer

@pytest.mark.parametrize("prec,fin,fout", [(0, 128, 128), (1, 256, 256), (0, 64, 32), (1, 128, 100), (0, 128, 256),
                                           (1, 64, 64), (1, 256, 36)])
@pytest.mark.parametrize("graph", ["hubs_and_empty_rows", "sbm", "rmat"])
def test_gcn_layer_fwd_fused(prec, fin, fout, graph, cfg1):
    """The one-kernel layer (T = A H kept on the chip, then the dense transform on the matrix
    cores) against the oracle's layer: without T (gcn_layer_fwd with d_T = NULL) and with T as a
    by-product.  Rows longer than 512 entries take the workgroup-shared path; m is not a
    multiple of the tile height."""
    rng = np.random.default_rng(fin + fout)
    if graph == "hubs_and_empty_rows":
        m, n = 4133, 9000
        rowptr, colidx, val = random_csr(m, n, 20, rng, empty_frac=0.1,
                                         hubs=[(5, 8000), (6, 513), (7, 512), (4132, 5000), (300, 300), (301, 2049)], dup=True)
    elif graph == "sbm":
        g = synth.sbm_graph(6000, 16, 40, 2, 3)
        rowptr, colidx, val, m, n = g.rowptr, g.colidx, g.val, g.m, g.n
    else:
        g = synth.rmat_graph(30_000, 1_500_000, 4)
        rowptr, colidx, val, m, n = g.rowptr, g.colidx, g.val, g.m, g.n
    H = synth.normal((n, fin), 1, synth.STREAM_H)
    W = synth.normal((fin, fout), 1, synth.STREAM_W, scale=1 / np.sqrt(fin))
    rp, ci, v = dev(rowptr), dev(colidx), dev(val)
    rtol = RTOL_BF16 if prec == 1 else RTOL_GEMM_FP32
    o = oracle.gcn_layer_fwd(rowptr, colidx, val, H, W, act=1, bf16=(prec == 1))
    T, Z, Ho = sagnn.gcn_layer_fwd(rp, ci, v, dev(H), dev(W), act=sagnn.ACT_RELU, prec=prec, want_t=False)
    torch.cuda.synchronize()
    assert T is None
    assert_close(Z, o["Z"], o["Zabs"], rtol, "fused Z")
    assert_close(Ho, o["H"], o["Zabs"], rtol, "fused H'")
    assert torch.equal(Ho, torch.clamp_min(Z, 0))
    T, Z2, _ = sagnn.gcn_layer_fwd(rp, ci, v, dev(H), dev(W), act=sagnn.ACT_IDENTITY, prec=prec, fused=True,
                                   want_h=False)
    torch.cuda.synchronize()
    assert_close(T, o["T"], o["Tabs"], RTOL_SPMM, "fused T")
    assert torch.equal(Z2, Z)
    zt, ztabs = oracle.gemm(T.cpu().numpy(), W, bf16=(prec == 1), want_abs=True)
    assert_close(Z, zt, ztabs, rtol, "fused Z vs oracle GEMM of the kernel's own T")


@pytest.mark.parametrize("groups,fin,fout", [("1", 64, 36), ("1", 128, 128), ("1", 256, 132), ("2", 64, 256), ("2", 128, 100)])
def test_fp32_layer_with_values_that_three_terms_do_not_hold(groups, fin, fout, monkeypatch):
    """fp32 operands of the sweep's epilogue that a split into three bfloat16 terms would lose, rows of A H with an infinity, a
    NaN, a tiny or a huge value, and such a value in W: what the product and the dense transform give of the same rows of A H."""
    monkeypatch.setenv("SAGNN_SWEEP", "1")
    monkeypatch.setenv("SAGNN_SWEEP_GROUPS", groups)
    g = synth.sbm_graph(6000, 16, 40, 2, 5)
    rp, ci, v = dev(g.rowptr), dev(g.colidx), dev(g.val)
    H = synth.normal((g.n, fin), 3, synth.STREAM_H)
    H[7, 3], H[1500, 5], H[3000, 1], H[4500] = np.inf, np.nan, 3e38, 1e-36
    W = synth.normal((fin, fout), 3, synth.STREAM_W, scale=1 / np.sqrt(fin))
    ws = sagnn.spmm_csr_prepare(rp, ci, v, g.n, fin)
    assert ws.info()["mode"] == 1 and sagnn.gcn_layer_fwd_form(ws, fin, fout) == 2
    for x in (None, np.inf, 1e-38):
        if x is not None:
            W[fin - 1, fout - 1] = x
        T = sagnn.spmm_csr_tallskinny(rp, ci, v, dev(H), ws=ws)
        Z0 = sagnn.dense_gemm_act(T, dev(W), want_z=True)[0]
        _, Z, _ = sagnn.gcn_layer_fwd(rp, ci, v, dev(H), dev(W), ws=ws, want_t=False, want_h=False)
        assert torch.equal(torch.isnan(Z), torch.isnan(Z0)) and torch.equal(torch.isposinf(Z), torch.isposinf(Z0))
        assert torch.equal(torch.isneginf(Z), torch.isneginf(Z0))
        bound = 2 * fin * 2.0 ** -24 * (T.double().abs() @ dev(W).double().abs())   # the error of either
        ok = torch.isfinite(Z0)
        assert bool(((Z.double() - Z0.double()).abs() <= bound + 1e-44)[ok].all())


@pytest.mark.parametrize("groups,fin,fout", [("1", 64, 36), ("1", 128, 128), ("1", 256, 132), ("2", 128, 100), ("4", 64, 64)])
def test_fp32_layer_rounds_a_sum_once_a_term_and_only_reads_a_schedule_without_split_rows(groups, fin, fout, monkeypatch):
    """One value a column of W, small whole numbers in H: A H is exact, and an output is one product of it, which fp32
    instructions round once.  No row is cut into pieces here, and W is read where it lies: the call writes nothing to the
    workspace."""
    monkeypatch.setenv("SAGNN_SWEEP", "1")
    monkeypatch.setenv("SAGNN_SWEEP_GROUPS", groups)
    g = synth.sbm_graph(6000, 16, 40, 2, 5)
    rp, ci, v = dev(g.rowptr), dev(g.colidx), dev(np.ones_like(g.val))
    H = dev(np.round(2.0 ** 14 * synth.uniform((g.n, fin), 3, synth.STREAM_H)).astype(np.float32))
    W = np.zeros((fin, fout), np.float32)
    W[np.arange(fout) * 7 % fin, np.arange(fout)] = synth.normal((fout,), 3, synth.STREAM_W)
    ws = sagnn.spmm_csr_prepare(rp, ci, v, g.n, fin)
    info = ws.info()
    assert info["mode"] == 1 and info["chunk_rows"] == 0 and info["split_rows"] == 0
    assert sagnn.gcn_layer_fwd_form(ws, fin, fout) == 2
    before = ws.buf.clone()
    _, Z, _ = sagnn.gcn_layer_fwd(rp, ci, v, H, dev(W), ws=ws, want_t=False, want_h=False)
    assert torch.equal(ws.buf, before)
    T = sagnn.spmm_csr_tallskinny(rp, ci, v, H)
    assert torch.equal(T, T.round()) and float(T.abs().max()) < 2 ** 24
    assert torch.equal(Z, (T.double() @ dev(W).double()).float())   # (24 bits by 24 in 53)


@pytest.mark.parametrize("prec,fin,fout", [(0, 128, 128), (1, 256, 256), (0, 64, 36), (1, 128, 100), (1, 256, 64),
                                           (2, 128, 128), (2, 256, 256), (2, 64, 36), (2, 128, 100)])
@pytest.mark.parametrize("graph", ["regular_all_rows_swept", "with_split_short_and_empty_rows"])
def test_gcn_layer_fwd_sweep_epilogue(prec, fin, fout, graph, monkeypatch):
    """The layer with d_T = NULL on a workspace prepared for the one-row-per-instruction sweep: the
    sweep kernel ends with the dense transform (form 2).  A near-regular graph whose rows are all
    swept, and one with rows cut into pieces, rows outside the sweep and empty rows (the small
    kernel for the rows the sweep does not finish)."""
    monkeypatch.setenv("SAGNN_SWEEP", "1")
    monkeypatch.setenv("SAGNN_SWEEP_GROUPS", "1")
    monkeypatch.setenv("SAGNN_SWEEP_MINDEG", "16")
    monkeypatch.setenv("SAGNN_SWEEP_PIECE", "1024")
    monkeypatch.setenv("SAGNN_SWEEP_SHORT_ROWS", "-1")   # short rows stay outside the sweep: the small kernel takes them
    rng = np.random.default_rng(fin * 3 + fout)
    if graph == "regular_all_rows_swept":
        g = synth.sbm_graph(6000, 16, 40, 2, 5)
        rowptr, colidx, val, m, n = g.rowptr, g.colidx, g.val, g.m, g.n
    else:
        m, n = 5003, 12000
        rowptr, colidx, val = random_csr(m, n, 30, rng, empty_frac=0.05,
                                         hubs=[(7, 5000), (8, 1025), (4000, 3), (4001, 15), (5002, 2100)])
    H = synth.normal((n, fin), 3, synth.STREAM_H)
    W = synth.normal((fin, fout), 3, synth.STREAM_W, scale=1 / np.sqrt(fin))
    rp, ci, v = dev(rowptr), dev(colidx), dev(val)
    ws = sagnn.spmm_csr_prepare(rp, ci, v, n, fin)
    info = ws.info()
    assert info["mode"] == 1 and info["groups"] == 1
    assert sagnn.gcn_layer_fwd_form(ws, fin, fout, prec) == 2
    if graph != "regular_all_rows_swept":
        assert info["split_rows"] >= 3 and info["chunk_rows"] > 0 and info["has_empty_rows"] == 1
    rtol = RTOL_BF16 if prec == 1 else RTOL_GEMM_FP32
    o = oracle.gcn_layer_fwd(rowptr, colidx, val, H, W, act=1, bf16=(prec == 1))
    Z0 = torch.full((m, fout), float("nan"), device="cuda")
    H0 = torch.full((m, fout), float("nan"), device="cuda")
    T, Z, Ho = sagnn.gcn_layer_fwd(rp, ci, v, dev(H), dev(W), act=sagnn.ACT_RELU, prec=prec, ws=ws,
                                   want_t=False, out=(None, Z0, H0))
    torch.cuda.synchronize()
    assert T is None
    assert_close(Z, o["Z"], o["Zabs"], rtol, "sweep epilogue Z")          # every row written (no NaN left)
    assert_close(Ho, o["H"], o["Zabs"], rtol, "sweep epilogue H'")
    assert torch.equal(Ho, torch.clamp_min(Z, 0))
    # only H' wanted, identity activation
    _, Zn, Hi = sagnn.gcn_layer_fwd(rp, ci, v, dev(H), dev(W), act=sagnn.ACT_IDENTITY, prec=prec, ws=ws,
                                    want_t=False, want_z=False)
    torch.cuda.synchronize()
    assert Zn is None and torch.equal(Hi, Z)
    # the schedules with lane groups (two / four rows of H per load) end with the same transform
    monkeypatch.setenv("SAGNN_SWEEP_GROUPS", "2")
    if fin in (64, 128):
        ws2 = sagnn.spmm_csr_prepare(rp, ci, v, n, fin)
        assert ws2.info()["groups"] == (2 if fin == 128 else 4)
        assert sagnn.gcn_layer_fwd_form(ws2, fin, fout, prec) == 2
        Z0.fill_(float("nan"))
        H0.fill_(float("nan"))
        _, Zg, Hg = sagnn.gcn_layer_fwd(rp, ci, v, dev(H), dev(W), act=sagnn.ACT_RELU, prec=prec, ws=ws2,
                                        want_t=False, out=(None, Z0, H0))
        torch.cuda.synchronize()
        assert_close(Zg, o["Z"], o["Zabs"], rtol, "sweep epilogue, lane groups, Z")
        assert_close(Hg, o["H"], o["Zabs"], rtol, "sweep epilogue, lane groups, H'")
    if fin == 64:
        # a workspace prepared for 128 columns (two lane groups) serves a 64-wide layer
        ws3 = sagnn.spmm_csr_prepare(rp, ci, v, n, 128)
        assert ws3.info()["groups"] == 2 and sagnn.gcn_layer_fwd_form(ws3, 64, fout, prec) == 2
        Z0.fill_(float("nan"))
        _, Zw, _ = sagnn.gcn_layer_fwd(rp, ci, v, dev(H), dev(W), act=sagnn.ACT_RELU, prec=prec, ws=ws3,
                                       want_t=False, want_h=False, out=(None, Z0, None))
        torch.cuda.synchronize()
        assert_close(Zw, o["Z"], o["Zabs"], rtol, "sweep epilogue, prepared 128 called 64")
    # a workspace of the 256-wide schedule cannot serve... nothing: every width has a form; an
    # unprepared call (no workspace) takes the row-range kernel
    # (the row-range kernel has no three-term form: such a call is an error, not a silent fp32 product)
    assert sagnn.gcn_layer_fwd_form(None, fin, fout, prec) == (0 if prec == 2 else 1)
    if prec == 2:
        with pytest.raises(sagnn.SagnnError):
            sagnn.gcn_layer_fwd(rp, ci, v, dev(H), dev(W), act=sagnn.ACT_RELU, prec=prec, want_t=False)


def test_gcn_layer_fwd_fused_degenerate_shapes():
    """No entries at all (every row of T is zero, so Z = 0 and H' = 0), a single row, and a
    matrix of one long row that the wavefronts of a workgroup share."""
    f = 128
    W = synth.normal((f, f), 2, synth.STREAM_W, scale=1 / np.sqrt(f))
    H = synth.normal((300, f), 2, synth.STREAM_H)
    empty = torch.zeros(0, dtype=torch.int32, device="cuda")
    rp = dev(np.zeros(8, np.int32))                       # 7 rows, no entries
    T, Z, Ho = sagnn.gcn_layer_fwd(rp, empty, torch.zeros(0, device="cuda"), dev(H), dev(W), want_t=False)
    torch.cuda.synchronize()
    assert T is None and Z.shape == (7, f) and not Z.any().item() and not Ho.any().item()
    for deg in (1, 299):                                  # one row; 299 > none of the thresholds, then a shared row below
        rowptr = np.array([0, deg], np.int32)
        colidx = np.arange(deg, dtype=np.int32)
        val = synth.normal((deg,), deg, synth.STREAM_G).astype(np.float32)
        o = oracle.gcn_layer_fwd(rowptr, colidx, val, H, W, act=1)
        _, Z, Ho = sagnn.gcn_layer_fwd(dev(rowptr), dev(colidx), dev(val), dev(H), dev(W), want_t=False)
        torch.cuda.synchronize()
        assert_close(Z, o["Z"], o["Zabs"], RTOL_GEMM_FP32, f"fused one row of {deg}")
        assert_close(Ho, o["H"], o["Zabs"], RTOL_GEMM_FP32, f"fused one row of {deg} H'")
    rng = np.random.default_rng(4)
    cols = np.sort(rng.integers(0, 300, size=3000)).astype(np.int32)      # one row of 3000 entries (duplicates summed)
    rowptr = np.array([0, 3000], np.int32)
    val = rng.standard_normal(3000).astype(np.float32)
    o = oracle.gcn_layer_fwd(rowptr, cols, val, H, W, act=1)
    _, Z, Ho = sagnn.gcn_layer_fwd(dev(rowptr), dev(cols), dev(val), dev(H), dev(W), want_t=False)
    torch.cuda.synchronize()
    assert_close(Z, o["Z"], o["Zabs"], RTOL_GEMM_FP32, "fused one shared row")


def test_gcn_layer_fwd_fused_strided_h_and_unsupported_shapes():
    rng = np.random.default_rng(2)
    m, n, f = 1000, 2000, 128
    rowptr, colidx, val = random_csr(m, n, 10, rng)
    H = synth.normal((n, f), 1, synth.STREAM_H)
    W = synth.normal((f, f), 1, synth.STREAM_W, scale=1 / np.sqrt(f))
    o = oracle.gcn_layer_fwd(rowptr, colidx, val, H, W, act=1)
    wide = torch.full((n, f + 12), 9.0, device="cuda")
    wide[:, :f] = dev(H)
    _, Z, _ = sagnn.gcn_layer_fwd(dev(rowptr), dev(colidx), dev(val), wide[:, :f], dev(W), want_t=False)
    torch.cuda.synchronize()
    assert_close(Z, o["Z"], o["Zabs"], RTOL_GEMM_FP32, "fused, ldh > f")
    for fin, fout, prec in ((256, 256, 0), (16, 16, 0), (192, 64, 1)):
        Hs = dev(synth.normal((n, fin), 1, synth.STREAM_H))
        Ws = dev(synth.normal((fin, fout), 1, synth.STREAM_W))
        with pytest.raises(sagnn.SagnnError) as ei:
            sagnn.gcn_layer_fwd(dev(rowptr), dev(colidx), dev(val), Hs, Ws, prec=prec, want_t=False)
        assert ei.value.code == -1
