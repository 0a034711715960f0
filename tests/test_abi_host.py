"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol the
header declares, and argument validation rejects bad calls before any HIP call is made."""
import ctypes
import os
import random
import re
import sysconfig

import numpy as np
import pytest
import torch

import paper_2504_04673_amd as sagnn
from paper_2504_04673_amd import binding, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "sagnn.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(?:int|const char\*)\s+([a-z_0-9]+)\s*\(", text)))


def test_header_symbols_are_exported():
    L = sagnn.lib()
    names = declared_functions()
    assert len(names) >= 12
    for n in names:
        assert hasattr(L, n), n
    assert sorted(binding.EXPORTS) == names


def test_binding_constants_match_the_header():
    """The binding repeats the header's flag and mode values; a change on one side only would
    silently select another path."""
    text = open(os.path.join(ROOT, "include", "sagnn.h")).read()
    defs = {k: int(v.rstrip("u"), 0) for k, v in re.findall(r"#define\s+(SAGNN_[A-Z0-9_]+)\s+(-?\d+u?)\b", text)}
    pairs = {"SAGNN_PLAN_VALIDATE": binding.PLAN_VALIDATE, "SAGNN_PLAN_OBLIVIOUS": binding.PLAN_OBLIVIOUS,
             "SAGNN_PLAN_MULTIPASS": binding.PLAN_MULTIPASS, "SAGNN_GEMM_FP32": binding.GEMM_FP32,
             "SAGNN_GEMM_BF16": binding.GEMM_BF16, "SAGNN_GEMM_FP32_BF16X3": binding.GEMM_FP32_BF16X3,
             "SAGNN_ACT_IDENTITY": binding.ACT_IDENTITY, "SAGNN_ACT_RELU": binding.ACT_RELU}
    for name, value in pairs.items():
        assert defs[name] == value, name
    assert len({binding.PLAN_VALIDATE, binding.PLAN_OBLIVIOUS, binding.PLAN_MULTIPASS}) == 3
    assert binding.PLAN_VALIDATE & binding.PLAN_OBLIVIOUS == 0 and binding.PLAN_MULTIPASS & 3 == 0


def test_version_and_strerror():
    L = sagnn.lib()
    assert L.sagnn_version() >= 100
    for code in (0, -1, -2, -3, -4, -99):
        assert len(L.sagnn_strerror(code)) > 0


def test_workspace_queries():
    L = sagnn.lib()
    b = ctypes.c_size_t(0)
    assert L.spmm_plan_workspace_bytes(10, 1000, 50, 4, ctypes.byref(b)) == 0 and b.value >= 1000 // 8
    assert L.spmm_plan_workspace_bytes(10, 1000, 50, 0, ctypes.byref(b)) == -1
    assert L.spmm_plan_workspace_bytes(10, 1 << 33, 50, 1, ctypes.byref(b)) == -1
    assert L.spmm_csr_workspace_bytes(10, 1000, 128, ctypes.byref(b)) == 0
    assert b.value >= 4 * 128 * 4
    assert L.spmm_csr_workspace_bytes(10, 1000, 6, ctypes.byref(b)) == -1
    plain = b.value
    assert L.spmm_csr_workspace_bytes_opt(10, 20, 1000, 128, None, ctypes.byref(b)) == 0 and b.value == plain
    tiles = sagnn.SpmmOptions()
    tiles.dense_tiles = 1
    # the tile region holds the rest CSR (8 bytes per entry) and the tile streams (8 bytes per entry)
    assert L.spmm_csr_workspace_bytes_opt(10, 20, 1000, 128, ctypes.byref(tiles), ctypes.byref(b)) == 0
    assert b.value >= plain + 16 * 1000
    assert L.spmm_csr_workspace_bytes_opt(10, 20, 1000, 100, ctypes.byref(tiles), ctypes.byref(b)) == 0  # no tile kernel at this width
    assert L.spmm_csr_workspace_bytes_opt(10, -1, 1000, 128, None, ctypes.byref(b)) == -1
    assert L.spmm_csr_workspace_bytes_opt(10, 20, 1000, 128, None, None) == -1
    assert L.gcn_bwd_workspace_bytes(1000, 256, 256, ctypes.byref(b)) == 0 and b.value >= 256 * 256 * 4
    assert L.gcn_bwd_workspace_bytes(1000, 102, 256, ctypes.byref(b)) == -1
    assert L.gcn_bwd_workspace_bytes(1000, 16, 260, ctypes.byref(b)) == -1


@pytest.mark.parametrize("f", [4, 16, 32, 64, 100, 128, 132, 256, 512])
def test_product_workspace_grows_with_the_entries(f):
    """On both sides of every count at which chunks or pieces get longer, a matrix of more entries needs no less room."""
    def size(nnz):
        b = ctypes.c_size_t(0)
        assert sagnn.lib().spmm_csr_workspace_bytes(1_000_000, nnz, f, ctypes.byref(b)) == 0
        return b.value

    steps = {8192 << e for e in range(18)} | {8192 * g * t for g in (1, 2, 4, 8, 16) for t in range(15, 130)}
    counts = sorted({c for s in steps for c in (s - 1, s, s + 1, s + s // 16)} | {0, 1, 4095, 2_147_483_647})
    sizes = [size(c) for c in counts]
    for a, b, x, y in zip(counts, counts[1:], sizes, sizes[1:]):
        assert x <= y, f"{x} bytes for {a} entries, {y} for {b}"


def test_product_workspace_grows_with_rows_entries_and_width():
    """Room for a matrix is room for every smaller one (widths that are never copied to aligned rows: there the room for
    the copy comes on top and is not asked for)."""
    rng = random.Random(5)
    for _ in range(20_000):
        small = rng.randint(0, 1 << rng.randint(0, 24)), rng.randint(0, (1 << rng.randint(0, 31)) - 1), 32 * rng.randint(1, 16)
        large = small[0] + rng.randint(0, 1 << rng.randint(0, 24)), min(small[1] + rng.randint(0, 1 << rng.randint(0, 31)),
                                                                        2_147_483_647), small[2] + 32 * rng.randint(0, 8)
        b = [ctypes.c_size_t(0), ctypes.c_size_t(0)]
        for x, (m, nnz, f) in zip(b, (small, large)):
            assert sagnn.lib().spmm_csr_workspace_bytes(m, nnz, f, ctypes.byref(x)) == 0
        assert b[0].value <= b[1].value, (small, large)


def test_scratch_of_the_other_calls_grows_with_their_sizes():
    """Room for a call is room for every smaller one: weight gradient (rows and both widths), column split, transpose,
    permutation."""
    rng = random.Random(6)
    L = sagnn.lib()

    def size(query, *args):
        b = ctypes.c_size_t(0)
        assert query(*args, ctypes.byref(b)) == 0
        return b.value

    def pair(high):
        return sorted(rng.randint(0, (1 << rng.randint(0, high)) - 1) for _ in range(2))

    widths = [4, 60, 64, 100, 124, 128, 132, 160, 192, 252, 256]
    for m in (0, 1, 128, 129, 32_768, 32_769, 65_536, 65_537, 10_000_000):
        sizes = [[size(L.gcn_bwd_workspace_bytes, m, fi, fo) for fo in widths] for fi in widths]
        for i in range(len(widths)):
            assert sizes[i] == sorted(sizes[i]) and [r[i] for r in sizes] == sorted(r[i] for r in sizes), (m, widths[i])
    for _ in range(20_000):
        (m0, m1), (e0, e1) = pair(24), pair(31)
        b0, b1 = sorted(rng.randint(1, 64) for _ in range(2))
        assert size(L.gcn_bwd_workspace_bytes, m0, 64, 100) <= size(L.gcn_bwd_workspace_bytes, m1, 64, 100)
        assert size(L.spmm_transpose_workspace_bytes, e0) <= size(L.spmm_transpose_workspace_bytes, e1)
        assert size(L.spmm_permute_workspace_bytes, m0, e0) <= size(L.spmm_permute_workspace_bytes, m1, e1)
        assert size(L.spmm_split_workspace_bytes, m0, b0) <= size(L.spmm_split_workspace_bytes, m1, b1)


def test_argument_validation_before_launch():
    L = sagnn.lib()
    # pack: bad f, null pointers, bad leading dimension
    assert L.spmm_pack_rows(None, 10, 16, 16, None, 5, None, 16, None) == -1
    assert L.spmm_pack_rows(None, 10, 16, 6, None, 0, None, 16, None) == -1
    assert L.spmm_pack_rows(None, 10, 8, 16, None, 0, None, 16, None) == -1
    assert L.spmm_pack_rows(None, 10, 16, 16, None, 0, None, 16, None) == 0     # N = 0: nothing to do
    # SpMM: null pointers with work to do, bad f
    assert L.spmm_csr_tallskinny(None, None, None, 4, 4, 4, None, 16, 16, None, 16, 0, None, 0, None) == -1
    assert L.spmm_csr_tallskinny(None, None, None, 0, 4, 0, None, 16, 16, None, 16, 0, None, 0, None) == 0
    assert L.spmm_csr_tallskinny(None, None, None, 4, 4, 4, None, 16, 18, None, 16, 0, None, 0, None) == -1
    assert L.spmm_csr_prepare(None, None, None, 4, 4, 4, 16, None, 0, None) == -1
    assert L.spmm_csr_prepare_tuned(None, None, None, 4, 4, 4, 16, None, 0, None, 16, None, 16, None, None, None) == -1
    assert L.spmm_csr_prepare_opt(None, None, None, 4, 4, 4, 16, None, 0, None, None) == -1
    bad = sagnn.SpmmOptions()
    bad.short_rows = 2                                    # not one of -1, 0, 1
    import ctypes as _c
    assert L.spmm_csr_prepare_opt(None, None, None, 4, 4, 4, 16, None, 0, _c.byref(bad), None) == -1
    bad = sagnn.SpmmOptions()
    bad.dense_tiles = 2                                   # not one of -1, 0, 1
    assert L.spmm_csr_prepare_opt(None, None, None, 4, 4, 4, 16, None, 0, _c.byref(bad), None) == -1
    assert L.spmm_csr_release(None) == -1
    assert L.spmm_csr_tile_info(None, None) == -1
    import numpy as _np
    info = _np.zeros(6, dtype=_np.int64)
    never_prepared = _c.c_void_p(0x1000)
    assert L.spmm_csr_tile_info(never_prepared, info.ctypes.data_as(_c.c_void_p)) == -1
    # plan: missing host arrays
    assert L.spmm_plan_needed_rows(None, None, 4, 4, 0, None, 1, None, 0, None, None, None, 0, 0, None) == -1
    # GEMM: unsupported sizes
    assert L.dense_gemm_act(None, 128, None, 128, 0, 10, 102, 128, 0, 0, None, 0, None, 0, None, 0, None) == -1
    assert L.dense_gemm_act(None, 128, None, 128, 0, 10, 128, 512, 0, 0, None, 0, None, 0, None, 0, None) == -1
    # split / stage loop: bad block count, missing arrays, too many blocks
    b = ctypes.c_size_t(0)
    assert L.spmm_split_workspace_bytes(100, 4, ctypes.byref(b)) == 0 and b.value > 0
    assert L.spmm_split_workspace_bytes(100, 257, ctypes.byref(b)) == -1
    assert L.spmm_split_colblocks(None, None, None, 4, 0, None, 2, None, None, None, None, None, 0, None) == -1
    assert L.spmm_stage_loop(None, 1, 4, None, 4, 16, 16, None, None, 4, None, 16, 0, None, None) == -1


def test_options_from_env_translation(monkeypatch):
    """The library reads no environment; the binding turns the experiment variables into the
    options struct (host only)."""
    for k in list(os.environ):
        if k.startswith("SAGNN_SWEEP") or k.startswith("SAGNN_TILE"):
            monkeypatch.delenv(k)
    o = sagnn.options_from_env()
    assert all(getattr(o, n) == 0 for n, _ in sagnn.SpmmOptions._fields_)
    monkeypatch.setenv("SAGNN_SWEEP", "1")
    monkeypatch.setenv("SAGNN_SWEEP_SLAB_MB", "0")
    monkeypatch.setenv("SAGNN_SWEEP_LPT", "0")
    monkeypatch.setenv("SAGNN_SWEEP_SYNC", "0")
    monkeypatch.setenv("SAGNN_SWEEP_PIECE", "1024")
    o = sagnn.options_from_env()
    assert (o.schedule, o.slab_kb, o.snake, o.sync_slabs, o.piece) == (2, -1, 1, -1, 1024)
    monkeypatch.setenv("SAGNN_SWEEP", "0")
    monkeypatch.setenv("SAGNN_SWEEP_SLAB_MB", "2")
    monkeypatch.setenv("SAGNN_SWEEP_SYNC", "8")
    o = sagnn.options_from_env()
    assert (o.schedule, o.slab_kb, o.sync_slabs) == (1, 2048, 8)
    monkeypatch.setenv("SAGNN_TILES", "1")
    monkeypatch.setenv("SAGNN_TILE_REUSE_X10", "40")
    o = sagnn.options_from_env()
    assert (o.dense_tiles, o.tile_reuse_x10) == (1, 40)
    src = open(os.path.join(ROOT, "paper_2504_04673_amd", "csrc", "spmm_sweep.hip")).read()
    assert "getenv" not in open(os.path.join(ROOT, "paper_2504_04673_amd", "csrc", "tiles.hip")).read()
    assert "getenv" not in src and "getenv" not in open(os.path.join(ROOT, "paper_2504_04673_amd", "csrc", "spmm.hip")).read()


def test_volume_stats_host_only():
    """spmm_volume_stats is host arithmetic: it runs without a GPU.  Hand-counted 3 x 3 case."""
    st = sagnn.spmm_volume_stats([[9, 1, 2], [4, 9, 0], [5, 6, 9]], 2, 4)
    assert st["total_bytes"] == 144 and st["avg_bytes"] == 48 and st["max_recv_bytes"] == 88
    assert st["max_send_bytes"] == 72 and st["cut_rows"] == 6 and st["cut_bytes"] == 48
    assert st["send_imbalance_pct"] == pytest.approx(50.0)
    assert sagnn.lib().spmm_volume_stats(None, 3, 2, 4, None) == -1


def test_binding_refuses_cpu_tensors():
    import torch
    with pytest.raises(ValueError):
        sagnn.spmm_pack_rows(torch.zeros(4, 4), torch.zeros(2, dtype=torch.int32))


def test_bench_refuses_more_than_one_gpu():
    """The benchmark measures one GPU's share: --gpus N > 1 exits with a message (no GPU needed)."""
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 2
    assert "ONE GPU" in r.stderr or "one GPU" in r.stderr.lower()
    assert r.stdout.strip() == ""


def test_step_calls_by_address_take_what_the_declared_ones_take():
    """The calls of a step go by address instead of through ctypes: the same results for the same arguments, and what has no
    integer (or, for a pointer, None or a host array) in a parameter's place, or another number of arguments, is refused."""
    L, calls = sagnn.lib(), binding._calls()
    for name in binding.STEP_CALLS:
        declared, bound = getattr(L, name), getattr(calls, name)
        none = [None if t is ctypes.c_void_p else 0 for t in declared.argtypes]
        for x in (0, 1, 4, -1, 1 << 40):          # all of them invalid calls: no pointer is given
            args = [a if a is None else x for a in none]
            assert bound(*args) == declared(*args), (name, x)
        for x in (np.int64(3), np.int32(-1), np.uint8(4), np.array(2), torch.tensor(1), True):
            args = [a if a is None else x for a in none]
            assert bound(*args) == declared(*args), (name, x)
        for args in (none[:-1], none + [0], [], [1.0 if a is None else a for a in none], ["" for a in none],
                     [a if a is None else np.array([1, 2]) for a in none], [a if a is None else 2.0 for a in none],
                     [0 if t is ctypes.c_void_p else None for t in declared.argtypes]):
            with pytest.raises(TypeError):
                bound(*args)
        for bad in (1.0, None, np.int64(0), np.array(0), torch.tensor(0)):              # each in each place, refused alike
            for i, t in enumerate(declared.argtypes):
                args = none[:i] + [bad] + none[i + 1:]
                try:
                    expected = declared(*args)
                except ctypes.ArgumentError:
                    with pytest.raises(ctypes.ArgumentError):
                        bound(*args)
                else:
                    assert bound(*args) == expected, (name, i, bad)
    # host arrays: block boundaries that begin at 0, ascend and end at n (what is refused then is the missing row pointer) or not
    for blocks in ([0, 3, 8], [1, 3, 8], [0, 3, 9], [0, 9, 8]):
        a, out = np.array(blocks, dtype=np.int64), np.zeros(3, dtype=np.int64)
        args = [1 << 12, 1 << 12, 1, 8, 0, a, 2, 1 << 12, 8, out, None, None, 0, 0, None]      # (no workspace)
        rc = calls.spmm_plan_needed_rows(*args)
        assert rc == L.spmm_plan_needed_rows(*[x.ctypes.data if isinstance(x, np.ndarray) else x for x in args])
        assert (rc == -3) == (blocks != [0, 3, 8]) and rc < 0
    with pytest.raises((TypeError, BufferError, ValueError)):
        calls.spmm_plan_needed_rows(*[np.zeros((4, 4), dtype=np.int64)[:, 1] if i == 5 else x for i, x in enumerate(args)])


def test_step_calls_without_their_extension_go_through_ctypes(monkeypatch):
    """Not built for this interpreter: the same results, host arrays in a pointer's place among the arguments."""
    by_address = binding._calls()
    monkeypatch.setattr(binding, "_bound", None)
    monkeypatch.setattr(build, "MARSHAL", build.MARSHAL + ".none")
    calls = binding._calls()
    assert calls is not by_address
    for name in binding.STEP_CALLS:
        for x in (0, 4, -1, np.int64(3)):             # all of them invalid calls: no pointer is given
            args = [None if t is ctypes.c_void_p else x for t in getattr(sagnn.lib(), name).argtypes]
            assert getattr(calls, name)(*args) == getattr(by_address, name)(*args), (name, x)
        for bad in (1.0, np.int64(0)):
            with pytest.raises(ctypes.ArgumentError):
                getattr(calls, name)(*[bad if a is None else a for a in args])
    for blocks in ([0, 3, 8], [1, 3, 8]):
        a, out = np.array(blocks, dtype=np.int64), np.zeros(3, dtype=np.int64)
        args = [1 << 12, 1 << 12, 1, 8, 0, a, 2, 1 << 12, 8, out, None, None, 0, 0, None]
        assert calls.spmm_plan_needed_rows(*args) == by_address.spmm_plan_needed_rows(*args) < 0


def test_extension_of_the_calls_is_built_for_this_interpreter_and_moved_into_place(monkeypatch, tmp_path):
    """Its name carries the interpreter's; it is out of date with its source; where there is no compiler the library is built
    without it, and none of another source is left behind."""
    assert build.MARSHAL.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    source, out = tmp_path / "marshal.c", str(tmp_path / os.path.basename(build.MARSHAL))
    source.write_text(open(build.MARSHAL_SOURCE).read())
    monkeypatch.setattr(build, "MARSHAL_SOURCE", str(source))
    monkeypatch.setattr(build, "MARSHAL", out)
    assert build.marshal_stale()
    assert build.build_marshal() == out and not build.marshal_stale()
    assert sorted(os.listdir(tmp_path)) == sorted(["marshal.c", os.path.basename(out)])
    os.utime(source, (os.path.getmtime(out) + 1,) * 2)
    assert build.marshal_stale() and build.stale()
    monkeypatch.setattr(build, "SOURCES", [])                        # (nothing but this to build)
    monkeypatch.setattr(build, "LIB", str(tmp_path / "lib.so"))
    monkeypatch.setenv("HIPCC", "true")
    monkeypatch.setenv("CC", str(tmp_path / "no_compiler"))
    with pytest.warns(UserWarning, match="ctypes"):
        build.build_hip()
    assert os.listdir(tmp_path) == ["marshal.c"]
