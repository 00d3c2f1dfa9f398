"""Host rules of the kernel launches (no GPU): which matrices get sliced aggregation
plans and which calls take them, the range of memory that the sliced kernel's buffer
resource covers, the node splits of the weight gradient and the side from which sent
rows are packed."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from gpu_helpers import random_partition_graph
from paper_2203_10428_amd import binding as B
from paper_2203_10428_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
_i64 = C.c_int64


@pytest.fixture(scope="session")
def probe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("probe") / "plan_probe.so")
    subprocess.run([build.HIPCC, *build.COMMON, "-shared", os.path.join(HERE, "plan_probe.cpp"), "-o", out], check=True)
    lib = C.CDLL(out)
    lib.probe_slice_bytes.restype = _i64
    lib.probe_slice_bytes.argtypes = [_i64] * 4
    lib.probe_pack_by_row.argtypes = [_i64] * 5
    lib.probe_plan.argtypes = [C.c_void_p, C.c_int, C.c_int, C.c_void_p]
    lib.probe_taken.argtypes = [C.c_void_p, C.c_int, _i64, _i64, _i64, _i64]
    return lib


@pytest.mark.parametrize("rows,ld,f", [(1, 100, 100), (7, 104, 100), (700, 512, 100), (3, 320, 257), (5000, 4096, 640)])
def test_sliced_reads_end_with_the_last_row(probe, rows, ld, f):
    """A source may be a view into a wider matrix: the resource ends with the last row's columns
    (rounded up to a float4), and holds all of every row's."""
    f4 = (f + 3) // 4
    for c4 in range(0, f4, 16):
        end = 16 * c4 + probe.probe_slice_bytes(rows, ld, f4, c4)
        assert end == 4 * (rows - 1) * ld + 16 * f4 <= 4 * ((rows - 1) * ld + f + 3)
    assert probe.probe_slice_bytes(0, ld, f4, 0) == 0
    assert probe.probe_slice_bytes((1 << 30) // ld + 2, ld, f4, 0) == -1          # 4 GiB and more


@pytest.mark.parametrize("slab", [16, 32])
def test_weight_gradient_splits_hold_nodes(probe, slab):
    """No split is launched without nodes (2,000 nodes, 56 splits asked for: 64-node chunks, 32 splits),
    but for those that keep tiles x splits a multiple of 8 where it was one."""
    out = (C.c_int * 2)()
    for K in (0, 1, 15, 16, 17, 33, 1000, 2000, 2001, 14500, 239000):
        for tiles in (1, 2, 3, 5, 8, 20):
            for asked in (1, 3, 7, 8, 24, 56, 63, 125, 768):
                probe.probe_tn_split(K, tiles, asked, slab, out)
                splits, chunk = out
                assert 1 <= splits <= asked and chunk % slab == 0 and chunk > 0 and splits * chunk >= K
                used = max(1, -(-K // chunk))
                assert splits == used or (tiles * asked % 8 == 0 and tiles * splits % 8 == 0 and splits - used < 8)
    probe.probe_tn_split(2000, 1, 56, 32, out)
    assert list(out) == [32, 64]


@pytest.mark.parametrize("f,ld,dst,most", [
    (4, 8, 0, 0), (40, 40, 0, 0), (44, 48, 0, 0),        # narrow: by slot whatever the map
    (48, 48, 0, 8), (64, 64, 0, 8), (80, 80, 0, 40), (512, 512, 0, 40),              # whole 64-byte lines
    (64, 64, 16, 0), (100, 104, 0, 2), (264, 264, 0, 2), (300, 304, 0, 8), (512, 520, 0, 8), (512, 512, 32, 8)])
def test_rows_packed_by_inner_row(probe, f, ld, dst, most):
    """The most slots per row at which rows of f floats are packed by inner row (never at one or fewer)."""
    rows = 1000
    by_row = [r for r in (1, 2, 8, 40) if probe.probe_pack_by_row(r * rows, rows, (f + 3) // 4, ld, dst)]
    assert by_row == [r for r in (2, 8, 40) if r <= most]


# ------------------------------------------------------------- sliced plans ---

PLAIN, NARROW, SLICED = range(3)
NEVER, MB = -1, 1 << 20
AT = 1 << 20                                             # an address of whole lines


@pytest.fixture
def clean(monkeypatch):
    for k in ("PGCN_AGG_CHUNKS", "PGCN_AGG_CHUNKS_T", "PGCN_AGG_CHUNKS_NARROW", "PGCN_AGG_SLICED", "PGCN_SEGMENT"):
        monkeypatch.delenv(k, raising=False)
    return monkeypatch


def plan(probe, part, transposed, which):
    out = (_i64 * 256)()
    n = probe.probe_plan(part.handle, transposed, which, out)
    return dict(zip(("chunks", "slots", "whole", "full"), out[:4]), cuts=list(out[4:n]))


def skewed_graph(n_inner, n_pool, m, seed, columns):
    """`m` edges of which 0.7 have an end among the first `columns` nodes of either kind."""
    rng = np.random.default_rng(seed)
    n = n_inner + n_pool
    u = rng.integers(0, n_inner, m)
    v = np.where(rng.random(m) < 0.7, rng.integers(0, columns, m) + n_inner * (rng.random(m) < 0.3), rng.integers(0, n, m))
    u, v = u[u != v], v[u != v]
    key = np.unique(np.concatenate([u * n + v, v * n + u]))
    rowptr = np.searchsorted(key, np.arange(n + 1) * n).astype(np.int64)
    return n, rowptr, (key % n).astype(np.int32), (np.arange(n) >= n_inner).astype(np.int32)


def uniform_graph(n_inner, n_pool, deg):
    return random_partition_graph(n_inner, n_pool, 2, deg, 3)


@pytest.mark.parametrize("graph,forward,transposed", [
    # below 2^20 non-zeros: plain plans
    (lambda: uniform_graph(8000, 4500, 100), (NEVER, NEVER), (NEVER, NEVER)),
    # long runs, whole chunks stay in an L2, no more chunks than the plain plan's
    (lambda: uniform_graph(9000, 4500, 140), (0, 0), (0, 0)),
    # an L2 holds a tenth of the gathers of a sparse uniform graph: whole launches of the transposed plan
    (lambda: uniform_graph(120000, 60000, 11), (NEVER, NEVER), (0, NEVER)),
    # skewed, short runs in one chunk a side, two in the forward plan: 6 to 7, 14 to 15, 27 non-zeros a run there
    (lambda: skewed_graph(120000, 60000, 900000, 5, 2000), (NEVER, NEVER), (0, 400 * MB)),
    (lambda: skewed_graph(60000, 30000, 1020000, 5, 2000), (400 * MB, 400 * MB), (0, 128 * MB)),
    (lambda: skewed_graph(30000, 15000, 1000000, 5, 2000), (0, 96 * MB), (0, 0))])
def test_default_choice_of_sliced_plans(probe, clean, graph, forward, transposed):
    n, rowptr, col, owner = graph()
    clean.setenv("PGCN_HUB", "0")                        # a dense block would take non-zeros off the runs
    part = B.pgcn_partition_setup(n, rowptr, col, owner, 2, 0, host_only=True)
    info = B.pgcn_partition_info(part)
    n_in, n_bd, nnz = info["n_inner"], info["n_bd"], info["nnz"]
    assert (nnz >= 1 << 20) == (transposed != (NEVER, NEVER)) and max(n_in, n_bd) > 4096
    for t, use, nrows, sides in ((0, forward, n_in, (n_in, n_bd)), (1, transposed, n_in + n_bd, (n_in,))):
        plain, sl = plan(probe, part, t, PLAIN), plan(probe, part, t, SLICED)
        assert (sl["whole"], sl["full"]) == use, (t, nnz / nrows)
        assert info["spmmt_chunks" if t else "spmm_chunks"] == (sl if sl["chunks"] else plain)["chunks"]
        if use == (NEVER, NEVER):
            assert sl["chunks"] == 0
            continue
        assert sl["slots"] <= plain["slots"]             # the scratch memory is sized by the plain plan
        cuts = sl["cuts"]
        assert cuts[0] == 0 and cuts[-1] == sum(sides) and all(s in cuts for s in np.cumsum(sides))
        for a, b in zip(cuts, cuts[1:]):
            assert 0 < b - a and (b - a <= 16500 or nnz // nrows < 64)
        rows = n_in if t else n_in + n_bd
        for f, kind in ((64, None), (65, None), (96, None), (112, "full"), (128, "full"), (144, None), (192, None),
                        (200, None), (224, "full"), (256, "whole"), (300, "full"), (512, "whole"), (602, "full")):
            at = sl[kind] if kind else NEVER
            tight = -(-f // 32) * 32
            for ld in {tight, max(tight, -(-max(at, 0) // (4 * rows * 32)) * 32), 1 << 13}:
                taken = probe.probe_taken(part.handle, t, f, AT, 0 if t else AT, ld) == SLICED
                assert taken == (at != NEVER and 4 * rows * ld >= at), (t, f, ld)


def test_calls_that_leave_the_sliced_plan(probe, clean):
    """Sources whose slices straddle lines and sources of 4 GiB run the plain plan, as narrow rows and
    refused widths do; PGCN_AGG_SLICED=1 keeps all but the 4 GiB ones."""
    n, rowptr, col, owner = uniform_graph(9000, 4500, 140)
    part = B.pgcn_partition_setup(n, rowptr, col, owner, 2, 0, host_only=True)
    took = lambda f, lo, hi, ld, t=0: probe.probe_taken(part.handle, t, f, lo, hi, ld)
    assert took(256, AT, AT, 256) == took(256, AT, 0, 256) == took(256, AT, 0, 256, 1) == SLICED
    assert took(256, AT, AT, 260) == took(256, AT + 64, AT, 256) == took(256, AT, AT + 16, 256) == PLAIN
    limit = 0xfffff000 // 4 // 8999 // 32 * 32           # the second row of 9,000 that passes 32-bit offsets
    assert took(256, AT, AT, limit - 32) == SLICED and took(256, AT, AT, limit + 32) == PLAIN
    n, rowptr, col, owner = skewed_graph(60000, 30000, 1020000, 5, 2000)
    clean.setenv("PGCN_AGG_SLICED", "1")
    part = B.pgcn_partition_setup(n, rowptr, col, owner, 2, 0, host_only=True)
    for f in (65, 72, 100, 144, 300, 602):
        assert took(f, AT + 16, AT, f // 4 * 4 + 4) == took(f, AT, 0, f // 4 * 4 + 4, 1) == SLICED
    assert took(64, AT, AT, 64) != SLICED and took(72, AT, AT, 1 << 15) == PLAIN
    clean.setenv("PGCN_AGG_SLICED", "0")
    part = B.pgcn_partition_setup(n, rowptr, col, owner, 2, 0, host_only=True)
    assert took(256, AT, AT, 1 << 11) == PLAIN and plan(probe, part, 1, SLICED)["chunks"] == 0
