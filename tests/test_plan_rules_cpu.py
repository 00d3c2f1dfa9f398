"""Host rules of the kernel launches (no GPU): the range of memory that the sliced
aggregation's buffer resource covers, the node splits of the weight gradient and the
side from which sent rows are packed."""
import ctypes as C
import os
import subprocess

import pytest

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
