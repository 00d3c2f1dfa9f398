"""Host side of the sliced aggregation (no GPU): the range of memory that its
buffer resource covers."""
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
