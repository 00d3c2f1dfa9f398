"""Packing of the sent rows from both sides: by send slot, and, for rows of some width, by
inner row where a partition sends rows more than once on average (the map of 12
partitions: by row at 48, 80, 256 and 512 columns, and at 300, in parts of lines).  A copy:
bit for bit."""
import numpy as np
import pytest
import torch

from gpu_helpers import random_partition_graph
from paper_2203_10428_amd import binding as B
from paper_2203_10428_amd.step import ld_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nparts,deg,by_row", [(2, 3, False), (12, 30, True)])
@pytest.mark.parametrize("cols", [1, 5, 41, 48, 80, 100, 256, 300, 512])
def test_pack(nparts, deg, by_row, cols):
    n_g, rowptr, col, owner = random_partition_graph(901, 700, nparts, deg, 5)
    part = B.pgcn_partition_setup(n_g, rowptr, col, owner, nparts, 0)
    idx = B.pgcn_partition_export(part)["send_idx"]
    info = B.pgcn_partition_info(part)
    assert (info["n_send"] > info["n_inner"]) == by_row and 0 < len(np.unique(idx)) < info["n_inner"] + (not by_row)
    src = torch.randn((info["n_inner"], ld_of(cols)), device="cuda")
    dst = torch.full((info["n_send"] + 1, ld_of(cols)), 7.0, device="cuda")
    B.pgcn_pack_boundary(part, B.PGCN_PACK_FEAT, src, dst, cols, ld_of(cols))
    assert torch.equal(dst[:-1, :cols], src[torch.from_numpy(idx).cuda().long(), :cols])
    assert torch.equal(dst[-1], torch.full_like(dst[-1], 7.0))
