"""Update GEMMs at the row counts where their tiles change: 64-wide tiles while
those of 128 columns number at most 128 (128 x 128 rows of one 128-wide column
tile are 16,384), 256-wide ones from 256 of them on (32,768 rows of 256 columns).
The graph has no edges, so P is the identity and the
products stand alone: Z = X W, J_in = M W^T, dW = X^T M.

Element bounds against fp64 of the same (bf16: rounded) operands: K terms summed
in fp32 in any order are within (K + 2) 2^-24 of the terms' magnitudes; by parts
six products stand for one and the dropped ones are below 2^-21 (1 + 2^-7)."""
import numpy as np
import pytest
import torch

from paper_2203_10428_amd import binding as B
from paper_2203_10428_amd.step import ld_of

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def part_of(n, _parts={}):
    if n not in _parts:
        _parts.clear()
        _parts[n] = B.pgcn_partition_setup(n, np.zeros(n + 1, np.int64), np.zeros(0, np.int32), np.zeros(n, np.int32), 1, 0)
    return _parts[n]


def mat(gen, n, f, scale=1.0):
    """[n, f] normal values in rows whose padding is NaN (never read as data)."""
    m = torch.full((n, ld_of(f)), float("nan"), device="cuda")
    m[:, :f] = torch.randn((n, f), generator=gen, device="cuda") * scale
    return m


# 32,640 rows: 255 row tiles (128-wide tiles for N <= 256, 256-wide for N = 512); 32,769: 257, the last of one row;
# 16,384 and 16,385: 128 and 129; 5,900: 47, so that two column tiles make a grid of 94, no multiple of 8
@pytest.mark.parametrize("n", [32640, 32769, 130, 16384, 16385, 5900])
@pytest.mark.parametrize("f_in,f_out", [(17, 256), (40, 128), (33, 300), (64, 512), (130, 65)])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_products(n, f_in, f_out, dt):
    part = part_of(n)
    gen = torch.Generator("cuda").manual_seed(f_in * 1000 + f_out)
    dtype = B.PGCN_BF16 if dt == "bf16" else B.PGCN_F32
    X, J, H = mat(gen, n, f_in), mat(gen, n, f_out, 1e-3), mat(gen, n, f_out)
    W = torch.rand((f_in, f_out), generator=gen, device="cuda") - 0.5
    nb = B.pgcn_workspace_size(part, f_in, f_out, dtype)
    common = dict(f_in=f_in, f_out=f_out, gemm_dtype=dtype, relu=False, ld_in=ld_of(f_in), ld_out=ld_of(f_out), W=W,
                  workspace=torch.full((nb,), 255, dtype=torch.uint8, device="cuda"), workspace_bytes=nb)
    A, Z = torch.empty_like(X), torch.empty((n, ld_of(f_out)), device="cuda")
    B.pgcn_layer_fwd(part, H_in=X, H_bd=None, A=A, A_bf16=None, H_out=Z, **common)
    dW, J_in = torch.empty_like(W), torch.empty_like(X)
    common["relu"] = True
    B.pgcn_layer_bwd(part, J_out=J, H_out=H, A=A, A_bf16=None, dW=dW, J_in=J_in, J_bd_out=None, **common)
    r = (lambda t: t.bfloat16().double()) if dt == "bf16" else (lambda t: t.double())
    x, w = r(X[:, :f_in]), r(W)
    m = r(torch.where(H[:, :f_out] > 0, J[:, :f_out], torch.zeros(())))

    def check(got, a, b, what):
        terms = a.shape[1]
        factor = (terms + 2) * U if dt == "bf16" else (6 * terms + 2) * U + 2.0 ** -21 * (1 + 2.0 ** -7)
        over = (got.double() - a @ b).abs() > factor * (a.abs() @ b.abs())
        assert not over.any(), (what, int(over.sum()))

    check(Z[:, :f_out], x, w, "Z")
    check(J_in[:, :f_in], m, w.T, "J_in")
    check(dW, x.T.contiguous(), m, "dW")
