"""The persistent coarse CG on coarse grids with more sites than workgroups,
from one right-hand side to sixteen in a row on one handle (each count grows
the work fields), in every storage: each solution's residual, measured with
the complex128 mat-vec.

All workgroups have to be resident at once: a solve whose grid does not find
room ends with an error at its wait limit.

The CG stops at a recursive residual of 1e-5 (complex64) or 1e-3 (16 bits).  In
complex64 the true one drifts from it by rounding, at most 6e-8 a step relative
to |b| for some tens of steps: 2e-5 in all.  In 16 bits the operator itself is
rounded to 2^-9 (bf16) or 2^-12 (fp16) of each matrix's largest entry, which
bounds the residual relative to |b| by that times the condition number (below
5 here): 2e-2 in all."""
import pytest

import synth
from tests.gpu_util import banner

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1402_2585_amd as hd  # noqa: E402


@pytest.mark.parametrize("nvec,prec", [(8, hd.DWF_C64), (6, hd.DWF_C64), (16, hd.DWF_C64), (8, hd.DWF_BF16),
                                       (12, hd.DWF_F16), (24, hd.DWF_BF16)])
def test_more_sites_than_workgroups(nvec, prec):
    dims, Ls = (24, 24, 24, 12), 1
    banner(f"coarse CG grid {dims} nvec {nvec} prec {prec}")
    op = hd.FineOperator(synth.gauge_field(dims, 0.3, 474), dims, Ls, 1.8, 0.3)
    h = hd.HDCG(op, (4, 4, 4, 4), synth.gaussian_half_field(dims, Ls, 475, nrhs=nvec))
    Nc = dims[0] * dims[1] * dims[2] * dims[3] // 256
    g = torch.Generator(device="cuda").manual_seed(7)
    for nr in (1, 2, 4, 8, 16):
        b = torch.randn((nr, Nc, nvec), generator=g, device="cuda", dtype=torch.complex64)
        x = torch.zeros_like(b)
        for _ in range(3):
            rc, it = hd.hdcg_coarse_solve(h.h, x, b, prec, nr, 1e-5 if prec == hd.DWF_C64 else 1e-3, 5000)
            assert rc == 0 and it > 0
        ax = torch.zeros((nr, Nc, nvec), device="cuda", dtype=torch.complex128)
        hd.coarse_apply(h.h, ax, x.to(torch.complex128), hd.DWF_C128, nr)
        for r in range(nr):
            res = ((b[r] - ax[r]).norm() / b[r].norm()).item()
            assert res <= (2e-5 if prec == hd.DWF_C64 else 2e-2), (nr, r, res, it)
    h.close()
    op.close()


@pytest.mark.parametrize("nvec,dims", [(12, (20, 20, 16, 16)), (64, (20, 20, 16, 16)), (33, (20, 20, 16, 16)),
                                       (10, (20, 20, 16, 16)), (16, (16, 16, 16, 16)), (28, (16, 16, 16, 16)),
                                       (32, (16, 16, 16, 16)), (16, (12, 20, 16, 16))])
def test_kept_rows_on_both_sides_of_their_rule(nvec, dims):
    """Where rows of the operator are kept on chip (more sites than CUs, or as
    many and an eighth of the rows, for an operator above 32 MB): all rows
    kept, a few, one row beyond a whole wave, and the cases beside the rule."""
    Ls = 1
    banner(f"coarse CG kept rows {dims} nvec {nvec}")
    op = hd.FineOperator(synth.gauge_field(dims, 0.3, 476), dims, Ls, 1.8, 0.3)
    h = hd.HDCG(op, (4, 4, 4, 4), synth.gaussian_half_field(dims, Ls, 477, nrhs=nvec))
    Nc = dims[0] * dims[1] * dims[2] * dims[3] // 256
    g = torch.Generator(device="cuda").manual_seed(8)
    b = torch.randn((1, Nc, nvec), generator=g, device="cuda", dtype=torch.complex64)
    x = torch.zeros_like(b)
    rc, it = hd.hdcg_coarse_solve(h.h, x, b, hd.DWF_C64, 1, 1e-5, 5000)
    assert rc == 0 and it > 0
    ax = torch.zeros((1, Nc, nvec), device="cuda", dtype=torch.complex128)
    hd.coarse_apply(h.h, ax, x.to(torch.complex128), hd.DWF_C128, 1)
    res = ((b - ax).norm() / b.norm()).item()
    assert res <= 2e-5, (res, it)
    h.close()
    op.close()
