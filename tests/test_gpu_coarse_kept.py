"""The complex64 coarse CG of one right-hand side keeps part of its operator in
registers and LDS: vector counts whose rows all fit the registers, end inside
the LDS part, leave threads idle or fill the workgroup, on fewer coarse sites
than workgroups and on more (only a workgroup's first site is kept).

The solution's residual is measured with the complex128 mat-vec.  The CG stops
at a recursive residual of 1e-5; the true one drifts from it by rounding, at
most 6e-8 a step relative to |b| for some tens of steps: 2e-5 in all."""
import pytest

import synth
from tests.gpu_util import banner

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1402_2585_amd as hd  # noqa: E402


@pytest.mark.parametrize("nvec,dims", [(1, (12, 12, 12, 12)), (4, (12, 12, 12, 16)), (7, (12, 12, 12, 12)),
                                       (20, (12, 12, 12, 12)), (40, (12, 12, 12, 12)), (64, (12, 12, 12, 12)),
                                       (12, (24, 24, 24, 12))])
def test_kept_rows_solve_to_tolerance(nvec, dims):
    Ls = 1
    banner(f"coarse CG with kept rows {dims} nvec {nvec}")
    op = hd.FineOperator(synth.gauge_field(dims, 0.3, 470), dims, Ls, 1.8, 0.3)
    h = hd.HDCG(op, (4, 4, 4, 4), synth.gaussian_half_field(dims, Ls, 471, nrhs=nvec))
    Nc = dims[0] * dims[1] * dims[2] * dims[3] // 256
    g = torch.Generator(device="cuda").manual_seed(5)
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


@pytest.mark.parametrize("nvec,nr,prec,dims", [(8, 4, hd.DWF_C64, (12, 12, 12, 12)), (8, 15, hd.DWF_C64, (12, 12, 12, 12)),
                                               (8, 16, hd.DWF_C64, (12, 12, 12, 12)), (7, 2, hd.DWF_C64, (12, 12, 12, 16)),
                                               (7, 6, hd.DWF_C64, (12, 12, 12, 12)), (9, 14, hd.DWF_C64, (12, 12, 12, 12)),
                                               (40, 3, hd.DWF_C64, (12, 12, 12, 12)), (12, 3, hd.DWF_C64, (24, 24, 24, 12)),
                                               (8, 4, hd.DWF_BF16, (12, 12, 12, 16)), (12, 10, hd.DWF_BF16, (12, 12, 12, 12)),
                                               (12, 11, hd.DWF_BF16, (12, 12, 12, 12)), (40, 3, hd.DWF_F16, (12, 12, 12, 12))])
def test_several_right_hand_sides_solve_to_tolerance(nvec, nr, prec, dims):
    Ls = 1
    banner(f"coarse CG staged {dims} nvec {nvec} nr {nr} prec {prec}")
    op = hd.FineOperator(synth.gauge_field(dims, 0.3, 472), dims, Ls, 1.8, 0.3)
    h = hd.HDCG(op, (4, 4, 4, 4), synth.gaussian_half_field(dims, Ls, 473, nrhs=nvec))
    Nc = dims[0] * dims[1] * dims[2] * dims[3] // 256
    g = torch.Generator(device="cuda").manual_seed(6)
    b = torch.randn((nr, Nc, nvec), generator=g, device="cuda", dtype=torch.complex64)
    b[nr - 1] *= 1e-3
    x = torch.zeros_like(b)
    rc, it = hd.hdcg_coarse_solve(h.h, x, b, prec, nr, 1e-5 if prec == hd.DWF_C64 else 1e-3, 5000)
    assert rc == 0 and it > 0
    ax = torch.zeros((nr, Nc, nvec), device="cuda", dtype=torch.complex128)
    hd.coarse_apply(h.h, ax, x.to(torch.complex128), hd.DWF_C128, nr)
    for r in range(nr):
        res = ((b[r] - ax[r]).norm() / b[r].norm()).item()
        assert res <= (2e-5 if prec == hd.DWF_C64 else 2e-2), (r, res, it)
    h.close()
    op.close()
