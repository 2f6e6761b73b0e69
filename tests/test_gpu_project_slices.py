"""Project onto a 16-bit subspace for several right-hand sides, a block's
entries split over several workgroups on small coarse grids: both sides of the
slice count (many slices, two, one), a second group of right-hand sides, and a
first use inside a captured graph, which has no room for slices yet.

Against the form for one right-hand side: the same exact products, so only the
order of the FP32 sums differs.  A sum of n values of random sign in FP32 is
off by at most 2^-25 sqrt(n / 2) of its size, 3.3e-6 for the longest here
(24576 entries), in either form: 1e-5 norm-wise."""
import pytest

import synth
from tests.gpu_util import banner

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1402_2585_amd as hd  # noqa: E402


def _setup(dims, Ls, nvec, nr):
    op = hd.FineOperator(synth.gauge_field(dims, 0.3, 480), dims, Ls, 1.8, 0.3)
    h = hd.HDCG(op, (4, 4, 4, 4), synth.gaussian_half_field(dims, Ls, 481, nrhs=nvec))
    x = op.to_native(synth.gaussian_half_field(dims, Ls, 482, nrhs=nr), hd.DWF_C64)
    n = x.numel() // nr
    want = h.new_coarse(hd.DWF_C64, nr)
    m = want.numel() // nr
    for r in range(nr):
        one = h.new_coarse(hd.DWF_C64, 1)
        hd.hdcg_project(h.h, one, x[r * n:(r + 1) * n].contiguous(), hd.DWF_BF16, 1)
        want.view(-1)[r * m:(r + 1) * m] = one.view(-1)
    return op, h, x, want


def _err(a, b):
    return ((a - b).norm() / b.norm()).item()


@pytest.mark.parametrize("dims,Ls,nvec,nr", [((12, 12, 12, 12), 16, 8, 2), ((12, 12, 12, 12), 16, 20, 17),
                                             ((12, 12, 12, 12), 2, 8, 3), ((16, 16, 16, 32), 4, 8, 4),
                                             ((16, 16, 16, 32), 4, 8, 17), ((20, 16, 16, 32), 2, 4, 2)])
def test_slices_against_one_right_hand_side(dims, Ls, nvec, nr):
    banner(f"project slices {dims} x Ls{Ls} nvec {nvec} nr {nr}")
    op, h, x, want = _setup(dims, Ls, nvec, nr)
    for _ in range(3):  # the tickets are zero again after each
        got = h.new_coarse(hd.DWF_C64, nr)
        hd.hdcg_project(h.h, got, x, hd.DWF_BF16, nr)
        assert _err(got, want) < 1e-5
    h.close()
    op.close()


def test_first_use_in_a_captured_graph():
    banner("project captured first")
    nr = 5
    op, h, x, want = _setup((12, 12, 12, 12), 8, 8, nr)
    got, eager = h.new_coarse(hd.DWF_C64, nr), h.new_coarse(hd.DWF_C64, nr)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        hd.hdcg_project(h.h, got, x, hd.DWF_BF16, nr)
    for _ in range(3):
        got.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert _err(got, want) < 1e-5
        eager.zero_()
        hd.hdcg_project(h.h, eager, x, hd.DWF_BF16, nr)
        torch.cuda.synchronize()
        assert _err(eager, want) < 1e-5
    h.close()
    op.close()
