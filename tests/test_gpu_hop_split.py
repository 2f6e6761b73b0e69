"""GPU parity of the hop stage split over a wave's rows (Ls <= 16) and of its
form marched along t, at every
packing of sites into the 16-lane rows (one to sixteen sites, full rows and
rows with idle lanes) and on both sides of its Ls limit, Shamir and Mobius,
against the oracle.

Tolerances as for the other fine-operator tests: 1e-12 in complex128, 5e-6 in
complex64 (max-norm); 16-bit fields against exact FP64 within four times the
unit roundoff 2^-8 (each stored field rounds once)."""
import numpy as np
import pytest

import synth
from oracle.dwf import DWF
from tests.gpu_util import banner, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1402_2585_amd as hd  # noqa: E402


@pytest.mark.parametrize("mobius", [False, True])
@pytest.mark.parametrize("Ls", [1, 2, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17])
def test_every_row_packing_against_oracle(Ls, mobius):
    dims, nr = (6, 4, 4, 4), 2
    banner(f"hop split {dims} x Ls{Ls} mobius={mobius}")
    U = synth.gauge_field(dims, 0.7, 170 + Ls)
    kw = dict(b5=1.5, c5=0.5) if mobius else {}
    op = hd.FineOperator(U, dims, Ls, 1.8, 0.02, (1, np.exp(0.3j), 1, -1), **kw)
    ref = DWF(U, dims, Ls, 1.8, 0.02, (1, np.exp(0.3j), 1, -1), **({"b": 1.5, "c": 0.5} if mobius else {}))
    b = synth.gaussian_half_field(dims, Ls, 190 + Ls, nrhs=nr)
    for shape in (None, (0, 0, 0, 0, 0, 0, 0, 0, 0, 1), (1, 2, 2, 2, 0, 0, 1, 0, 0, 2)):
        if shape:
            hd.dwf_set_hop_shape(op.h, shape)
        for dag in (0, 1):
            want = [ref.mpc_dag(v) if dag else ref.mpc(v) for v in b]
            for prec, tol in ((hd.DWF_C128, 1e-12), (hd.DWF_C64, 5e-6)):
                got = op.to_canonical(op.mpc(op.to_native(b, prec), prec, dag, nr), prec, nr).cpu().numpy()
                for r in range(nr):
                    assert rel_err(got[r], want[r]) < tol, (shape, dag, prec, r)
            x16 = op.convert(op.to_native(b, hd.DWF_C64), hd.DWF_BF16, hd.DWF_C64, nr)
            xin = op.to_canonical(op.convert(x16, hd.DWF_C64, hd.DWF_BF16, nr), hd.DWF_C64, nr).cpu().numpy()
            y16 = op.mpc(x16, hd.DWF_BF16, dag, nr)
            got = op.to_canonical(op.convert(y16, hd.DWF_C64, hd.DWF_BF16, nr), hd.DWF_C64, nr).cpu().numpy()
            for r in range(nr):
                v = xin[r].astype(np.complex128)
                exact = ref.mpc_dag(v) if dag else ref.mpc(v)
                e = np.linalg.norm((got[r] - exact).ravel()) / np.linalg.norm(exact.ravel())
                assert e < 4 * 2.0 ** -8, (shape, dag, r, e)
    op.close()


@pytest.mark.parametrize("Ls,block", [(16, (2, 4, 2, 4)), (16, (2, 2, 2, 8)), (16, (1, 2, 2, 8)), (12, (1, 2, 2, 8)),
                                      (8, (2, 4, 4, 2)), (8, (2, 2, 2, 8))])
def test_marched_along_t_against_oracle(Ls, block):
    """A block of more than 256 / Ls sites is marched along t: chunks that
    cover T once and several times, tiles whose neighbour across the face is
    the tile itself (extents equal to the lattice's), one and three right-hand
    sides on 8 and on 6 tiles a chunk (the folded grid and the plain one)."""
    dims, nr = ((8, 8, 4, 8) if block != (1, 2, 2, 8) else (6, 4, 4, 8)), 3
    banner(f"hop march {dims} x Ls{Ls} block {block}")
    U = synth.gauge_field(dims, 0.7, 270 + Ls)
    op = hd.FineOperator(U, dims, Ls, 1.8, 0.02)
    split = hd.FineOperator(U, dims, Ls, 1.8, 0.02)
    ref = DWF(U, dims, Ls, 1.8, 0.02)
    hd.dwf_set_hop_shape(op.h, block + (1, 0, 0, 4, 0, 1))
    hd.dwf_set_hop_shape(split.h, (1, 2, 2, 1, 1, 0, 0, 4, 0, 1))
    b = synth.gaussian_half_field(dims, Ls, 290 + Ls, nrhs=nr)
    want = [ref.H(v) for v in b]
    for n in (1, nr):
        for prec, tol in ((hd.DWF_C128, 1e-12), (hd.DWF_C64, 5e-6)):
            got = op.to_canonical(op.H(op.to_native(b[:n], prec), prec, n), prec, n).cpu().numpy().reshape(b[:n].shape)
            for r in range(n):
                assert rel_err(got[r], want[r]) < tol, (n, prec, r)
        x16 = op.convert(op.to_native(b[:n], hd.DWF_C64), hd.DWF_BF16, hd.DWF_C64, n)
        got, one = op.H(x16, hd.DWF_BF16, n).double(), split.H(x16, hd.DWF_BF16, n).double()
        # the same roundings but for sums that differ in the last FP32 place
        assert ((got - one).norm() / one.norm()).item() < 2e-4
    # M_IRS-style use: the fused norm of the stages, through a CG
    x = op.new_field(zero=True)
    rc, st = hd.cg_solve(op.h, x, op.to_native(b[0]), 1, 1e-8, 5000)
    assert rc == 0 and st["converged"] == 1
    r = b[0] - ref.H(op.to_canonical(x).cpu().numpy())
    assert np.sqrt(np.vdot(r, r).real / np.vdot(b[0], b[0]).real) <= 1e-8
    op.close()
    split.close()
