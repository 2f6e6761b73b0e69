"""CG steps whose last hop stage updates the residual (Ls <= 16, split and
marched) and the form with one more kernel (Ls > 16), against the oracle: the
fixed-count CG with a shift on one and three right-hand sides, of one step
(no residual at all) and of three, and the CG solvers without a shift.

Tolerances: complex64 2e-5 (max-norm, as M_IRS's other tests), 16-bit fields
2e-2 norm-wise (theirs for seven steps)."""
import numpy as np
import pytest

import synth
from oracle import hdcg as ohdcg
from oracle.dwf import DWF
from tests.gpu_util import banner, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1402_2585_amd as hd  # noqa: E402

DIMS = (12, 12, 12, 12)
SPLIT, MARCH, LINEAR = (1, 2, 2, 1), (2, 2, 2, 4), (0, 0, 0, 0)


@pytest.mark.parametrize("Ls,mobius,block,rg", [(16, False, SPLIT, 1), (16, False, MARCH, 1), (16, False, SPLIT, 2),
                                                (12, False, MARCH, 1), (12, True, LINEAR, 1), (8, False, LINEAR, 2),
                                                (5, True, SPLIT, 1), (3, False, LINEAR, 1), (20, False, SPLIT, 1)])
def test_cg_steps_against_oracle(Ls, mobius, block, rg):
    banner(f"CG steps {DIMS} x Ls{Ls} mobius={mobius} block {block} rg {rg}")
    U = synth.gauge_field(DIMS, 0.7, 370 + Ls)
    op = hd.FineOperator(U, DIMS, Ls, 1.8, 0.05, **(dict(b5=1.5, c5=0.5) if mobius else {}))
    hd.dwf_set_hop_shape(op.h, block + (1, 0, 0, 0, 0, rg))
    ref = DWF(U, DIMS, Ls, 1.8, 0.05, **({"b": 1.5, "c": 0.5} if mobius else {}))
    h = hd.HDCG(op, (4, 4, 4, 4), synth.gaussian_half_field(DIMS, Ls, 380, nrhs=2))
    b = synth.gaussian_half_field(DIMS, Ls, 390, nrhs=3).astype(np.complex64).astype(np.complex128)
    for steps in (1, 3):
        want = {r: ohdcg.m_irs(ref, b[r], steps, 1.0) for r in (0, 2)}
        for n in (1, 3):
            for prec, tol in ((hd.DWF_C64, 2e-5), (hd.DWF_BF16, 2e-2)):
                h.set_params(irs_prec=prec, n_irs=steps)
                out = op.new_field(hd.DWF_C64, n)
                out.fill_(1.0)
                hd.hdcg_mirs(h.h, out, op.to_native(b[:n], hd.DWF_C64), n)
                got = op.to_canonical(out, hd.DWF_C64, n).cpu().numpy().reshape(b[:n].shape)
                for r in {0, n - 1}:
                    e = (rel_err(got[r], want[r]) if prec == hd.DWF_C64
                         else np.linalg.norm((got[r] - want[r]).ravel()) / np.linalg.norm(want[r].ravel()))
                    assert e < tol, (steps, n, prec, r, e)
    x = op.new_field(zero=True)
    for solve in (hd.cg_solve, hd.cg_solve_mixed):
        x.zero_()
        rc, st = solve(op.h, x, op.to_native(b[0]), 1, 1e-8)
        assert rc == 0 and st["converged"] == 1
        r = b[0] - ref.H(op.to_canonical(x).cpu().numpy().reshape(b[0].shape))
        assert np.sqrt(np.vdot(r, r).real / np.vdot(b[0], b[0]).real) <= 1e-8
    h.close()
    op.close()
