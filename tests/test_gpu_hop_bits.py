"""Every launch shape of the hop stages gives the same bits of M_pc, its
adjoint and H: linear and blocked, one site a wave and several, one right-hand
side a workgroup and several, marched along t, any order; Ls <= 16 and, with
either number of load phases, above.  A tuned operator's results are then the
same whichever shape the tuner measured to be the fastest."""
import pytest

import synth
from oracle.dwf import DWF
from tests.gpu_util import banner, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1402_2585_amd as hd  # noqa: E402

DIMS = (8, 8, 4, 8)
LINEAR = (0, 0, 0, 0, 0, 0, 0, 0, 0, 1)
SPLIT = [(2, 2, 1, 1, 1, 0, 0, 1, 0, 1), (1, 2, 2, 1, 1, 0, 1, 4, 0, 3), (2, 2, 2, 2, 1, 0, 0, 2, 0, 1),
         (0, 0, 0, 0, 1, 16, 0, 0, 0, 2)]
MARCH = [(2, 4, 2, 4, 1, 0, 0, 4, 0, 1), (2, 2, 2, 8, 0, 0, 1, 3, 0, 1)]


def _fields(op, b, prec, n):
    x = op.to_native(b[:n], hd.DWF_C64 if prec == hd.DWF_BF16 else prec)
    return op.convert(x, hd.DWF_BF16, hd.DWF_C64, n) if prec == hd.DWF_BF16 else x


@pytest.mark.parametrize("Ls,mobius", [(16, False), (16, True), (12, False), (12, True), (8, False), (10, False), (6, True),
                                       (5, False), (3, True)])
def test_same_bits_for_every_shape(Ls, mobius):
    banner(f"bits of every launch shape Ls{Ls} mobius={mobius}")
    U = synth.gauge_field(DIMS, 0.7, 180 + Ls)
    kw = dict(b5=1.5, c5=0.5) if mobius else {}
    op, ref = hd.FineOperator(U, DIMS, Ls, 1.8, 0.02, **kw), hd.FineOperator(U, DIMS, Ls, 1.8, 0.02, **kw)
    hd.dwf_set_hop_shape(ref.h, LINEAR)
    b = synth.gaussian_half_field(DIMS, Ls, 181, nrhs=3)
    for prec in (hd.DWF_C128, hd.DWF_C64, hd.DWF_BF16):
        for n in (1, 3):
            x = _fields(ref, b, prec, n)
            want = [ref.mpc(x, prec, 0, n), ref.mpc(x, prec, 1, n), ref.H(x, prec, n)]
            for shape in SPLIT + MARCH:
                hd.dwf_set_hop_shape(op.h, shape)
                got = [op.mpc(x, prec, 0, n), op.mpc(x, prec, 1, n), op.H(x, prec, n)]
                for k in range(3):
                    assert torch.equal(got[k], want[k]), (prec, n, shape, k)
    op.close()
    ref.close()


@pytest.mark.parametrize("Ls,mobius", [(17, False), (20, False), (24, True)])
def test_shapes_above_16_slices(Ls, mobius):
    """Blocks, orders and load phases of the form for Ls > 16 against the
    oracle (1e-12 in complex128, 5e-6 in complex64, max-norm)."""
    banner(f"launch shapes Ls{Ls} mobius={mobius}")
    U = synth.gauge_field(DIMS, 0.7, 182 + Ls)
    op = hd.FineOperator(U, DIMS, Ls, 1.8, 0.02, **(dict(b5=1.5, c5=0.5) if mobius else {}))
    ref = DWF(U, DIMS, Ls, 1.8, 0.02, **({"b": 1.5, "c": 0.5} if mobius else {}))
    b = synth.gaussian_half_field(DIMS, Ls, 183, nrhs=1)
    want = ref.H(b[0])
    for block in ((0, 0, 0, 0), (2, 2, 1, 1), (1, 2, 2, 1)):
        for order in (0, 2, 3, 4):
            for phases in (2, 4):
                hd.dwf_set_hop_shape(op.h, block + (1, 0, 0, order, phases, 1))
                for prec, tol in ((hd.DWF_C128, 1e-12), (hd.DWF_C64, 5e-6)):
                    got = op.to_canonical(op.H(op.to_native(b, prec), prec, 1), prec, 1).cpu().numpy().reshape(b.shape)
                    assert rel_err(got[0], want) < tol, (block, order, phases, prec)
    op.close()
