"""The hop's launch shape belongs to a field storage and to one or several
right-hand sides: what the autotuner chose for one does not enter another's
calls."""
import pytest

import synth
from tests.gpu_util import banner

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1402_2585_amd as hd  # noqa: E402

DEFAULT = (2, 2, 1, 1, 1, 0, 0, 1, 0, 1)


def test_a_choice_stays_with_its_storage_and_count():
    dims, Ls = (16, 16, 16, 16), 16
    banner("launch shape per storage")
    U = synth.gauge_field(dims, 0.7, 171)
    op, fresh = hd.FineOperator(U, dims, Ls, 1.8, 0.02), hd.FineOperator(U, dims, Ls, 1.8, 0.02)
    b = synth.gaussian_half_field(dims, Ls, 172, nrhs=2)
    hd.dwf_tune_hop(op.h, hd.DWF_C64, 1)
    shape, _, tuned = hd.dwf_get_hop_shape(op.h, hd.DWF_C64, 1)
    assert tuned
    print("complex64:", shape, flush=True)
    for prec, n in ((hd.DWF_C64, 2), (hd.DWF_C128, 1), (hd.DWF_C128, 2), (hd.DWF_BF16, 1), (hd.DWF_BF16, 2)):
        got, _, tuned = hd.dwf_get_hop_shape(op.h, prec, n)
        assert not tuned and tuple(got) == DEFAULT, (prec, n, got)
        x = op.to_native(b[:n], hd.DWF_C64 if prec == hd.DWF_BF16 else prec)
        if prec == hd.DWF_BF16:
            x = op.convert(x, hd.DWF_BF16, hd.DWF_C64, n)
        for dag in (0, 1):
            assert torch.equal(op.mpc(x, prec, dag, n), fresh.mpc(x, prec, dag, n)), (prec, n, dag)
    # a fixed shape serves every storage, and leaves nothing behind
    fixed = (1, 2, 2, 1, 0, 8, 1, 4, 2, 2)
    hd.dwf_set_hop_shape(op.h, fixed)
    assert tuple(hd.dwf_get_hop_shape(op.h, hd.DWF_BF16, 1)[0]) == fixed
    hd.dwf_set_hop_shape(op.h, (-1,) + (0,) * 9)
    assert tuple(hd.dwf_get_hop_shape(op.h, hd.DWF_C64, 1)[0]) == tuple(shape)
    assert tuple(hd.dwf_get_hop_shape(op.h, hd.DWF_C128, 1)[0]) == DEFAULT
    op.close()
    fresh.close()
