"""The hop's launch shape belongs to a field storage and to one or several
right-hand sides: what the autotuner chose for one does not enter another's
calls."""
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

DEFAULT = (2, 2, 1, 1, 1, 0, 0, 1, 0, 1)


def test_a_choice_stays_with_its_storage_and_count():
    dims, Ls = (16, 16, 16, 8), 16
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


@pytest.mark.parametrize("mobius", [False, True])
@pytest.mark.parametrize("Ls", [6, 10, 14])
def test_even_ls_against_oracle(Ls, mobius):
    """The even Ls with code of their own that no other test covers, on
    several right-hand sides at once and one, straight-line and looping.
    Tolerances as for the other fine-operator tests."""
    dims, nr = (6, 4, 4, 4), 3
    banner(f"hop Ls{Ls} mobius={mobius}")
    U = synth.gauge_field(dims, 0.7, 173 + Ls)
    op = hd.FineOperator(U, dims, Ls, 1.8, 0.02, **(dict(b5=1.5, c5=0.5) if mobius else {}))
    ref = DWF(U, dims, Ls, 1.8, 0.02, **({"b": 1.5, "c": 0.5} if mobius else {}))
    b = synth.gaussian_half_field(dims, Ls, 174 + Ls, nrhs=nr)
    for shape in ((0, 0, 0, 0, 0, 0, 0, 0, 0, 1), (1, 2, 2, 2, 0, 0, 0, 0, 0, 2)):
        hd.dwf_set_hop_shape(op.h, shape)
        for n in (1, nr):
            want = [ref.H(v) for v in b[:n]]
            for prec, tol in ((hd.DWF_C128, 1e-12), (hd.DWF_C64, 5e-6)):
                got = op.to_canonical(op.H(op.to_native(b[:n], prec), prec, n), prec, n).cpu().numpy().reshape(b[:n].shape)
                for r in range(n):
                    assert rel_err(got[r], want[r]) < tol, (shape, n, prec, r)
            # 16 bits: four stored fields round to 2^-8 each
            x16 = op.convert(op.to_native(b[:n], hd.DWF_C64), hd.DWF_BF16, hd.DWF_C64, n)
            xin = op.to_canonical(op.convert(x16, hd.DWF_C64, hd.DWF_BF16, n), hd.DWF_C64, n).cpu().numpy().reshape(b[:n].shape)
            y = op.convert(op.H(x16, hd.DWF_BF16, n), hd.DWF_C64, hd.DWF_BF16, n)
            got = op.to_canonical(y, hd.DWF_C64, n).cpu().numpy().reshape(b[:n].shape)
            for r in range(n):
                exact = ref.H(xin[r].astype(np.complex128))
                assert np.linalg.norm((got[r] - exact).ravel()) / np.linalg.norm(exact.ravel()) < 4 * 2.0 ** -8, (shape, n, r)
    op.close()


def test_streaming_follows_the_shape():
    """Non-temporal accesses are an entry of the shape: on by default in
    complex128 where the links exceed 32 MB (16^4: 37.7 MB), off and on as a
    fixed shape says; the same bits either way."""
    dims, Ls = (16, 16, 16, 16), 4
    banner("streaming in the launch shape")
    U = synth.gauge_field(dims, 0.7, 175)
    op = hd.FineOperator(U, dims, Ls, 1.8, 0.02)
    small = hd.FineOperator(synth.gauge_field((8, 8, 8, 8), 0.7, 175), (8, 8, 8, 8), Ls, 1.8, 0.02)
    assert hd.dwf_get_hop_shape(op.h, hd.DWF_C128, 1)[0][6] == 1
    assert hd.dwf_get_hop_shape(op.h, hd.DWF_C64, 1)[0][6] == 0
    assert hd.dwf_get_hop_shape(small.h, hd.DWF_C128, 1)[0][6] == 0
    x = op.to_native(synth.gaussian_half_field(dims, Ls, 176))
    out = []
    for nt in (0, 1):
        hd.dwf_set_hop_shape(op.h, (2, 2, 1, 1, 1, 0, nt, 1, 0, 1))
        assert hd.dwf_get_hop_shape(op.h, hd.DWF_C128, 1)[0][6] == nt
        out.append(op.H(x))
    assert torch.equal(out[0], out[1])
    op.close()
    small.close()
