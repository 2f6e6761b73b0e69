"""Rounding error of the hop stage's M_5^-1 (Ls <= 16), isolated from the rest
of the operator.

With unit links in x and none in y, z, t, an input of small integers on the
odd sites of one x plane reaches the planes two sites away only through
Dh M_5^-1 Dh / 4: the first hop is exact, the second adds two numbers.  M_5^-1's
own error is then most of what is left.

Tolerance, in units of 2^-24 (complex64) and 2^-53 (complex128), root mean
square over 10^4 values and more, relative to theirs: the O(Ls) recurrence
y_s = x_s / alpha + kap y_{s-1} with its two roundings a slice, then the sum and
the factor 1/4, has 0.96 to 0.98 units at kap = 1 / 3.3 for these Ls (numpy
emulation of the same inputs).  M_5^-1 must not be further off than that; 5 %
for the finite sample: 1.03."""
import numpy as np
import pytest

from oracle.gamma import gammas
from tests.gpu_util import banner

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1402_2585_amd as hd  # noqa: E402

DIMS, X0, M5, MASS = (8, 4, 4, 8), 2, 1.7, 0.01


def _exact(psi, Ls, step, dag):
    """-1/4 (1 + sign g_x) M_5^-1 (1 + sign g_x) psi of [site][s][spin][colour] in 80-bit arithmetic."""
    ld = np.longdouble
    alpha, m = ld((4 - M5) + 1), ld(MASS)
    kap = 1 / alpha
    pw = [kap ** n / (alpha * (1 + m * kap ** Ls)) for n in range(Ls)]
    low = np.array([[pw[(s - t) % Ls] * (1 if s >= t else -m) for t in range(Ls)] for s in range(Ls)])
    up = low.T
    if dag:
        low, up = up, low
    # a neighbour at x - 1 (step +1) enters with 1 + g_x, one at x + 1 with 1 - g_x; swapped in the adjoint
    G = (np.eye(4) + (step if not dag else -step) * gammas()[0]).astype(np.clongdouble)

    def spin(f):
        return np.stack([sum(G[i, j] * f[:, :, j] for j in range(4)) for i in range(4)], 2)

    f = spin(psi.astype(np.clongdouble))
    g = np.empty_like(f)
    for half, a in ((0, low), (1, up)):
        for s in range(Ls):
            g[:, s, 2 * half:2 * half + 2] = sum(a[s, t] * f[:, t, 2 * half:2 * half + 2] for t in range(Ls))
    return -spin(g) / 4


@pytest.mark.parametrize("dag", [0, 1])
@pytest.mark.parametrize("Ls", [4, 7, 8, 12, 16])
def test_m5_inverse_rounds_no_worse_than_the_recurrence(Ls, dag):
    banner(f"rounding of M_5^-1 Ls{Ls} dag={dag}")
    X, Y, Z, T = DIMS
    U = np.zeros((T, Z, Y, X, 4, 3, 3), dtype=np.complex128)
    U[..., 0, :, :] = np.eye(3)
    op = hd.FineOperator(U, DIMS, Ls, M5, MASS)
    rng = np.random.default_rng(50 + Ls)
    n = X * Y * Z * T // 2
    b = np.zeros((Ls, n, 4, 3), dtype=np.complex128)
    rows = [(y, z, t) for t in range(T) for z in range(Z) for y in range(Y) if (X0 + y + z + t) % 2]
    cb = np.array([((X0 + X * (y + Y * (z + Z * t))) >> 1) for y, z, t in rows])
    b[:, cb] = rng.integers(-1000, 1001, (Ls, len(rows), 4, 3)) + 1j * rng.integers(-1000, 1001, (Ls, len(rows), 4, 3))
    psi = b[:, cb].transpose(1, 0, 2, 3)
    for prec, eps in ((hd.DWF_C64, 2.0 ** -24), (hd.DWF_C128, 2.0 ** -53)):
        got = op.to_canonical(op.mpc(op.to_native(b, prec), prec, dag, 1), prec, 1).cpu().numpy().reshape(b.shape)
        e2 = w2 = 0.0
        for step in (1, -1):
            # parity of a site two further on in x is the same, and its checkerboard index one further on
            out = got[:, cb + step].transpose(1, 0, 2, 3)
            want = _exact(psi, Ls, step, dag)
            e2 += float((np.abs(out.astype(np.clongdouble) - want) ** 2).sum())
            w2 += float((np.abs(want) ** 2).sum())
        units = np.sqrt(e2 / w2) / eps
        print(prec, "rms error", round(units, 4), flush=True)
        assert units < 1.03, (prec, units)
    op.close()
