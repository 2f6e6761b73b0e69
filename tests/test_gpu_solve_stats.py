"""hdcg_solve's count of applications of H: an M_IRS of n steps applies H n - 1
times and M_pc once more."""
import pytest

import synth
from tests.gpu_util import banner

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1402_2585_amd as hd  # noqa: E402


@pytest.mark.parametrize("n_irs,graph", [(1, 1), (4, 1), (7, 0)])
def test_mirs_applications(n_irs, graph):
    banner(f"matmuls of M_IRS({n_irs}) graph {graph}")
    dims, Ls = (12, 12, 12, 12), 4
    op = hd.FineOperator(synth.gauge_field(dims, 0.3, 490), dims, Ls, 1.8, 0.1)
    h = hd.HDCG(op, (4, 4, 4, 4), synth.gaussian_half_field(dims, Ls, 491, nrhs=8), n_irs=n_irs, graph=graph,
                irs_prec=hd.DWF_BF16)
    x = op.new_field(zero=True)
    rc, st = hd.hdcg_solve(h.h, x, op.to_native(synth.gaussian_half_field(dims, Ls, 492)), 1, 1e-8)
    assert rc == 0
    # one M_IRS (on 16-bit fields, nothing else is) for each application of Q but
    # those that start an inner solve
    uses = st["matmuls_bf16"] / (n_irs - 0.5)
    print(n_irs, st["matmuls_bf16"], st["coarse_solves"], st["inner_iterations"], flush=True)
    assert uses == int(uses) and st["inner_iterations"] <= uses <= st["coarse_solves"]
    h.close()
    op.close()
