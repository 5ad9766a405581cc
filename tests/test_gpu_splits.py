"""Sweep splits by the rule (shape entries with 0 splits, eight wavefronts): odd
shares of workgroups per CU, i-blocks padded to the eight XCDs (one i per lane)
or by a column (two), remainders.  Two chained steps against the same steps in
a fixed shape of four wavefronts and 16 splits, whose sums differ by rounding."""
import numpy as np
import pytest

from paper_1801_07986_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

G, C, EPS, DT = 1.0, 40.0, 1e-3, 1e-5


@pytest.fixture
def steps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1801_07986_amd as pn
    from paper_1801_07986_amd import _binding

    pn.load()

    def run(N, prec, shape):
        pn.pn_set_shape(-1, 0, 0, 0, 0, 0)
        pn.pn_set_stage_kernel(-1, 0, 0, 0)
        pn.pn_set_shape(prec, N, N, *shape)
        pos, vel, mass = inputs.plummer_bh(N, 0.1, N)
        P, V, M = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (pos, vel, mass))
        used = pn.pn_query_shape(prec, N)
        pn.pn_step(P, V, M, G, C, EPS, DT, 2, prec)
        return P.cpu().numpy(), V.cpu().numpy(), used

    yield run
    _binding.install_tuned_shapes()


@pytest.mark.parametrize("N,ipt", [(2, 1), (33, 1), (129, 1), (600, 1), (1450, 1), (2306, 1),
                                   (3009, 1), (4097, 1), (8193, 1), (8193, 2), (9001, 2),
                                   (16385, 2), (30722, 1)])
def test_rule_against_fixed_shape(steps, N, ipt):
    for prec, tx, tv in ((0, 1e-12, 1e-12), (1, 1e-8, 1e-6)):
        print(f"[case] N={N} ipt={ipt} prec={prec}", flush=True)
        p, v, used = steps(N, prec, (ipt, 8, 0))
        q, w, _ = steps(N, prec, (1, 4, 16))
        assert used[0] == ipt and used[1] == 8 and 1 <= used[2] <= 16
        assert np.abs(p - q).max() <= tx * np.abs(q).max()
        assert np.abs(v - w).max() <= tv * np.abs(w).max()
