"""The one-launch stages at the sizes where their sweep changes: one packet per
lane at most (up to 512 / ns stars) or packets through LDS, 1024 at a time;
and remainders of the stars per workgroup.  Three RK4 steps against the FP64
oracle, with the bounds of the other sizes."""
import numpy as np
import pytest

import oracle
from paper_1801_07986_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

G, C, EPS, DT = 1.0, 40.0, 1e-3, 1e-5


@pytest.fixture
def stage():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1801_07986_amd as pn
    from paper_1801_07986_amd import _binding

    pn.load()

    def force(ns):
        pn.pn_set_stage_kernel(-1, 0, 0, 0)
        for prec in (pn.PN_FP64, pn.PN_MIXED):
            pn.pn_set_stage_kernel(prec, 2, 1 << 28, ns)
        return pn

    yield force
    _binding.install_tuned_shapes()


@pytest.mark.parametrize("ns,stars", [(2, 255), (2, 256), (2, 257), (4, 128), (4, 129), (8, 64),
                                      (8, 65), (16, 32), (16, 33), (8, 1024), (8, 1025),
                                      (4, 2049), (16, 2048)])
def test_stage_edges(stage, ns, stars):
    pn = stage(ns)
    pos, vel, mass = inputs.plummer_bh(stars + 1, 0.1, 700 + stars)
    rp, rv = oracle.step(pos, vel, mass, G, C, EPS, DT, 3)
    for prec, tx, tv in ((pn.PN_FP64, 1e-12, 1e-12), (pn.PN_MIXED, 1e-8, 1e-6)):
        print(f"[case] ns={ns} stars={stars} prec={prec}", flush=True)
        P, V, M = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (pos, vel, mass))
        pn.pn_step(P, V, M, G, C, EPS, DT, 3, prec)
        dp = np.abs(P.cpu().numpy() - rp).max() / np.abs(rp).max()
        dv = np.abs(V.cpu().numpy() - rv).max() / np.abs(rv).max()
        assert dp <= tx and dv <= tv
