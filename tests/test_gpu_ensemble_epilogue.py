"""The epilogue of an ensemble in its three forms (nine, five and four wavefronts
per workgroup, by the number of workgroups): they add the same sums, so the
members of a large ensemble equal those of a small one bit for bit."""
import numpy as np
import pytest

from paper_1801_07986_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

G, C, EPS, DT = 1.0, 20.0, 1e-3, 1e-4


@pytest.fixture
def pn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1801_07986_amd as pkg
    from paper_1801_07986_amd import _binding

    pkg.load()
    yield pkg
    _binding.install_tuned_shapes()


def _run(pn, N, copies, prec):
    """Two different systems of N bodies, in turn, `copies` times."""
    parts = [inputs.plummer_bh(N, 0.1, 800 + N + k) for k in range(2)]
    P, V, M = (torch.from_numpy(np.concatenate([parts[k % 2][i] for k in range(copies)])).cuda()
               for i in range(3))
    off = [N * k for k in range(copies + 1)]
    pn.pn_step_batched(off, [G] * copies, [C] * copies, [EPS] * copies, P, V, M, DT, 2, prec)
    return P.reshape(copies, N, 3), V.reshape(copies, N, 3)


# one star, a whole block, remainders; splits 1 to 3 and 9 (two ranges of 5 and 4)
@pytest.mark.parametrize("N,splits", [(2, 1), (65, 1), (66, 2), (300, 2), (400, 3), (1200, 9)])
@pytest.mark.parametrize("prec", [0, 1])
def test_forms_agree_bit_for_bit(pn, N, splits, prec):
    pn.pn_set_batch_shape(prec, 1, splits)
    blocks = (N - 1 + 63) // 64
    p, v = _run(pn, N, 2, prec)
    assert torch.isfinite(p).all()
    assert N == 2 or not torch.equal(p[0], p[1])  # (a single star is centred: one system)
    for wgs in (256, 257, 512, 513, 1025):
        copies = (wgs - 1) // blocks + 1
        print(f"[case] N={N} splits={splits} prec={prec} workgroups={copies * blocks}", flush=True)
        q, w = _run(pn, N, copies, prec)
        for k in range(2):
            assert bool((q[k::2] == p[k]).all()) and bool((w[k::2] == v[k]).all())
