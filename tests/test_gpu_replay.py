"""Runs long enough to replay a step graph (256 steps in a row on one set of
buffers and parameters), where something changes between the replays: each
equals the same run of direct launches bit for bit."""
import numpy as np
import pytest

from paper_1801_07986_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

G, C, EPS, DT = 1.0, 40.0, 1e-3, 1e-5


@pytest.fixture
def pn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1801_07986_amd as pkg
    from paper_1801_07986_amd import _binding

    pkg.load()
    yield pkg
    _binding.install_tuned_shapes()


def _dev(N, seed):
    return tuple(torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda:0")
                 for a in inputs.plummer_bh(N, 0.1, seed))


@pytest.mark.parametrize("stage_ns", [0, 2])
def test_launch_shape_changes_between_replays(pn, stage_ns):
    """Chained stages and one-launch stages, whose buffers move within the
    scratch memory with the sweep's split count."""
    runs = []
    for flags in (0, pn.PN_NOGRAPH):
        pn.pn_set_stage_kernel(-1, 0, 0, 0)
        if stage_ns:
            pn.pn_set_stage_kernel(pn.PN_FP64, 2, 1000, stage_ns)
        P, V, M = _dev(300, 51)
        for splits in (16, 4, 16):
            print(f"[case] ns={stage_ns} flags={flags} splits={splits}", flush=True)
            pn.pn_set_shape(-1, 0, 0, 0, 0, 0)
            pn.pn_set_shape(pn.PN_FP64, 2, 1000, 1, 4, splits)
            pn.pn_step(P, V, M, G, C, EPS, DT, 300, pn.PN_FP64, flags=flags)
            torch.cuda.synchronize()
        runs.append((P, V))
    assert torch.equal(runs[0][0], runs[1][0]) and torch.equal(runs[0][1], runs[1][1])
