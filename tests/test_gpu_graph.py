"""Step graphs: captured once 256 steps in a row were asked for on one set of
buffers, replayed 16 steps at a time (ensembles: one), the rest launched
directly.  Runs that replay the graph many times, with other GPU work and
synchronisations between the calls, equal direct launches bit for bit; so does
a run on other buffers in between, which leaves the cached graph alone."""
import numpy as np
import pytest

from paper_1801_07986_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

G, C, EPS, DT = 1.0, 40.0, 1e-3, 1e-5


@pytest.fixture(scope="module")
def pn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1801_07986_amd as pkg

    pkg.load()
    return pkg


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda:0")


def _advance(pn, kind, prec, P, V, M, n, flags=0):
    if kind == "hermite":
        pn.pn_step_hermite(P, V, M, G, C, EPS, DT, n, flags=flags)
    elif kind == "ensemble":
        N = M.shape[0]
        pn.pn_step_batched([0, N // 3, N], [G] * 2, [C] * 2, [EPS] * 2, P, V, M, DT, n, prec,
                           flags=flags)
    else:
        pn.pn_step(P, V, M, G, C, EPS, DT, n, prec, flags=flags)


# one-launch stages (N = 100), chained stages, the Hermite steps, an ensemble
CASES = [("step", 100, 0), ("step", 100, 1), ("step", 2200, 0), ("step", 2200, 1),
         ("hermite", 150, 0), ("ensemble", 300, 0), ("ensemble", 300, 1)]


@pytest.mark.parametrize("kind,N,prec", CASES)
def test_replayed_runs_equal_direct_launches(pn, kind, N, prec):
    pos, vel, mass = inputs.plummer_bh(N, 0.1, 40 + N)
    M = _dev(mass)
    runs = []
    # 300 steps: one call (captures, replays at once), 100 + 150 + 50 (captured
    # in the third call; a Hermite call starts afresh, so it is compared with
    # direct launches in the same parts), other buffers in between
    for parts, flags, other in (((300,), 0, False), ((300,), pn.PN_NOGRAPH, False),
                                ((100, 150, 50), 0, True), ((100, 150, 50), pn.PN_NOGRAPH, False),
                                ((300, 40), 0, False), ((300, 40), pn.PN_NOGRAPH, False)):
        P, V = _dev(pos), _dev(vel)
        for n in parts:
            _advance(pn, kind, prec, P, V, M, n, flags)
            assert float((P * P).sum()) > 0.0  # eager work and a synchronisation
            if other:
                P2, V2 = _dev(pos), _dev(vel)
                _advance(pn, kind, prec, P2, V2, M, 3, flags)
        runs.append((P.cpu().numpy(), V.cpu().numpy()))
    for a, b in ((0, 1), (2, 3), (4, 5)):
        assert np.array_equal(runs[a][0], runs[b][0]) and np.array_equal(runs[a][1], runs[b][1])
    if kind != "hermite":
        assert np.array_equal(runs[0][0], runs[2][0]) and np.array_equal(runs[0][1], runs[2][1])


def test_calls_in_a_row_replay_the_graph(pn):
    """Ten calls of 40 steps on one set of buffers (the graph is captured in the
    seventh and replayed from then on) equal one direct run of 400."""
    pos, vel, mass = inputs.plummer_bh(200, 0.1, 9)
    M = _dev(mass)
    P, V = _dev(pos), _dev(vel)
    for _ in range(10):
        _advance(pn, "step", 0, P, V, M, 40)
        torch.cuda.synchronize()
    D, W = _dev(pos), _dev(vel)
    _advance(pn, "step", 0, D, W, M, 400, pn.PN_NOGRAPH)
    assert torch.equal(P, D) and torch.equal(V, W)
