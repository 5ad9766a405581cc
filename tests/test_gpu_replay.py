"""Runs long enough to replay a step graph (256 steps in a row on one set of
buffers and parameters), where something changes between the replays: each
equals the same run of direct launches bit for bit.  (Shorter runs are launched
directly whatever their flags, so comparisons of 2 to 60 steps with and without
PN_NOGRAPH elsewhere in the tests compare direct launches with each other.)"""
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


def _advance(pn, kind, prec, S, n, flags=0, stream=None):
    P, V, M = S
    if kind == "hermite":
        pn.pn_step_hermite(P, V, M, G, C, EPS, DT, n, stream=stream, flags=flags)
    elif kind == "ensemble":
        N = M.shape[0]
        pn.pn_step_batched([0, N // 3, N], [G, 2 * G], [C, C / 2], [EPS] * 2, P, V, M, DT, n, prec,
                           stream=stream, flags=flags)
    else:
        pn.pn_step(P, V, M, G, C, EPS, DT, n, prec, stream=stream, flags=flags)


# one-launch stages, chained stages, the Hermite steps, an ensemble
KINDS = [("step", 100, 0), ("step", 100, 1), ("step", 2200, 0), ("step", 2200, 1),
         ("hermite", 150, 0), ("ensemble", 300, 0), ("ensemble", 300, 1)]


def _equal(a, b):
    return torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("kind,N,prec", KINDS)
@pytest.mark.parametrize("first", [255, 256, 257])
def test_threshold(pn, kind, N, prec, first):
    runs = []
    for flags in (0, pn.PN_NOGRAPH):
        S = _dev(N, 60)
        for n in (first, 17, 15, 33):
            _advance(pn, kind, prec, S, n, flags)
            torch.cuda.synchronize()
        runs.append(S)
    assert _equal(*runs)


@pytest.mark.parametrize("kind,N,prec", KINDS)
def test_another_system_between_replays(pn, kind, N, prec):
    """The graph stays cached while another system (of another size, so for an
    ensemble other descriptors in the same memory) takes a few steps, and is
    replayed again after each."""
    runs = []
    for flags in (0, pn.PN_NOGRAPH):
        S, T = _dev(N, 61), _dev(N - 7, 62)
        _advance(pn, kind, prec, S, 300, flags)
        for n in (3, 20, 1):
            _advance(pn, kind, prec, T, n, flags)
            _advance(pn, kind, prec, S, 50, flags)
            torch.cuda.synchronize()
        runs.append(S + T)
    assert _equal(runs[0], runs[1]) and _equal(runs[0][3:], runs[1][3:])


@pytest.mark.parametrize("kind,N,prec", KINDS)
def test_scratch_grows_between_replays(pn, kind, N, prec):
    runs = []
    for flags in (0, pn.PN_NOGRAPH):
        pn.pn_release()  # (small scratch memory again)
        S = _dev(N, 63)
        _advance(pn, kind, prec, S, 300, flags)
        _advance(pn, kind, prec, _dev(20000, 64), 1, flags)
        _advance(pn, kind, prec, S, 300, flags)
        torch.cuda.synchronize()
        runs.append(S)
    assert _equal(*runs)


def test_schemes_alternate(pn):
    """Runge-Kutta, Hermite and Runge-Kutta runs on one state, each long enough to
    capture its own graph."""
    runs = []
    for flags in (0, pn.PN_NOGRAPH):
        S = _dev(200, 65)
        for kind in ("step", "hermite", "step", "hermite"):
            _advance(pn, kind, 0, S, 300, flags)
            torch.cuda.synchronize()
        runs.append(S)
    assert _equal(*runs)


@pytest.mark.parametrize("kind,N,prec", KINDS)
def test_two_streams(pn, kind, N, prec):
    """Two systems in turn on two streams, asynchronously, each call long enough
    to capture and replay (one graph is cached, so each call captures anew while
    the other stream's replays may still run)."""
    alone = []
    for seed in (66, 67):
        S = _dev(N, seed)
        for n in (260, 300, 280):
            _advance(pn, kind, prec, S, n, pn.PN_NOGRAPH)
        alone.append(S)
    a, b = _dev(N, 66), _dev(N, 67)
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for n in (260, 300, 280):
        _advance(pn, kind, prec, a, n, pn.PN_ASYNC, sa)
        _advance(pn, kind, prec, b, n, pn.PN_ASYNC, sb)
    torch.cuda.synchronize()
    assert _equal(a, alone[0]) and _equal(b, alone[1])


@pytest.mark.parametrize("kind,N,prec", KINDS)
def test_caller_captures_steps(pn, kind, N, prec):
    """Asynchronous steps on a stream that the caller captures go into the caller's
    graph, also when the library has a graph of its own for them: three replays,
    with eager work and a synchronisation after each, equal three direct calls."""
    S, D = _dev(N, 68), _dev(N, 68)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    for T, flags in ((D, pn.PN_NOGRAPH), (S, 0)):  # (S last: its graph is cached, and an
        _advance(pn, kind, prec, T, 300, flags, s)  # ensemble's descriptors are in place)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        _advance(pn, kind, prec, S, 40, pn.PN_ASYNC, s)
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert float((S[0] * S[0]).sum()) > 0.0
    assert torch.isfinite(S[0]).all()
    for _ in range(3):
        _advance(pn, kind, prec, D, 40, pn.PN_NOGRAPH, s)
    torch.cuda.synchronize()
    assert _equal(S, D)
