"""The star-star 1PN sums of a Runge-Kutta step, in every form of its sweep:
one-launch stages with 2, 4, 8 and 16 stars per workgroup, where every lane loads
one packet (up to 512 / ns stars) and through LDS (eight wavefronts, 64 packets
each at a time: the tiles end at 512 and 1024 stars), and chained stages with the
split rule.

The light speed is small (c = 2), so that these sums are a good part of the
acceleration, and the velocity change v1 - v0 of one step is compared with the
oracle's, star by star, against the summed magnitudes of the star's own pair
terms, S_i.  Bounds, per unit of dt S_i:
  mixed 6e-6: FP32 pair terms (some twenty roundings of 6e-8 and a reciprocal
    square root of 1.2e-7, cubed: 2e-6) and FP32 partial sums of up to 64 terms
    (64 x 6e-8 = 4e-6);
  FP64 1e-12 (the sweep's accuracy target), and a rounding of the velocity itself.
What is checked must show: for three quarters of the stars the velocity change
from the 1PN sums of pairs (Q, C2 and Q7 of the sweep) is at least 100 times the
mixed bound."""
import numpy as np
import pytest

import oracle
from paper_1801_07986_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

G, C, EPS, DT, M_BH = 1.0, 2.0, 1e-2, 1e-4, 0.1
TOL = {0: 1e-12, 1: 6e-6}


@pytest.fixture
def pn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1801_07986_amd as pkg
    from paper_1801_07986_amd import _binding

    pkg.load()
    yield pkg
    _binding.install_tuned_shapes()


def _pair_terms(pos, vel, mass):
    """Per star: the acceleration lam (Q + C2 v + 7 Q7) and S, in FP64 by torch."""
    lam = 1.0 / C ** 2
    P, V, M = (torch.from_numpy(x).cuda() for x in (pos, vel, mass))
    d0 = P[1:] - P[0]
    R0 = (d0 * d0).sum(1).add(EPS ** 2).sqrt()
    u = G * M[0] / R0
    b = (u / R0 ** 2)[:, None] * d0
    x, v, gm = P[1:], V[1:], G * M[1:]
    v2, bn = (v * v).sum(1), b.norm(dim=1)
    part, scale = torch.empty_like(x), torch.empty_like(gm)
    for i0 in range(0, len(gm), 256):
        i = slice(i0, i0 + 256)
        dx = x[i, None, :] - x[None, :, :]
        R = (dx * dx).sum(2).add(EPS ** 2).sqrt()
        w = gm[None, :] / R
        k = torch.arange(i0, min(i0 + 256, len(gm)), device="cuda")
        w[k - i0, k] = 0.0
        n = dx / R[:, :, None]
        nv = (n * v[None]).sum(2)
        vv = (v[i, None, :] * v[None]).sum(2)
        s = (-2.0 * v2 + u)[None] + 4.0 * vv + 1.5 * nv ** 2 - 0.5 * (dx * b[None]).sum(2)
        dd = (n * (4.0 * v[i, None, :] - 3.0 * v[None])).sum(2)
        w2 = w / R
        q = (w2[:, :, None] * (s[:, :, None] * n - dd[:, :, None] * v[None])).sum(1)
        c2, q7 = (w2 * dd).sum(1), (w[:, :, None] * (-0.5 * b[None])).sum(1)
        part[i] = lam * (q + c2[:, None] * v[i] + 7.0 * q7)
        vi, vj = v2[i].sqrt()[:, None], v2.sqrt()[None]
        mag = 2.0 * v2[None] + u[None] + 4.0 * vi * vj + 1.5 * v2[None] + 0.5 * R * bn[None]
        mag = mag + (4.0 * vi + 3.0 * vj) * (vi + vj) + (v2[i] + 4.0 * u[i])[:, None]
        scale[i] = (w2 * (1.0 + lam * mag) + lam * 3.5 * w * bn[None]).sum(1)
    return part.cpu().numpy(), scale.cpu().numpy()


_reference = {}


def _check(pn, N, prec):
    if N not in _reference:
        if len(_reference) > 8:
            _reference.clear()
        pos, vel, mass = inputs.plummer_bh(N, M_BH, 900 + N)
        _reference[N] = (pos, vel, mass, oracle.step(pos, vel, mass, G, C, EPS, DT, 1)[1],
                         *_pair_terms(pos, vel, mass))
    pos, vel, mass, rv, part, scale = _reference[N]
    size = np.linalg.norm(part, axis=1)
    assert np.mean(size >= 100 * TOL[1] * scale) >= 0.75
    P, V, M = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (pos, vel, mass))
    pn.pn_step(P, V, M, G, C, EPS, DT, 1, prec)
    err = np.linalg.norm(V.cpu().numpy() - rv, axis=1)[1:]
    bound = TOL[prec] * DT * scale + 4e-16 * np.abs(vel).max()
    print(f"N={N} prec={prec}: error / bound {(err / bound).max():.2e}, "
          f"1PN sums / scale {np.median(size / scale):.2e}", flush=True)
    assert (err <= bound).all()


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "mixed"])
@pytest.mark.parametrize("ns", [2, 4, 8, 16])
def test_one_launch_stages(pn, ns, prec):
    pn.pn_set_stage_kernel(-1, 0, 0, 0)
    pn.pn_set_stage_kernel(prec, 2, 1 << 28, ns)
    for stars in sorted({512 // ns - 1, 512 // ns, 512 // ns + 1, 511, 512, 513, 1024, 1025}):
        print(f"[case] ns={ns} stars={stars}", flush=True)
        _check(pn, stars + 1, prec)


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "mixed"])
@pytest.mark.parametrize("N,ipt", [(129, 1), (600, 1), (2306, 1), (2306, 2), (4097, 1)])
def test_chained_stages(pn, N, ipt, prec):
    pn.pn_set_stage_kernel(-1, 0, 0, 0)
    pn.pn_set_shape(-1, 0, 0, 0, 0, 0)
    pn.pn_set_shape(prec, 2, 1 << 28, ipt, 8, 0)
    print(f"[case] N={N} ipt={ipt}", flush=True)
    _check(pn, N, prec)
