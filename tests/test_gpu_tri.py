"""The sweeps over unordered pairs (pn_diagnostics, pn_encounters) where their
grid can go wrong: systems smaller than a j-chunk, at the edges of the 256-star
blocks and of the groups of four j, and several blocks of chunks.

Diagnostics against the oracle: energies within 1e-12 of themselves, momenta
within 1e-13 (Newtonian) and 1e-12 (1PN) of the summed magnitude of the stars'
momenta times their own scale (sums of at most 2049^2 terms of 1.1e-16
relative rounding, which add up to 5e-14 at worst for terms of one sign).
Encounters against the full distance matrix: exactly the same indices, also
where many pairs tie (a cubic lattice: the smallest indices win), distances to
the last bits.
"""
import numpy as np
import pytest

import oracle
from paper_1801_07986_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [3, 4, 6, 17, 18, 256, 257, 258, 260, 513, 770, 1025, 2049]


@pytest.fixture(scope="module")
def pn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1801_07986_amd as pkg

    pkg.load()
    return pkg


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda:0")


@pytest.mark.parametrize("N", SIZES)
@pytest.mark.parametrize("eps", [0.0, 1e-2])
def test_diagnostics_edges(pn, N, eps):
    pos, vel, mass = inputs.random_cluster(N - 1, seed=N)
    mass[1:] *= np.random.default_rng(N).uniform(0.5, 2.0, N - 1)
    got = np.array(pn.pn_diagnostics(_dev(pos), _dev(vel), _dev(mass), 1.0, 3.0, eps))
    ref = np.array(oracle.diagnostics(pos, vel, mass, 1.0, 3.0, eps))
    scale = np.abs(mass[:, None] * vel).sum()
    e = np.abs(got - ref)
    print(f"N={N} eps={eps}: E_N {e[0] / abs(ref[0]):.1e} E_1PN {e[1] / abs(ref[1]):.1e} "
          f"P_N {e[2:5].max() / scale:.1e} P_1PN {e[5:].max() / scale:.1e}")
    assert e[0] <= 1e-12 * abs(ref[0]) and e[1] <= 1e-12 * abs(ref[1])
    assert e[2:5].max() <= 1e-13 * scale and e[5:].max() <= 1e-12 * scale


@pytest.mark.parametrize("N", SIZES)
@pytest.mark.parametrize("lattice", [False, True])
def test_encounters_edges(pn, N, lattice):
    pos, vel, mass = inputs.random_cluster(N - 1, seed=100 + N)
    if lattice:  # every distance occurs many times, all exact
        side = int(np.ceil((N - 1) ** (1.0 / 3.0)))
        k = np.arange(N - 1)
        order = np.random.default_rng(N).permutation(N - 1)
        pos[1:] = np.stack([k % side, k // side % side, k // side ** 2], 1)[order]
        pos[0] = [-1.0, -1.0, -1.0]
    r_close = 0.6 if not lattice else 4.0
    got = pn.pn_encounters(_dev(pos), _dev(vel), _dev(mass), 1.0, 3.0, r_close)
    d = pos[1:] - pos[0]
    r = np.sqrt((d * d).sum(1))
    x = pos[1:]
    r2 = ((x[:, None, :] - x[None, :, :]) ** 2).sum(2)
    r2[np.tril_indices(N - 1)] = np.inf  # pairs i < j, in row order: ties to the smallest
    at = int(r2.argmin())
    assert got["pair"] == (at // (N - 1) + 1, at % (N - 1) + 1)
    assert got["nearest_to_bh"] == int(r.argmin()) + 1
    assert got["n_close_bh"] == int((r < r_close).sum())
    assert abs(got["min_r_pair"] - np.sqrt(r2.min())) <= 4e-16 * np.sqrt(r2.min())
    assert abs(got["min_r_bh"] - r.min()) <= 4e-16 * r.min()
