"""Monte Carlo generator (heatbath, over-relaxation, multi-hit) on the GPU against the FP64 oracle.

Small lattices: the links after whole sweeps and the multi-hit averages element by element against
the oracle driven by the same Philox counters (1e-12 at beta 5.8-6.2: ulp-level differences of
log/cos/sqrt between the two sides do not grow, and a changed accept/reject decision would show as an
O(1) difference; 1e-8 at strong coupling, see the case), and the rejected-pair counts exactly. Full sizes: over-relaxation keeps the plaquette; links stay in
SU(3); the strong- and weak-coupling plaquettes pinned in the oracle tests.
"""
import numpy as np
import pytest

from oracle import mc, observables, su3
from paper_1208_1186_amd import gf, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gf.load()


def _unit(dims):
    shp = synth.lattice_shape(dims)
    return np.broadcast_to(np.eye(3, dtype=np.complex128), shp + (4, 3, 3)).copy()


@pytest.mark.parametrize("dims,start,beta,n_or,sweeps,tol", [
    ((4, 4, 4, 4), "cold", 6.0, 2, 3, 1e-12),
    ((6, 4, 4, 8), "synth", 5.8, 1, 3, 1e-12),
    ((8, 8, 8, 8), "synth", 6.2, 0, 3, 1e-12),
    # strong coupling: alpha < 1 often puts x0 near -1, where the direction's scale sqrt(1 - x0^2)
    # turns an ulp of difference in delta (log and cos on the two sides) into ulp / sqrt(1 - x0^2),
    # and the next sweep amplifies that again through the staples, so one sweep is compared; a
    # changed accept/reject decision would still show as an O(1) difference (and in the counts)
    ((4, 6, 2, 4), "synth", 0.4, 1, 1, 1e-8),
])
def test_sweeps_match_oracle(dims, start, beta, n_or, sweeps, tol):
    print(f"mc sweeps {dims} {start} beta {beta} n_or {n_or}", flush=True)
    u = _unit(dims) if start == "cold" else synth.make_config(dims, 3)
    seed = 0x1234_5678_9ABC_DEF0
    links = torch.from_numpy(u).cuda()
    m = gf.MonteCarlo(dims, beta, seed)
    want = u
    for sweep in range(sweeps):
        rej = m.update(links, sweep, n_or, count_rejected=True)
        want, wrej = mc.update(want, beta, seed, sweep, n_or)
        assert rej == wrej
        got = links.cpu().numpy()
        assert np.max(np.abs(got - want)) < tol, sweep
    assert abs(m.plaquette(links) - observables.plaquette(want)) < max(1e-13, tol)
    m.close()


@pytest.mark.parametrize("dims,beta,n_hits", [((4, 4, 4, 4), 6.0, 5), ((6, 4, 4, 8), 2.0, 3)])
def test_multihit_matches_oracle(dims, beta, n_hits):
    u = synth.make_config(dims, 4)
    links = torch.from_numpy(u).cuda()
    m = gf.MonteCarlo(dims, beta, 77)
    got = m.multihit(links, 9, n_hits).cpu().numpy()
    want = mc.multihit(u, beta, 77, 9, n_hits)
    assert np.max(np.abs(got - want)) < 1e-12
    assert torch.equal(links, torch.from_numpy(u).cuda())  # input untouched
    m.close()


@pytest.mark.parametrize("dims,n_or,n_hits", [
    ((2, 2, 2, 2), 1, 1),    # 8 sites of a parity in a tile of 64; neighbours up and down are the same site
    ((6, 10, 2, 4), 2, 2),   # 240: the last tile and the last 64-site run are part full
    ((32, 8, 8, 2), 1, 1),   # whole tiles, planes visited with z in groups; one hit (its own launch)
    ((16, 8, 8, 2), 1, 12),  # z in groups for the multi-hit only
])
def test_tiles_and_orders_match_oracle(dims, n_or, n_hits):
    """Where the even/odd tiles, the runs of 64 sites and the plane orders have their edges; the bound of the
    tests above (ulp-level differences of log, cos and sqrt)."""
    u = synth.make_config(dims, 13)
    links = torch.from_numpy(u).cuda()
    m = gf.MonteCarlo(dims, 6.0, 1 << 40)
    rej = m.update(links, 3, n_or, count_rejected=True)
    want, wrej = mc.update(u, 6.0, 1 << 40, 3, n_or)
    assert rej == wrej and np.max(np.abs(links.cpu().numpy() - want)) < 1e-12
    got = m.multihit(links, 7, n_hits).cpu().numpy()
    assert np.max(np.abs(got - mc.multihit(links.cpu().numpy(), 6.0, 1 << 40, 7, n_hits))) < 1e-12
    m.close()


@pytest.mark.parametrize("dims,n_hits", [
    ((32, 16, 8, 2), 1),     # planes of 8 blocks of 64 sites: one to an XCD; z in groups
    ((32, 16, 2, 2), 2),     # without the groups
    ((32, 32, 4, 2), 3),     # two blocks of a plane to an XCD, without the groups
    ((32, 32, 8, 2), 1),     # and with them
    ((48, 32, 8, 4), 2),     # three
    ((32, 32, 16, 10), 1),   # beyond 131072 sites one and two hits reserve LDS
    ((32, 32, 16, 10), 2),
])
def test_multihit_bands_match_oracle(dims, n_hits):
    """Planes of a multiple of eight blocks, whose bands of rows go to the XCDs: every site is written (the output is
    NaN before) and has its own average; the bound of the tests above."""
    print(f"multi-hit bands {dims} hits {n_hits}", flush=True)
    u = synth.make_config((8, 8, 8, 8), 14).reshape(-1, 4, 3, 3)
    u = u[np.random.default_rng(15).integers(0, len(u), int(np.prod(dims)))].reshape(synth.lattice_shape(dims) + (4, 3, 3))
    m = gf.MonteCarlo(dims, 6.0, 78)
    out = torch.full(synth.lattice_shape(dims) + (3, 3), complex("nan"), dtype=torch.complex128, device="cuda:0")
    m.multihit(torch.from_numpy(u).cuda(), 5, n_hits, out)
    got = out.cpu().numpy()
    assert np.max(np.abs(got - mc.multihit(u, 6.0, 78, 5, n_hits))) < 1e-12
    m.close()


def test_overrelaxation_and_unitarity_at_32x32x32x32():
    dims = (32, 32, 32, 32)
    links = torch.from_numpy(synth.make_config(dims, 0)).cuda()
    m = gf.MonteCarlo(dims, 6.0, 5)
    m.update(links, 0, 0)
    p0 = m.plaquette(links)
    # an over-relaxation-only pass is not exposed; a heatbath sweep with its own random numbers moves
    # the plaquette, so compare two updates that differ only by over-relaxation sweeps at the end:
    a = links.clone()
    m.update(a, 1, 0)
    b = links.clone()
    m.update(b, 1, 3)
    pa, pb = m.plaquette(a), m.plaquette(b)
    assert abs(pa - pb) < 1e-12, (pa, pb)
    assert p0 != pa
    for t in (a, b):
        sample = t[::7, ::5, ::3, ::2].cpu().numpy()
        assert su3.unitarity_error(sample) < 1e-14 and su3.det_error(sample) < 1e-14
    m.close()


@pytest.mark.parametrize("beta,want,tol", [
    (0.3, 0.3 / 18 + 0.09 / 216, 1.5e-3),   # strong coupling
    (60.0, 1 - 2 / 60.0, 1e-3),             # one-gluon exchange
])
def test_plaquette_limits_at_16x16x16x16(beta, want, tol):
    dims = (16, 16, 16, 16)
    links = torch.from_numpy(_unit(dims)).cuda()
    m = gf.MonteCarlo(dims, beta, 31)
    ps = []
    for sweep in range(60):
        m.update(links, sweep, 1)
        if sweep >= 20:
            ps.append(m.plaquette(links))
    assert abs(np.mean(ps) - want) < tol, np.mean(ps)
    m.close()


def test_several_sweeps_in_one_call_are_bitwise_single_calls():
    dims = (8, 4, 6, 4)
    u = synth.make_config(dims, 8)
    a = torch.from_numpy(u).cuda()
    b = torch.from_numpy(u).cuda()
    m = gf.MonteCarlo(dims, 6.0, 99)
    ra = m.update(a, 5, 2, count_rejected=True, n_sweeps=3)
    rb = sum(m.update(b, 5 + k, 2, count_rejected=True) for k in range(3))
    assert torch.equal(a, b) and ra == rb
    with pytest.raises(gf.GfError):
        m.update(a, 0xFFFFFFFF, 0, n_sweeps=2)  # the last sweep index would not fit in 32 bits
    m.close()
