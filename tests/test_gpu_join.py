"""The loop kernel that measures and transforms in (x, y) at once: shapes at the edges of its rule, plane
orders, and its transform buffer across the calls that use the same memory.

Against the FP64 oracle: in double the bounds of the loop test of every shape (links 1e-12, theta 1e-10
relative, F 1e-13). In float a link is a product of three matrices (2 x 3 terms of up to 6 x 6e-8 each) formed
from rows that each update rounds again, so 1e-6 an update and 5e-6 after three; theta and F average such errors.
"""
import numpy as np
import pytest

from oracle import landau
from paper_1208_1186_amd import gf, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gf.load()


@pytest.mark.parametrize("dims,precision", [
    ((8, 8, 24, 8), "fp64_18"), ((8, 8, 12, 12), "fp32_18"),
    ((12, 12, 8, 8), "fp32_12"), ((12, 12, 8, 8), "fp64_12"),      # part waves; in double the two launches
    ((16, 16, 32, 4), "fp64_18"), ((16, 16, 12, 12), "fp64_12"),   # first plane counts of its rule; bricks of 4 x 4
    ((16, 16, 8, 8), "fp32_12"), ((32, 32, 32, 4), "fp64_12"),     # below it: the two launches
    ((32, 32, 16, 16), "fp64_12"), ((32, 32, 48, 8), "fp32_12"),
])
def test_updates_match_oracle(dims, precision):
    print(f"joined loop {dims} {precision}", flush=True)
    n = 3 if np.prod(dims) < 1 << 17 else 1
    u = synth.make_config(dims, 31)
    links = torch.from_numpy(u).cuda()
    fx = gf.GaugeFixer(links, precision, check_every=2)
    fx.iterate(n)
    ref, hist = u, [(landau.theta(u), landau.functional(u))]
    for _ in range(n):
        ref, *_ = landau.fa_step(ref, 0.08)
        hist.append((landau.theta(ref), landau.functional(ref)))
    th, f = fx.history(n + 1)
    fx.close()
    want = np.array(hist)
    dl, dth, df = (5e-6, 1e-4, 1e-5) if precision.startswith("fp32") else (1e-12, 1e-10, 1e-13)
    assert np.max(np.abs(links.cpu().numpy() - ref)) < dl
    assert np.max(np.abs(th - want[:, 0]) / want[:, 0]) < dth
    assert np.max(np.abs(f - want[:, 1])) < df


@pytest.mark.parametrize("dims,precision", [((16, 16, 24, 8), "fp64_18"), ((8, 8, 12, 12), "fp64_12"),
                                            ((12, 12, 16, 16), "fp32_12")])
def test_plane_orders_are_bitwise_equal(dims, precision):
    u = synth.make_config(dims, 32)
    runs = []
    for zb in (1, 2, 4, 8, 0, -1):
        links = torch.from_numpy(u).cuda()
        fx = gf.GaugeFixer(links, precision)
        try:
            fx.set_loop_traversal(zb)
        except gf.GfError:
            continue
        fx.iterate(7)
        runs.append((links, fx.history(8)))
        fx.close()
    assert len(runs) >= 2
    for links, h in runs[1:]:
        assert torch.equal(links, runs[0][0])
        assert np.array_equal(h[0], runs[0][1][0]) and np.array_equal(h[1], runs[0][1][1])


@pytest.mark.parametrize("precision", ["fp64_18", "fp32_12"])
def test_other_uses_of_the_transform_buffer(precision):
    """Stage calls, a saved and restored state and a stop between updates leave the iterates what they are in
    one uninterrupted run."""
    dims = (8, 8, 24, 8)
    u = synth.make_config(dims, 33)
    la = torch.from_numpy(u).cuda()
    a = gf.GaugeFixer(la, precision, check_every=4)
    tol = a.iterate(9).theta * 1.000001  # a stop after 9 updates, one into the third check interval
    l9 = la.clone()
    a.iterate(8)
    lb = torch.from_numpy(u).cuda()
    b = gf.GaugeFixer(lb, precision, check_every=4)
    field = torch.randn(u.shape[:4] + (3, 3), dtype=torch.complex128, device="cuda")
    out = torch.empty_like(field)
    b.iterate(2)
    gf.gf_stage_divergence(b.ctx, out.data_ptr())
    b.iterate(1)
    gf.gf_stage_filter(b.ctx, field.data_ptr(), out.data_ptr())
    b.iterate(1)
    gf.gf_stage_gauge(b.ctx, field.data_ptr(), out.data_ptr())
    state = b.save_state()
    b.iterate(3)
    b.load_state(state)
    r = b.fix_until(tol, 100)
    assert r.iters == 9 and torch.equal(lb, l9)
    b.iterate(8)
    assert torch.equal(lb, la)
    a.close()
    b.close()


@pytest.mark.parametrize("dims,precision", [((8, 8, 24, 8), "fp64_18"), ((16, 16, 16, 16), "fp32_12"),
                                            ((12, 12, 8, 8), "fp64_12")])
def test_divergence_stage_leaves_the_measured_values(dims, precision):
    """Looking at the divergence changes no reported value, not in the last bit, and is the oracle's of those links
    (per entry: the sum of 8 links' roundings, 1e-12 in double, 1e-5 in float)."""
    u = synth.make_config(dims, 34)
    links = torch.from_numpy(u).cuda()
    fx = gf.GaugeFixer(links, precision)
    fx.iterate(2)
    before, hist = fx.quality(), fx.history(3)
    delta = torch.empty(u.shape[:4] + (3, 3), dtype=torch.complex128, device="cuda")
    gf.gf_stage_divergence(fx.ctx, delta.data_ptr())
    torch.cuda.synchronize()
    after = fx.history(3)
    assert fx.quality() == before
    assert np.array_equal(after[0], hist[0]) and np.array_equal(after[1], hist[1])
    want = landau.divergence(links.cpu().numpy())
    assert np.max(np.abs(delta.cpu().numpy() - want)) < (1e-5 if precision.startswith("fp32") else 1e-12)
    fx.close()


@pytest.mark.parametrize("dims,precision,joined", [
    ((8, 8, 12, 12), "fp64_18", True), ((8, 8, 12, 12), "fp32_12", True),      # widest (z, t) rows not compiled
    ((16, 16, 12, 12), "fp64_12", True), ((16, 16, 12, 12), "fp32_18", True),
    ((16, 16, 24, 8), "fp32_12", True), ((16, 16, 32, 4), "fp64_18", True),    # and the first number of planes
    ((16, 16, 8, 8), "fp64_18", False), ((12, 12, 12, 12), "fp64_12", False), ((32, 32, 24, 8), "fp32_12", False),
    ((24, 24, 12, 12), "fp32_12", False),
])
def test_rule_of_the_joined_loop(dims, precision, joined):
    """Which loop a shape takes is its planes' size and number alone; its (z, t) pass is a compiled one. Bounds of
    the first test."""
    u = synth.make_config(dims, 35)
    links = torch.from_numpy(u).cuda()
    fx = gf.GaugeFixer(links, precision)
    gf.gf_set_timing(fx.ctx, 1)
    fx.iterate(2)
    launches = {k: n for k, (_, n) in gf.gf_kernel_times(fx.ctx).items()}
    tiling = fx.fft_tiling()
    fx.set_fft_tiling(*tiling)  # an error for columns that are not compiled
    fx.close()
    assert launches["fft_zt_filter"] == 2 and launches["update_measure"] == 2
    assert launches["fft_xy_fwd"] == (0 if joined else 2)
    ref = u
    for _ in range(2):
        ref, *_ = landau.fa_step(ref, 0.08)
    assert np.max(np.abs(links.cpu().numpy() - ref)) < (5e-6 if precision.startswith("fp32") else 1e-12)


@pytest.mark.parametrize("precision", ["fp64_18", "fp32_12", "mixed"])
def test_restored_run_measures_once(precision):
    """A state keeps the transform its next update starts from: the run that continues it measures nothing again, and
    does where a stage call had used the buffer before the state was saved. Iterates as without the stop."""
    dims = (8, 8, 24, 8)
    u = synth.make_config(dims, 36)
    la = torch.from_numpy(u).cuda()
    a = gf.GaugeFixer(la, precision)
    a.iterate(3)
    saved = a.save_state()
    field = torch.randn(u.shape[:4] + (3, 3), dtype=torch.complex128, device="cuda")
    gf.gf_stage_filter(a.ctx, field.data_ptr(), torch.empty_like(field).data_ptr())
    saved_after_stage = a.save_state()
    a.iterate(4)
    for state, measured in ((saved, 0), (saved_after_stage, 1)):
        lb = torch.from_numpy(u).cuda()
        b = gf.GaugeFixer(lb, precision)
        b.load_state(state)
        gf.gf_set_timing(b.ctx, 1)
        b.iterate(4)
        assert gf.gf_kernel_times(b.ctx)["divergence"][1] == measured
        assert torch.equal(lb, la) and b.quality() == a.quality()
        assert all(np.array_equal(x, y) for x, y in zip(b.history(8), a.history(8)))
        b.close()
    a.close()


def test_state_without_the_mark_measures_again():
    """A state whose header does not carry the mark (bytes of some other value in its place) is restored all the same:
    the run measures its links before it goes on."""
    dims = (8, 8, 24, 8)
    u = synth.make_config(dims, 37)
    la = torch.from_numpy(u).cuda()
    a = gf.GaugeFixer(la, "fp64_18")
    a.iterate(3)
    n = gf.gf_state_bytes(a.ctx)
    saved, unmarked = (torch.zeros(n, dtype=torch.uint8, device="cuda") for _ in range(2))
    gf.gf_get_state(a.ctx, saved.data_ptr(), n)
    field = torch.randn(u.shape[:4] + (3, 3), dtype=torch.complex128, device="cuda")
    gf.gf_stage_filter(a.ctx, field.data_ptr(), torch.empty_like(field).data_ptr())
    gf.gf_get_state(a.ctx, unmarked.data_ptr(), n)
    differ = (saved[:256] != unmarked[:256]).nonzero().flatten()
    assert 0 < len(differ) <= 4  # one word
    unmarked[differ] = 1
    a.iterate(4)
    lb = torch.from_numpy(u).cuda()
    b = gf.GaugeFixer(lb, "fp64_18")
    b.load_state(unmarked)
    b.iterate(4)
    assert torch.equal(lb, la)
    a.close()
    b.close()
