"""GPU parity of the tile pair kernel (FP64 real space and the short-range
repulsion) where it can go wrong: tile and chunk remainders, every number of
waves per tile, copies across both periodic boundaries, cutoffs of half a
period, many image families, tiles much longer than the cutoff.

The kernel's own error is its erfcx fit, below 2e-11 of each pair term; with
pair terms that cancel to a tenth of their magnitude the relative RMS stays
below 2e-10, and the bound is the FP64 path's 1e-9.  The WCA terms have no fit:
1e-12."""
import numpy as np
import pytest

from paper_2405_06333_amd import inputs
from tests.gpu_common import gpu_slab, oracle_slab, rel_rms, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


@pytest.fixture(scope="module")
def R():
    from paper_2405_06333_amd import rbe2d
    rbe2d.lib()
    return rbe2d


def wl(seed, N, Lx, Ly, H, rc, alpha=1.0, gt=0.7, gb=-0.6, M=4):
    return inputs.Workload(f"tile{seed}", N, Lx, Ly, H, gt, gb, alpha, rc, 8, M, seed=seed, margin=0.05 * H)


CASES = [
    # tile remainders in one box
    wl(1, 1, 12, 12, 5, 4), wl(2, 2, 12, 12, 5, 4), wl(3, 63, 12, 12, 5, 4), wl(4, 64, 12, 12, 5, 4),
    wl(5, 65, 12, 12, 5, 4), wl(6, 128, 12, 12, 5, 4), wl(7, 129, 12, 12, 5, 4),
    # chunk remainders and several batches of runs: many families in a thin slab
    wl(8, 700, 14, 14, 0.9, 3.5, gt=1.0, gb=-1.0, M=10),
    # taller than wide; a tile spans many layers' worth of cells
    wl(9, 900, 8.4, 8.4, 30, 4),
    # long boxes: copies across one boundary at nearly, and exactly, half a period
    wl(10, 1500, 60, 8.1, 6, 4), wl(11, 1500, 8.1, 60, 6, 4), wl(12, 800, 9, 9, 6, 4.5), wl(13, 800, 9, 40, 6, 4.5),
    # sparse: tiles much longer than the cutoff, empty columns
    wl(14, 90, 150, 150, 10, 4), wl(15, 300, 400, 30, 3, 4),
    # no images
    wl(16, 1000, 20, 17, 12, 4, gt=0.0, gb=0.0, M=0),
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_real_space_and_derivatives(torch, R, orc, w):
    pos, q = inputs.sample(w)
    q = q * np.linspace(0.5, 1.5, w.N)          # every charge its own
    slab = gpu_slab(R, w, "fp64")
    kset = slab.draw_kset(w.seed)
    slab.set_kset(kset)
    P, Q = to_dev(torch, pos), to_dev(torch, q)
    F, E = slab.forces(P, Q, flags=R.REAL, want_energy=True)
    o = oracle_slab(orc, w, slab.Lz_ext)
    ref = orc.evaluate(o, pos, q, kset, parts=("real",))
    assert rel_rms(F.cpu().numpy(), ref.F) <= 1e-9
    assert abs(float(E[1]) - ref.E_real) <= 1e-9 * (np.abs(q * ref.phi).sum() + 1e-300)
    # the variant with the gamma derivatives
    slab.energy(P, Q)
    one = torch.ones((), dtype=torch.float64, device="cuda")
    dr, dq, dg = slab.energy_backward(P, Q, one)
    full = orc.evaluate(o, pos, q, kset)
    assert rel_rms(-dr.cpu().numpy(), full.F) <= 1e-9
    assert rel_rms(dq.cpu().numpy(), full.phi) <= 1e-9
    scale = abs(full.E_real) + abs(full.E_k) + abs(full.E_self) + abs(full.E_ibc)
    assert np.abs(dg.cpu().numpy() - orc.dE_dgamma(o, pos, q, kset)).max() <= 1e-9 * max(1.0, 10.0 * scale)
    slab.check()


@pytest.mark.parametrize("N", [700, 9000, 24576, 24577, 40000, 70000, 140000])
def test_waves_per_tile(torch, R, orc, N):
    """16, 5, 2 and 1 blocks of 4 waves, 2 waves and 1 wave share a tile as the
    system grows."""
    L = float(np.sqrt(N / 1.5))
    w = wl(20, N, L, L, 6.0, 3.0, M=2)
    pos, q = inputs.sample(w)
    slab = gpu_slab(R, w, "fp64")
    kset = slab.draw_kset(w.seed)
    slab.set_kset(kset)
    P, Q = to_dev(torch, pos), to_dev(torch, q)
    F = slab.forces(P, Q, flags=R.REAL)
    t = np.random.default_rng(0).choice(N, 96, replace=False)
    ref = orc.evaluate(oracle_slab(orc, w, slab.Lz_ext), pos, q, kset, targets=t, parts=("real",))
    assert rel_rms(F.cpu().numpy()[t], ref.F) <= 1e-9
    # the tuned split (a summation order) gives the same forces
    slab.autotune(P, Q)
    assert rel_rms(slab.forces(P, Q, flags=R.REAL).cpu().numpy(), F.cpu().numpy()) <= 1e-12


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("w", [wl(30, 65, 5, 5, 4, 2), wl(31, 1500, 30, 5, 6, 2.5), wl(32, 2000, 4.5, 40, 9, 2.2),
                               wl(33, 9000, 40, 30, 8, 3)], ids=lambda w: w.name)
def test_short_range(torch, R, orc, w, precision):
    pos, q = inputs.sample(w)
    slab = gpu_slab(R, w, precision)
    md = R.md_params(sigma=1.0, eps=0.9, sigma_wall=0.6, eps_wall=0.7, wall_margin=0.01)
    F, E = slab.short_forces(to_dev(torch, pos), to_dev(torch, q), md, want_energy=True)
    ref, ep, ew = orc.short_range(pos, w.Lx, w.Ly, w.H, 1.0, 0.9, 0.6, 0.7)
    assert rel_rms(F.cpu().numpy(), ref) <= 1e-12
    assert np.allclose(E.cpu().numpy()[0], [ep, ew], rtol=1e-12, atol=0)


@pytest.mark.parametrize("N", [24576, 24577, 60000])
def test_short_range_by_tiles_or_targets(torch, R, N):
    """FP32 handles: tiles up to 24576 ions, one thread per ion beyond; the same
    FP64 terms as an FP64 handle's tiles.  They shift an image before or after
    the difference is taken, 3e-14 apart in a box of 270; that is 14 times as
    much relative to the force at r = 0.01: 4e-11, bound 1e-10."""
    L = float(np.sqrt(N / 1.5))
    w = wl(21, N, L, 1.1 * L, 6.0, 3.0, M=2)
    pos, q = inputs.sample(w)
    P, Q = to_dev(torch, pos), to_dev(torch, q)
    mp = R.md_params(sigma=0.6, eps=1.0, sigma_wall=0.5, eps_wall=1.0)
    out = []
    for precision in ("fp32", "fp64"):
        F = torch.full((N, 3), 0.25, dtype=torch.float64, device="cuda")
        _, E = gpu_slab(R, w, precision).short_forces(P, Q, mp, F=F, want_energy=True)
        out.append((F.cpu().numpy() - 0.25, E.cpu().numpy()))
    assert rel_rms(out[0][0], out[1][0]) <= 1e-10
    assert rel_rms(out[0][1], out[1][1]) <= 1e-10


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("Ly, H", [(6e5, 4.0), (1.0, 2.0e5)], ids=["long", "tall"])
def test_boxes_far_longer_than_wide(torch, R, orc, precision, Ly, H):
    """The margin of the cell search grows with the box; in these it alone
    reaches past the copies in x.  Ions in one corner, so that they interact."""
    w = wl(40, 200, 1.0, Ly, H, 0.5, alpha=0.1, M=0)    # (FP32 handles refuse a wider k-range)
    rng = np.random.default_rng(w.seed)
    pos = rng.uniform([0.0, 0.0, 0.2], [1.0, min(Ly, 12.0), 3.8 if H < 10 else 14.2], (w.N, 3))
    q = np.where(np.arange(w.N) % 2 == 0, 1.0, -1.0)
    kset = np.tile(np.array([[1, 0, 0]], dtype=np.int32), (w.P, 1))
    slab = gpu_slab(R, w, precision)
    slab.set_kset(kset)
    P, Q = to_dev(torch, pos), to_dev(torch, q)
    if precision == "fp64":     # (FP32 handles: the short-range tiles alone)
        F = slab.forces(P, Q, flags=R.REAL)
        ref = orc.evaluate(oracle_slab(orc, w, slab.Lz_ext), pos, q, kset, parts=("real",))
        assert rel_rms(F.cpu().numpy(), ref.F) <= 1e-9
    F, E = slab.short_forces(P, Q, R.md_params(sigma=0.4, eps=0.9, sigma_wall=0.2, eps_wall=0.7, wall_margin=0.01),
                             want_energy=True)
    ref, ep, ew = orc.short_range(pos, w.Lx, w.Ly, w.H, 0.4, 0.9, 0.2, 0.7)
    assert rel_rms(F.cpu().numpy(), ref) <= 1e-10     # (y / Ly and back: 1e-16 of the position)
    assert np.allclose(E.cpu().numpy()[0], [ep, ew], rtol=1e-10, atol=0)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N", [60, 700, 9000])
def test_ions_without_a_place_leave_the_others_alone(torch, R, precision, N):
    """An ion whose position is not finite has no neighbours; every other ion
    has what it has without it (summation order aside).  REAL alone and the
    short-range forces: with k-space the charges of all ions meet."""
    L = max(9.0, float(np.sqrt(N / 1.5)))
    w = wl(41, N, L, L, 6.0, 3.0, M=2)
    pos, q = inputs.sample(w)
    rng = np.random.default_rng(w.seed)
    lost = np.sort(rng.choice(N, max(1, N // 50), replace=False))
    kept = np.setdiff1d(np.arange(N), lost)
    bad = pos.copy()
    for k, i in enumerate(lost):
        bad[i, k % 3] = (np.nan, np.inf, -np.inf)[(k // 3) % 3]
    mp = R.md_params(sigma=0.6, eps=1.0, sigma_wall=0.5, eps_wall=1.0)
    slab = gpu_slab(R, w, precision)
    slab.set_kset(slab.draw_kset(w.seed))
    calls = [lambda p, c: slab.short_forces(p, c, mp)]
    if precision == "fp64":
        calls.append(lambda p, c: slab.forces(p, c, flags=R.REAL))
    for f in calls:
        F = f(to_dev(torch, bad), to_dev(torch, q)).cpu().numpy()[kept]
        ref = f(to_dev(torch, pos[kept]), to_dev(torch, q[kept])).cpu().numpy()
        assert np.isfinite(F).all()
        assert rel_rms(F, ref) <= 1e-12
