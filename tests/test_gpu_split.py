"""GPU parity of the FP32 pair kernel's split form (few targets: x-columns and
image families in separate blocks) at the edges of its range: several image
families per layer of blocks, none, coincident and very close ions, and both
sides of the largest target count that splits the families.

Bound: the FP32 path's 1e-5 (its pair terms carry 7e-7)."""
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


def wl(seed, N, Lx, Ly, H, rc, gt=0.8, gb=-0.7, M=4):
    return inputs.Workload(f"split{seed}", N, Lx, Ly, H, gt, gb, 1.0, rc, 8, M, seed=seed, margin=0.05 * H,
                           precision="fp32")


@pytest.mark.parametrize("w", [
    wl(1, 65, 12, 12, 5, 4), wl(2, 700, 14, 14, 0.9, 3.5, gt=1.0, gb=-1.0, M=10), wl(3, 700, 14, 11, 2.0, 3.5, M=3),
    wl(4, 900, 20, 20, 6, 4, gt=0.0, gb=0.0, M=0), wl(5, 16384, 90, 90, 6, 3, M=2), wl(6, 16385, 90, 80, 6, 3, M=2),
    wl(8, 49152, 150, 150, 6, 3, M=2), wl(9, 49153, 150, 140, 6, 3, M=2),
], ids=lambda w: w.name)
def test_families_and_columns(torch, R, orc, w):
    pos, q = inputs.sample(w)
    pos[1] = pos[0] + [0.0, 0.0, 1e-4]              # a close pair: exact FP64 displacement
    slab = gpu_slab(R, w, "fp32")
    kset = slab.draw_kset(w.seed)
    slab.set_kset(kset)
    F, E = slab.forces(to_dev(torch, pos), to_dev(torch, q), flags=R.REAL, want_energy=True)
    t = np.arange(w.N) if w.N < 2000 else np.random.default_rng(0).choice(np.arange(2, w.N), 96, replace=False)
    # (the oracle gives energies for all targets only)
    ref = orc.evaluate(oracle_slab(orc, w, slab.Lz_ext), pos, q, kset, targets=None if w.N < 2000 else t,
                       parts=("real",))
    F = F.cpu().numpy()
    # the close pair's force would hide the others: apart from them
    far = t >= 2
    assert rel_rms(F[t][far], ref.F[far]) <= 1e-5
    if w.N < 2000:
        assert rel_rms(F[:2], ref.F[:2]) <= 1e-5
        assert abs(float(E[1]) - ref.E_real) <= 1e-5 * np.abs(q * ref.phi).sum()
    slab.check()


def test_coincident_ions(torch, R):
    """Two ions at one place do not interact (their force would be undefined)."""
    w = wl(7, 200, 12, 12, 5, 4, M=0)
    pos, q = inputs.sample(w)
    slab = gpu_slab(R, w, "fp32")
    slab.set_kset(slab.draw_kset(w.seed))
    pos[1] = pos[0]
    F = slab.forces(to_dev(torch, pos), to_dev(torch, q), flags=R.REAL).cpu().numpy()
    one = np.delete(np.arange(w.N), 1)
    alone = slab.forces(to_dev(torch, pos[one]), to_dev(torch, q[one]), flags=R.REAL).cpu().numpy()
    assert np.isfinite(F).all()
    assert np.allclose(F[0], alone[0], rtol=1e-5, atol=1e-5 * np.abs(alone).max())
