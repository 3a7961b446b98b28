"""GPU parity of whole calls at the sizes where their launches change: one or
two streams, the cell list in one launch or four, the force pass split over
the waves of a block or not (with the energies in its launch or in one of
their own).

Bounds: the FP64 path's 1e-9 and the FP32 path's 1e-5."""
import numpy as np
import pytest

from paper_2405_06333_amd import inputs
from tests.gpu_common import energy_scale, gpu_slab, oracle_slab, rel_rms, to_dev

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-9, "fp32": 1e-5}


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


def wl(N, P, M=3):
    L = max(10.0, (N / 1.2) ** 0.5)
    return inputs.Workload(f"n{N}_p{P}", N, L, L * 1.1, 6.0, 0.8, -0.7, 1.0, 4.0, P, M, seed=N + P, margin=0.3)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N, P", [(1, 64), (64, 15), (65, 16), (200, 9), (257, 300), (1024, 40), (1025, 40), (4096, 33),
                                  (4097, 33)])
def test_force_calls(torch, R, orc, precision, N, P):
    w = wl(N, P)
    pos, q = inputs.sample(w)
    slab = gpu_slab(R, w, precision)
    kset = slab.draw_kset(w.seed)
    slab.set_kset(kset)
    pd, qd = to_dev(torch, pos), to_dev(torch, q)
    ref = orc.evaluate(oracle_slab(orc, w, slab.Lz_ext), pos, q, kset, targets=None)
    for _ in range(3):      # (the cell counts are clear again after each call)
        F, E = slab.forces(pd, qd, want_energy=True)
        assert rel_rms(F.cpu().numpy(), ref.F) <= TOL[precision]
        for eg, er in zip(E.cpu().numpy(), ref.energies()):
            assert abs(eg - er) <= TOL[precision] * energy_scale(ref)
    # accumulation, and each half alone: their sum is the whole
    G = slab.forces(pd, qd, flags=R.REAL)
    H = torch.full_like(F, 0.5)
    slab.forces(pd, qd, out=H, flags=R.KSPACE | R.IBC | R.ACCUMULATE)
    assert torch.allclose(G + H - 0.5, F, rtol=0, atol=1e-13 * float(F.abs().max()) + 1e-13)
    slab.check()


@pytest.mark.parametrize("M", [16, 17, 32, 33, 40])
def test_tables_of_the_call_without_a_handle(torch, R, M):
    """One launch carries 32 image orders and 32 image families; the rest
    follow in launches of their own.  Same inputs, same sums: only the order of
    FP64 sums may differ from the handle's."""
    w = inputs.Workload(f"tab{M}", 90, 12.0, 12.0, 0.1, 0.99, 0.98, 1.0, 4.0, 40, M, seed=M, margin=0.005)
    pos, q = inputs.sample(w)
    slab = gpu_slab(R, w, "fp64")
    kset = slab.draw_kset(w.seed)
    slab.set_kset(kset)
    pd, qd = to_dev(torch, pos), to_dev(torch, q)
    F, E = slab.forces(pd, qd, want_energy=True)
    Fs, Es = R.forces_noalloc(slab.params, to_dev(torch, kset, torch.int32), pd, qd, want_energy=True)
    assert rel_rms(Fs.cpu().numpy(), F.cpu().numpy()) <= 1e-12
    assert rel_rms(Es.cpu().numpy(), E.cpu().numpy()) <= 1e-12


def test_call_without_a_handle_changes_precision(torch, R):
    """FP32, FP64 with other sizes, and FP32 again: each call's workspaces are
    its own (an FP64 call once wrote the FP32 source records where the last
    FP32 call had kept them, across its own tables)."""
    for precision, N, P, M in (("fp32", 3000, 128, 8), ("fp64", 2141, 227, 5), ("fp32", 700, 40, 0), ("fp64", 65, 300, 2)):
        w = wl(N, P, M)
        pos, q = inputs.sample(w)
        slab = gpu_slab(R, w, precision)
        kset = slab.draw_kset(w.seed)
        slab.set_kset(kset)
        pd, qd = to_dev(torch, pos), to_dev(torch, q)
        F = slab.forces(pd, qd).cpu().numpy()
        for _ in range(2):
            Fs = R.forces_noalloc(slab.params, to_dev(torch, kset, torch.int32), pd, qd)
            assert rel_rms(Fs.cpu().numpy(), F) <= 1e-12


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N", [0, 300])
def test_call_without_a_handle_or_a_kset(torch, R, precision, N):
    """Without the k-space part the k-set may be NULL."""
    import ctypes
    w = wl(max(N, 1), 40)
    pos, q = inputs.sample(w)
    slab = gpu_slab(R, w, precision)
    kset = slab.draw_kset(w.seed)
    pd, qd = to_dev(torch, pos), to_dev(torch, q)
    flags = R.REAL | R.IBC
    want = R.forces_noalloc(slab.params, to_dev(torch, kset, torch.int32), pd, qd, flags=flags)
    F, E = torch.zeros_like(pd), torch.zeros(5, dtype=torch.float64, device="cuda")
    st = R.lib().rbe2d_forces_noalloc(ctypes.byref(slab.params), None, N, pd.data_ptr(), qd.data_ptr(), F.data_ptr(),
                                      E.data_ptr(), flags, None, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert st == R.RBE2D_OK
    assert torch.equal(F, want if N else torch.zeros_like(pd))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N", [24577, 98305, 140000])
def test_two_streams_from_a_first_call_on(torch, R, precision, N):
    """Two streams, forked before or after the cell list: the first call on new
    inputs equals the calls after it, bit by bit, and its parts add up."""
    w = wl(N, 33, M=2)
    pos, q = inputs.sample(w)
    slab = gpu_slab(R, w, precision)
    slab.set_kset(slab.draw_kset(w.seed))
    pd, qd = to_dev(torch, pos), to_dev(torch, q)
    F = slab.forces(pd, qd)
    e = slab.energy(pd, qd)
    for _ in range(3):
        assert torch.equal(slab.forces(pd, qd), F)
        assert torch.equal(slab.energy(pd, qd), e)
    G = slab.forces(pd, qd, flags=R.REAL) + slab.forces(pd, qd, flags=R.KSPACE | R.IBC)
    assert rel_rms(G.cpu().numpy(), F.cpu().numpy()) <= 1e-13
    slab.check()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N, P", [(1, 1025), (64, 1024), (65, 1030), (500, 4099), (4097, 1500), (17000, 1025)])
def test_many_wave_vectors(torch, R, orc, precision, N, P):
    """P about and beyond 1024: force passes in rows, with the energies, the
    potentials and the variances that end them."""
    w = wl(N, P)
    pos, q = inputs.sample(w)
    slab = gpu_slab(R, w, precision)
    kset = slab.draw_kset(w.seed)
    slab.set_kset(kset)
    pd, qd = to_dev(torch, pos), to_dev(torch, q)
    t = None if N <= 500 else np.random.default_rng(0).choice(N, 64, replace=False)
    o = oracle_slab(orc, w, slab.Lz_ext)
    ref = orc.evaluate(o, pos, q, kset, targets=t)
    at = np.arange(N) if t is None else t
    tol = TOL[precision]
    F, E = slab.forces(pd, qd, want_energy=True)
    assert torch.equal(slab.forces(pd, qd), F)
    assert rel_rms(F.cpu().numpy()[at], ref.F) <= tol
    if t is None:
        for eg, er in zip(E.cpu().numpy(), ref.energies()):
            assert abs(eg - er) <= tol * energy_scale(ref)
    # half of it on top of something: the sum of both calls
    H = torch.full_like(F, 0.5)
    slab.forces(pd, qd, out=H, flags=R.KSPACE | R.ACCUMULATE)
    G = slab.forces(pd, qd, flags=R.REAL | R.IBC)
    assert torch.allclose(G + H - 0.5, F, rtol=0, atol=1e-13 * float(F.abs().max()) + 1e-13)
    e = slab.energy(pd, qd)
    one = torch.ones((), dtype=torch.float64, device="cuda")
    dr, dq, _ = slab.energy_backward(pd, qd, one)
    # (the adjoint's FP32 sums go by sines and cosines, the forces' by polar amplitudes)
    assert rel_rms(-dr.cpu().numpy()[at], ref.F) <= tol
    assert rel_rms(dq.cpu().numpy()[at], ref.phi) <= tol
    assert abs(float(e[0]) - float(E[0])) <= 1e-12 * energy_scale_of(E)
    slab.check()


def energy_scale_of(E):
    return float(E[1:].abs().sum()) + 1e-300


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_variance_of_many_wave_vectors(torch, R, orc, precision):
    w = wl(300, 1100)
    pos, q = inputs.sample(w)
    slab = gpu_slab(R, w, precision)
    kset = slab.draw_kset(w.seed)
    slab.set_kset(kset)
    var = slab.force_variance(to_dev(torch, pos), to_dev(torch, q)).cpu().numpy()
    ref = orc.force_variance_estimate(oracle_slab(orc, w, slab.Lz_ext), pos, q, kset)
    assert rel_rms(var, ref) <= TOL[precision]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N, P", [(300, 512), (300, 513), (300, 1300), (100001, 520)])
def test_drawn_tables(torch, R, orc, precision, N, P):
    """k-sets drawn in MD steps, whose tables are sorted in chunks: the forces of
    the last step are those of its k-set at its positions."""
    w = wl(N, P, M=2)
    pos, q = inputs.sample(w)
    slab = gpu_slab(R, w, precision)
    slab.sample_kset(5, 0)
    P_, Q_ = to_dev(torch, pos), to_dev(torch, q)
    F_, V_ = slab.forces(P_, Q_), torch.zeros_like(P_)
    slab.md_run(P_, V_, Q_, F_, 1e-4, 0.2, w.H - 0.2, 5, 7, 3)
    slab.check()
    kset = slab.draw_kset(5, 9)
    assert np.array_equal(slab.get_kset(), kset)
    t = None if N <= 500 else np.random.default_rng(0).choice(N, 48, replace=False)
    ref = orc.evaluate(oracle_slab(orc, w, slab.Lz_ext), P_.cpu().numpy(), q, kset, targets=t)
    F = F_.cpu().numpy()
    assert rel_rms(F if t is None else F[t], ref.F) <= TOL[precision]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N, P", [(300, 40), (300, 1100), (5000, 40), (30000, 40), (140000, 17)])
def test_captured_calls(torch, R, precision, N, P):
    """Force calls, energies and steps captured by the caller: every replay, with
    eager work between them, equals the eager call."""
    w = wl(N, P, M=2)
    pos, q = inputs.sample(w)
    slab = gpu_slab(R, w, precision)
    slab.set_kset(slab.draw_kset(w.seed))
    pd, qd, p2 = to_dev(torch, pos), to_dev(torch, q), to_dev(torch, pos[::-1])
    one = torch.ones((), dtype=torch.float64, device="cuda")
    F, E = torch.empty_like(pd), torch.empty(5, dtype=torch.float64, device="cuda")

    def call():
        slab.forces(pd, qd, out=F, energy_out=E, want_energy=True)
        e = slab.energy(pd, qd)
        return (F, E, e) + tuple(slab.energy_backward(pd, qd, one))

    want = [t.clone() for t in call()]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = call()
    for _ in range(3):
        for t in out:
            t.fill_(7.0)
        slab.forces(p2, qd)                 # eager work on other positions
        g.replay()
        torch.cuda.synchronize()
        for t, u in zip(out, want):
            assert torch.equal(t, u)
    slab.check()
