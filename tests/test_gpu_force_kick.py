"""GPU: the fused passes of the separate-call step. hpf_force_kick equals gather (either
stencil) + bonds + angles + second half kick, and hpf_verlet_scatter the first half step plus
the density of the new positions, bit for bit; step() over both equals the separate calls."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import dev, host  # noqa: E402
from paper_1310_2041_amd import engine, hpf  # noqa: E402
from synth import workloads as wl  # noqa: E402


def _same(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


def _tables(rng, N, D, A, bad):
    """Bond and angle tables with empty slots anywhere, and `bad` out-of-range entries each."""
    bonds = rng.integers(-1, N, (D, N)).astype(np.int32)
    ang = np.zeros((3 * A, N), np.int32)
    for r in range(A):
        ang[3 * r] = np.where(rng.random(N) < 0.4, -1, rng.integers(0, N, N))
        ang[3 * r + 1] = rng.integers(0, N, N)
        ang[3 * r + 2] = rng.integers(0, 2, N) + 2 * rng.integers(0, 2, N)
    for _ in range(bad):
        if D:
            bonds[rng.integers(D), rng.integers(N)] = N + 3
        if A:
            ang[3 * rng.integers(A) + 1, rng.integers(N)] = -1
            ang[3 * rng.integers(A) + 2, rng.integers(N)] = 9
    return bonds, ang


@pytest.mark.parametrize("stag", [False, True])
@pytest.mark.parametrize("N,D,A,r0,bad", [(1, 0, 0, 0.0, 0), (255, 2, 0, 0.0, 0), (257, 3, 3, 0.5, 2),
                                          (3000, 5, 1, 0.0, 0), (70001, 4, 5, 0.5, 5)])
def test_force_kick_equals_the_separate_calls(stag, N, D, A, r0, bad):
    rng = np.random.default_rng(N + D)
    K, M, L = 3, (14, 17, 15), (13.1, 16.4, 14.9)
    R = dev((rng.random((N, 3)) * L).astype(np.float32), torch.float32)
    T = dev(rng.integers(0, K, N).astype(np.uint8), torch.uint8)
    V0 = dev(rng.standard_normal((N, 3)).astype(np.float32), torch.float32)
    im = dev((0.5 + rng.random(N)).astype(np.float32), torch.float32) if N % 2 else None
    bonds, ang = _tables(rng, N, D, A, bad)
    bonds, ang = dev(bonds, torch.int32) if D else None, dev(ang, torch.int32) if A else None
    mesh = hpf.hpf_mesh_make(L, M, N)
    nm = int(np.prod(M))
    pot = dev(rng.standard_normal((K, nm)).astype(np.float32), torch.float32)
    G = torch.empty((K, nm, 3), dtype=torch.float32, device="cuda")
    hpf.hpf_field_gradient(pot, mesh, K, G)
    par = dict(k=(12.0, 7.0), theta0=(2.0, 3.1), form=(0, 1))
    part = [torch.full((6, hpf.HPF_NPART), 7.0, dtype=torch.float64, device="cuda") for _ in range(2)]
    F = [torch.empty_like(R) for _ in range(2)]
    Vel = [V0.clone(), V0.clone()]
    hpf.hpf_get_device_status(clear=True)
    if stag:
        hpf.hpf_force_gather_staggered(R, T, mesh, K, pot, F[0])
    else:
        hpf.hpf_force_gather(R, T, mesh, K, G, F[0])
    hpf.bond_forces(R, bonds, 100.0, r0, L, F[0], part[0][0])
    if A:
        hpf.angle_forces(R, ang, box=L, F=F[0], e_part=part[0][1], **par)
    else:
        part[0][1] = 0.0
    hpf.verlet_step(None, Vel[0], F[0], 0.03, L, 2, inv_mass=im, kin_part=part[0][2:])
    flags = hpf.hpf_get_device_status(clear=True)
    hpf.hpf_force_kick(R, T, mesh, K, pot if stag else G, bonds, 100.0, r0, L, F[1], Vel[1], 0.03, stag, ang,
                       par["k"], par["theta0"], par["form"], inv_mass=im, e_part=part[1][0], ea_part=part[1][1],
                       kin_part=part[1][2:])
    assert hpf.hpf_get_device_status(clear=True) == flags
    assert _same(F[0], F[1]) and _same(Vel[0], Vel[1])
    assert torch.equal(part[0].view(torch.int64), part[1].view(torch.int64))   # bits: a degenerate angle gives NaN


@pytest.mark.parametrize("halo,moved,bad", [(0, 0.0, 0), (1, 0.4, 5), (2, 3.0, 0)])
def test_verlet_scatter_equals_half_step_and_density(halo, moved, bad):
    s = wl.small_system(700, 9, (21.0, 17.5, 30.2), (19, 16, 27), K=4, seed=halo, n_solvent=2500)
    st = engine.HpfState.from_system(s, halo=halo)
    if bad:
        st.R[:bad, 0] = float("nan")
    st.sort()
    rng = np.random.default_rng(3)
    st.R += dev((rng.standard_normal((s.N, 3)) * moved).astype(np.float32), torch.float32)
    st.F.copy_(dev(rng.standard_normal((s.N, 3)).astype(np.float32), torch.float32))
    R, V = st.R.clone(), st.Vel.clone()
    hpf.hpf_get_device_status(clear=True)
    hpf.verlet_step(R, V, st.F, 0.03, st.box, 1)
    want = torch.zeros_like(st.counts)
    hpf.hpf_density_scatter(R, st.T, st.mesh, st.K, want)
    flags = hpf.hpf_get_device_status(clear=True)
    hpf.hpf_verlet_scatter(st.R, st.Vel, st.F, st.T, 0.03, st.box, st.mesh, st.K, st.cell_start, st.B, st.halo,
                           st.counts, st.scatter_work)
    hpf.hpf_density_finish_cells(st.counts, s.N, st.mesh, st.K, st.B, st.halo, st.scatter_work)
    assert hpf.hpf_get_device_status(clear=True) == flags
    assert _same(st.R, R) and _same(st.Vel, V)
    assert torch.equal(st.counts, want)


@pytest.mark.parametrize("stencil", ["centred", "staggered"])
def test_steps_equal_the_separate_calls(stencil):
    """12 steps with sorts, energies and the angle table, against the calls one by one; then the
    same steps replayed from a graph, twice, with eager work between."""
    s = wl.lipid_system(300, 5000, seed=8)
    a = engine.HpfState.from_system(s, stencil=stencil)
    b = engine.HpfState.from_system(s, stencil=stencil)
    for st in (a, b):
        st.start(sort=True)

    def plain(st, sort):
        hpf.verlet_step(st.R, st.Vel, st.F, st.dt, st.box, 1)
        if sort:
            st.sort()
        st.forces(report=True)
        hpf.verlet_step(None, st.Vel, st.F, st.dt, st.box, 2, kin_part=st.part[engine.ROW_KE:engine.ROW_KE + 4])
        hpf.hpf_reduce_partials(st.part, engine.N_ROWS, st.energy)

    def check():
        assert torch.equal(a.tag, b.tag)
        assert _same(a.R, b.R) and _same(a.Vel, b.Vel) and _same(a.F, b.F)
        assert np.allclose(host(a.energy), host(b.energy), rtol=1e-12, atol=1e-9)

    for i in range(12):
        a.step(report=True, sort=i % 5 == 4)
        plain(b, i % 5 == 4)
    check()
    g = engine.Graph(lambda: [a.step(report=True, sort=i in (2, 5)) for i in range(8)])
    for _ in range(2):
        g.launch(torch.cuda.current_stream())
        for i in range(8):
            plain(b, i in (2, 5))
        torch.cuda.synchronize()
        check()
