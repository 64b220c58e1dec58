"""GPU: the energies of the depositing pass in each form that its launch chooses between, the first
half step with its deposit over masses, brick sizes and the workgroup's edges, and steps whose field
is kept for some of them -- each against the separate calls."""
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


def _system(n, B, halo, D, M=(25, 23, 27)):
    s = wl.small_system(max(1, n // 6), 6, tuple(1.09 * m for m in M), M, seed=n, n_solvent=n % 6 + 5)
    s.R[: s.N // 2] = np.mod(s.R[: s.N // 2], np.float32(9.7))          # most in one corner
    s.bonds = np.random.default_rng(n).integers(-1, s.N, (D, s.N)).astype(np.int32)
    st = engine.HpfState.from_system(s, sort_brick=B, halo=halo)
    st.sort()
    return st


@pytest.mark.parametrize("masses", [False, True])
@pytest.mark.parametrize("thermo", [False, True])
@pytest.mark.parametrize("B,halo,D,r0,n", [(16, 2, 2, 0.0, 4001), (16, 1, 1, 0.5, 2999), (16, 2, 3, 0.0, 3007),
                                           (8, 1, 2, 0.0, 5003), (8, 1, 2, 0.5, 4999), (8, 1, 3, 0.5, 5003),
                                           (8, 2, 3, 0.0, 777), (8, 1, 4, 0.5, 1501)])
def test_depositing_pass_energies(masses, thermo, B, halo, D, r0, n):
    _check_energies(_system(n, B, halo, D), masses, thermo, B, halo, r0, n)


@pytest.mark.parametrize("bricks,D,r0", [(256, 2, 0.0), (320, 2, 0.5), (320, 3, 0.0), (704, 3, 0.5), (832, 4, 0.5),
                                         (896, 4, 0.0), (1088, 4, 0.5), (1088, 3, 0.0), (1088, 1, 0.0)])
def test_depositing_pass_energies_with_the_thermostat_by_bricks(bricks, D, r0):
    """Both sides of the numbers of bricks at which its workgroup changes."""
    st = _system(20000, 8, 1, D, M=(64, 64, bricks // 8))
    assert hpf.sort_key_count(st.mesh, 8) == bricks
    _check_energies(st, bricks % 256 == 0, True, 8, 1, r0, bricks)


def _check_energies(st, masses, thermo, B, halo, r0, n):
    """All beads can be binned, so that every sum is finite. The two passes group the same FP64 terms
    differently: each sum is within 1e-12 of the sum of its terms' sizes."""
    if thermo:
        st.set_thermostat(10.0, seed=5)
    torch.manual_seed(n)
    st.G.normal_()
    im = torch.rand(st.N, device="cuda") + 0.5 if masses else None
    R = [torch.empty_like(st.R) for _ in range(2)]
    V = [st.Vel.clone() for _ in range(2)]
    part = [torch.full((5, hpf.HPF_NPART), 3.0, dtype=torch.float64, device="cuda") for _ in range(2)]
    kw = dict(thermostat=st.thermostat(), inv_mass=im)
    hpf.hpf_advance(st.R, R[0], V[0], st.T, st.mesh, st.K, st.G, st.bonds, 30.0, r0, st.box, 0.03,
                    e_part=part[0][0], kin_part=part[0][1:], **kw)
    hpf.hpf_advance_scatter(st.R, R[1], V[1], st.T, st.mesh, st.K, st.G, st.bonds, 30.0, r0, st.box, 0.03,
                            st.cell_start, B, halo, st.counts, st.scatter_work, e_part=part[1][0],
                            kin_part=part[1][1:], **kw)
    assert hpf.hpf_get_device_status(clear=True) == 0
    assert _same(R[0], R[1]) and _same(V[0], V[1])
    a, b = part[0].sum(1), part[1].sum(1)
    scale = part[0].abs().sum(1)
    assert bool(torch.isfinite(scale).all()) and bool((scale[:2] > 0).all())
    assert bool(((a - b).abs() <= 1e-12 * scale).all())


@pytest.mark.parametrize("masses", [False, True])
@pytest.mark.parametrize("B,halo,M,fill", [(8, 1, (24, 24, 25), (0, 1, 511, 512, 513, 1024, 1025)),
                                           (8, 2, (24, 33, 24), (3000, 0, 1)), (16, 2, (48, 33, 40), (5000, 511, 0, 1)),
                                           (8, 1, (96, 96, 88), (700, 0, 255, 256, 257, 513)),
                                           (8, 1, (24, 24, 24), ())])
def test_verlet_scatter_over_masses_and_brick_fills(masses, B, halo, M, fill):
    """fill[b] beads in brick b, none anywhere else."""
    rng = np.random.default_rng(B + len(fill))
    nb = [-(-m // B) for m in M]
    ids = np.repeat(np.arange(len(fill)), fill)
    N = len(ids)
    xyz = np.stack([ids % nb[0], ids // nb[0] % nb[1], ids // (nb[0] * nb[1])], 1) * float(B)
    s = wl.small_system(1, max(N, 1), tuple(float(m) for m in M), M, K=2, seed=5)
    pos = np.minimum(xyz + 0.01 + rng.random((N, 3)) * (B - 0.1), np.asarray(M) - 0.01).astype(np.float32)
    s.bonds[:] = -1
    st = engine.HpfState.from_system(s, sort_brick=B, halo=halo)
    mesh = st.mesh
    st.R[:N] = dev(pos, torch.float32)
    st.sort()
    im = torch.rand(max(N, 1), device="cuda") + 0.5 if masses else None
    if N == 0:                                     # no beads at all, with the arrays of none
        st.cell_start.zero_()
    R, V, F, T = st.R[:N].clone(), st.Vel[:N].clone(), torch.randn((N, 3), device="cuda") * 20, st.T[:N].clone()
    im = im[:N] if masses else None
    R2, V2 = R.clone(), V.clone()
    hpf.hpf_get_device_status(clear=True)
    hpf.verlet_step(R, V, F, 0.05, st.box, 1, inv_mass=im)
    want = torch.zeros_like(st.counts)
    hpf.hpf_density_scatter(R, T, mesh, 2, want)
    hpf.hpf_verlet_scatter(R2, V2, F, T, 0.05, st.box, mesh, 2, st.cell_start, B, halo, st.counts, st.scatter_work,
                           inv_mass=im)
    hpf.hpf_density_finish_cells(st.counts, N, mesh, 2, B, halo, st.scatter_work)
    assert _same(R, R2) and _same(V, V2)
    assert torch.equal(st.counts, want)
    assert hpf.hpf_get_device_status(clear=True) == 0


@pytest.mark.parametrize("stencil", ["centred", "staggered"])
def test_steps_with_a_field_interval_equal_the_separate_calls(stencil):
    """field_every = 3 over 14 steps, with sorts on steps that rebuild the field (6), that follow one
    (4) and that do not (11): step() changes between its two half steps."""
    s = wl.lipid_system(200, 3000, seed=9)
    a, b = (engine.HpfState.from_system(s, stencil=stencil, field_every=3) for _ in range(2))
    for st in (a, b):
        st.start(sort=True)
    for i in range(1, 15):
        sort = i in (4, 6, 11)
        a.step(report=True, sort=sort)
        hpf.verlet_step(b.R, b.Vel, b.F, b.dt, b.box, 1)
        if sort:
            b.sort()
        b.forces(report=True, rebuild=i % 3 == 0)
        hpf.verlet_step(None, b.Vel, b.F, b.dt, b.box, 2, kin_part=b.part[engine.ROW_KE:engine.ROW_KE + 4])
        hpf.hpf_reduce_partials(b.part, engine.N_ROWS, b.energy)
        assert torch.equal(a.tag, b.tag)
        assert _same(a.R, b.R) and _same(a.Vel, b.Vel) and _same(a.F, b.F), i
        assert np.allclose(host(a.energy), host(b.energy), rtol=1e-12, atol=1e-9)
