"""GPU: the depositing pass over the forms its launch chooses between -- 768-thread workgroups
whose lanes load corners in pairs (16-cell bricks), the thermostat's 256-thread ones, bond tables
of one to three rows, with and without a bond length -- equals hpf_advance bit for bit, with the
density of the new positions exact; bricks that hold none, one and odd numbers of beads."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import dev  # noqa: E402
from paper_1310_2041_amd import engine, hpf  # noqa: E402
from synth import workloads as wl  # noqa: E402


def _state(B, halo, D, n):
    """n beads: most in one corner of the box, single ones elsewhere, some that cannot be binned."""
    s = wl.small_system(max(1, n // 6), 6, (27.3, 25.1, 29.9), (25, 23, 27), K=2, seed=n, n_solvent=n % 6 + 5)
    s.R[: s.N // 2] = np.mod(s.R[: s.N // 2], np.float32(9.7))
    s.bonds = np.random.default_rng(n).integers(-1, s.N, (D, s.N)).astype(np.int32) if D > 2 else s.bonds[:D]
    st = engine.HpfState.from_system(s, sort_brick=B, halo=halo)
    if n > 100:
        st.R[3] = float("nan")
    st.sort()
    torch.manual_seed(n)
    st.G.normal_()
    return st


@pytest.mark.parametrize("thermo", [False, True])
@pytest.mark.parametrize("B,halo,D,r0,n", [(16, 2, 2, 0.0, 1), (16, 2, 2, 0.0, 4001), (16, 1, 1, 0.5, 2999),
                                           (16, 2, 3, 0.0, 3007), (8, 1, 3, 0.5, 5003), (8, 2, 3, 0.0, 777),
                                           (8, 1, 4, 0.5, 1501)])
def test_depositing_pass_forms_equal_the_plain_pass(thermo, B, halo, D, r0, n):
    st = _state(B, halo, D, n)
    if thermo:
        st.set_thermostat(10.0, seed=5)
    R = [torch.empty_like(st.R), torch.empty_like(st.R)]
    V = [st.Vel.clone(), st.Vel.clone()]
    part = [torch.zeros((5, hpf.HPF_NPART), dtype=torch.float64, device="cuda") for _ in range(2)]
    kw = dict(thermostat=st.thermostat())
    hpf.hpf_get_device_status(clear=True)
    hpf.hpf_advance(st.R, R[0], V[0], st.T, st.mesh, st.K, st.G, st.bonds, 30.0, r0, st.box, 0.03,
                    e_part=part[0][0], kin_part=part[0][1:], **kw)
    flags = hpf.hpf_get_device_status(clear=True)
    hpf.hpf_advance_scatter(st.R, R[1], V[1], st.T, st.mesh, st.K, st.G, st.bonds, 30.0, r0, st.box, 0.03,
                            st.cell_start, B, halo, st.counts, st.scatter_work, e_part=part[1][0],
                            kin_part=part[1][1:], **kw)
    hpf.hpf_density_finish_cells(st.counts, st.N, st.mesh, st.K, B, halo, st.scatter_work)
    assert hpf.hpf_get_device_status(clear=True) == flags
    assert torch.equal(R[0].view(torch.int32), R[1].view(torch.int32))
    assert torch.equal(V[0].view(torch.int32), V[1].view(torch.int32))
    want = torch.zeros_like(st.counts)
    hpf.hpf_density_scatter(R[0], st.T, st.mesh, st.K, want)
    hpf.hpf_get_device_status(clear=True)
    assert torch.equal(st.counts, want)
    a, b = part[0].sum(1), part[1].sum(1)
    if bool(torch.isfinite(a).all()):
        scale = part[0].abs().sum(1) + 1e-300
        assert bool(((a - b).abs() / scale).max() <= 1e-12)
