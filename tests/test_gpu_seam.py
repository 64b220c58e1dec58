"""GPU: the sums of the deposit boxes on meshes whose last brick along an axis is thin, as wide as
two halos and one cell more, in bricks hardly wider than the halo and in two bricks an axis -- where
a point lies in three boxes or more along an axis, or just does not -- equal the any-order scatter,
and the potential fused with the sum equals the potential of those counts bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1310_2041_amd import engine, hpf  # noqa: E402
from synth import workloads as wl  # noqa: E402


@pytest.mark.parametrize("M,B,halo,K", [((17, 18, 19), 8, 1, 2), ((25, 26, 28), 8, 2, 3), ((29, 24, 25), 8, 2, 1),
                                        ((10, 11, 13), 3, 2, 2), ((11, 12, 13), 8, 1, 4), ((33, 34, 37), 16, 2, 2),
                                        ((13, 27, 20), 6, 0, 5), ((19, 18, 17), 8, 1, 8)])
def test_box_sums_at_the_seam(M, B, halo, K):
    s = wl.small_system(900, 6, tuple(1.08 * m for m in M), M, K=K, seed=B + halo + K, n_solvent=2000)
    st = engine.HpfState.from_system(s, sort_brick=B, halo=halo)
    st.sort()
    want = torch.zeros_like(st.counts)
    hpf.hpf_density_scatter(st.R, st.T, st.mesh, st.K, want)
    st.counts.fill_(-1)
    hpf.hpf_density_scatter_cells(st.R, st.T, st.mesh, st.K, st.cell_start, B, halo, st.counts, st.scatter_work)
    assert torch.equal(st.counts, want)
    # the beads a few tenths of a cell further, deposited by the step's pass
    st.counts.zero_()
    st.G.zero_()
    st.Vel.normal_(0.0, 8.0)
    R2, V = torch.empty_like(st.R), st.Vel.clone()
    hpf.hpf_advance_scatter(st.R, R2, V, st.T, st.mesh, st.K, st.G, st.bonds, 0.0, 0.0, st.box, 0.03, st.cell_start, B,
                            halo, st.counts, st.scatter_work)
    counts = st.counts.clone()
    hpf.hpf_density_finish_cells(counts, st.N, st.mesh, st.K, B, halo, st.scatter_work)
    want.zero_()
    hpf.hpf_density_scatter(R2, st.T, st.mesh, st.K, want)
    assert torch.equal(counts, want)
    V1, V2 = torch.empty_like(st.V), torch.empty_like(st.V)
    w = torch.zeros((2, hpf.HPF_NPART), dtype=torch.float64, device="cuda")
    hpf.hpf_field_potential(want, st.mesh, st.field, V1, w[0])
    hpf.hpf_field_potential_cells(st.counts, st.N, st.mesh, st.field, B, halo, st.scatter_work, V2, w[1])
    assert torch.equal(V1.view(torch.int32), V2.view(torch.int32))
    assert not st.counts.any()
    a, b = w.sum(1).tolist()
    assert a == pytest.approx(b, rel=1e-12)
    assert hpf.hpf_get_device_status() == 0
    assert np.isfinite(a)
