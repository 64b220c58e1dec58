"""GPU: the cell-list scatter's lists of strays, kept in each brick's own stretch -- bricks with
no bead, one bead, all of them strays or none -- over both workgroup sizes (few bricks, many, and
boxes that fill a CU's LDS): the counts equal those of the any-order scatter."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1310_2041_amd import engine, hpf  # noqa: E402
from synth import workloads as wl  # noqa: E402


@pytest.mark.parametrize("n,M,B,halo,K", [(1, 10, 4, 1, 1), (500, (30, 29, 31), 4, 0, 2), (20011, 30, 4, 2, 2),
                                          (1200, (33, 19, 20), 8, 1, 3), (30011, (23, 21, 40), 16, 2, 2),
                                          (9001, (90, 97, 99), 16, 2, 2)])
def test_strays_of_every_brick_are_counted_once(n, M, B, halo, K):
    s = wl.small_system(max(1, n // 10), min(n, 10), tuple(1.1 * m for m in np.broadcast_to(M, 3)), M, K=K, seed=n,
                        n_solvent=n % 10 if n > 10 else 0)
    st = engine.HpfState.from_system(s, sort_brick=B, halo=halo)
    st.sort()
    L = torch.tensor(s.L, device="cuda", dtype=torch.float32).expand(3)
    R0 = st.R.clone()
    for share in (0.0, 0.01, 0.5, 1.0):
        moved = torch.rand(st.N, device="cuda", generator=torch.Generator("cuda").manual_seed(n)) < share
        far = torch.rand((st.N, 3), device="cuda", generator=torch.Generator("cuda").manual_seed(n + 1))
        st.R[:, :3] = torch.where(moved[:, None], far * L * 0.999, R0[:, :3])
        # the beads listed in one half of the bricks all leave for one corner cell
        if share == 0.5:
            st.R[: st.N // 2, :3] = 0.3
        st.counts.fill_(-1)
        for _ in range(2):
            hpf.hpf_density_scatter_cells(st.R, st.T, st.mesh, st.K, st.cell_start, B, halo, st.counts,
                                          st.scatter_work)
        want = torch.zeros_like(st.counts)
        hpf.hpf_density_scatter(st.R, st.T, st.mesh, st.K, want)
        assert torch.equal(st.counts, want)
        assert hpf.hpf_get_device_status() == 0
