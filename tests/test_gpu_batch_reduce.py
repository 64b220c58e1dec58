"""GPU: a batch's energies over replicas whose rows hold one item, exactly a wavefront of them,
one more and several -- against each system run by itself (sums in FP64 only regroup)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1310_2041_amd import engine, hpf  # noqa: E402
from synth import workloads as wl  # noqa: E402


@pytest.mark.parametrize("fuse,brick,chunk", [(True, 4, 512), (True, 8, 512), (False, 8, 512), (False, 8, 4096)])
def test_batch_energies_equal_single_systems(fuse, brick, chunk):
    systems = [wl.small_system(nc, 10, L, M, seed=nc) for nc, L, M in
               [(1, 13.3, 13), (3276, 17.2, 16), (3277, 17.2, 17), (7000, 23.4, 23)]]
    b = engine.BatchState(systems, sort_every=4, brick=brick, bead_chunk=chunk, mesh_chunk=max(chunk, 2048),
                          fuse_deposit=fuse)
    b.start()
    b.step(3, report_last=True)
    E = b.energies()
    for r, s in enumerate(systems):
        st = engine.HpfState.from_system(s)
        st.start(sort=True)
        st.prime()
        e = st.run_fused(3, report_every=3, sort_every=4)[-1]
        for j, key in enumerate(["KE", "E_bond", "W", "E_tot"]):
            assert E[r, j] == pytest.approx(e[key], rel=1e-12, abs=1e-9)
        np.testing.assert_allclose(E[r, 4:7], np.asarray(e["P"]), rtol=0, atol=1e-9)
    assert hpf.hpf_get_device_status() == 0
