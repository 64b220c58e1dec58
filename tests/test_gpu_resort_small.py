"""GPU: the re-sort's passes for small bricks -- a wavefront per brick, bricks too large for one
among them (stayers and movers at that limit and past the LDS), empty bricks, numbers of bricks
that are no multiple of a workgroup's -- against the full sort."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import host  # noqa: E402
from paper_1310_2041_amd import engine, hpf  # noqa: E402
from synth import workloads as wl  # noqa: E402


def _check(s, B, moved):
    st = engine.HpfState.from_system(s, sort_brick=B, halo=0)
    st.sort()
    st.R.copy_(moved(st.R))
    ref = engine.HpfState.from_system(s, sort_brick=B, halo=0)
    for n in ("R", "Vel", "T", "tag", "bonds"):
        getattr(ref, n).copy_(getattr(st, n))
    st.work.view(torch.int32)[: st.work.numel() // 4].fill_(0x7eadbeef)
    hpf.hpf_get_device_status(clear=True)
    st.resort, ref.resort = True, False
    st.sort()
    ref.sort()
    for x, y in zip(st.host_beads(), ref.host_beads()):
        assert np.array_equal(x, y)
    assert np.array_equal(host(st.cell_start), host(ref.cell_start))
    assert hpf.hpf_get_device_status(clear=True) == 0


@pytest.mark.parametrize("share", [0.0, 0.02, 0.5, 1.0])
@pytest.mark.parametrize("n,M,B", [(1, 9, 3), (300, (9, 12, 15), 3), (3000, (13, 9, 11), 1), (20000, 40, 3),
                                   (90000, (100, 101, 70), 4), (250000, 104, 8)])
def test_small_bricks(n, M, B, share):
    s = wl.small_system(max(1, n // 10), min(n, 10), tuple(1.1 * m for m in np.broadcast_to(M, 3)), M, seed=n,
                        n_solvent=n % 10 if n > 10 else 0)
    g = torch.Generator("cuda").manual_seed(n)

    def moved(R):
        far = torch.rand(R.shape, device="cuda", generator=g) * torch.tensor(s.L, device="cuda").float() * 0.999
        return torch.where(torch.rand(len(R), 1, device="cuda", generator=g) < share, far, R)

    _check(s, B, moved)


@pytest.mark.parametrize("stay,come", [(1023, 64), (1024, 65), (1025, 63), (1025, 0), (0, 64), (0, 65), (10, 2048),
                                       (10, 2049), (5000, 700)])
def test_a_large_brick_among_small_ones(stay, come):
    """`stay` beads of one brick of 4096 stay in it, `come` beads come in from others; the brick's
    neighbours by its workgroup hold a few beads."""
    rng = np.random.default_rng(stay + come)
    N = stay + come + 9000
    s = wl.small_system(1, N, 64.0, 64, seed=3)
    s.bonds[:] = -1
    pos = rng.random((N, 3)) * 64.0
    big = np.array([20.0, 40.0, 8.0])
    pos[(np.floor(pos / 4) == big / 4).all(1)] += 4.0          # only those meant to be there
    order = rng.permutation(N)
    pos[order[:stay]] = big + 0.01 + rng.random((stay, 3)) * 3.9
    s.R[:, :3] = pos.astype(np.float32)
    come_tags = torch.from_numpy(np.sort(order[stay:stay + come])).cuda()
    st = engine.HpfState.from_system(s, sort_brick=4, halo=0)
    assert hpf.sort_key_count(st.mesh, 4) == 4096
    to = torch.from_numpy((big + 0.01 + rng.random((N, 3)) * 3.9).astype(np.float32)).cuda()
    st.sort()
    tags = st.tag.clone()

    def moved(R):
        return torch.where(torch.isin(tags, come_tags)[:, None], to, R)

    _check(s, 4, moved)
