"""GPU: the cell scatter's long lists of strays, which all workgroups share -- one brick's beads
all gone, lists at the length from which they are shared, more long lists than there is room to
name, a droplet in a mesh of many bricks -- single system and batch: the counts equal those of
the any-order scatter."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1310_2041_amd import engine, hpf  # noqa: E402
from synth import workloads as wl  # noqa: E402

LONG = 2048


def _placed(fill, M, K, seed, extra=0):
    """fill[b] beads in brick b of 8 cells, `extra` anywhere; positions and the system."""
    rng = np.random.default_rng(seed)
    nb = [-(-m // 8) for m in M]
    ids = np.repeat(list(fill), list(fill.values()))
    xyz = np.stack([ids % nb[0], ids // nb[0] % nb[1], ids // (nb[0] * nb[1])], 1) * 8.0
    pos = np.concatenate([xyz + 0.01 + rng.random((len(ids), 3)) * 7.9, rng.random((extra, 3)) * M])
    s = wl.small_system(1, len(pos), tuple(float(m) for m in M), M, K=K, seed=seed)
    s.R[:, :3] = np.minimum(pos, np.asarray(M) - 0.01).astype(np.float32)
    s.bonds[:] = -1
    return s


def _moved(R, tag, gone, M, seed):
    """The beads of tags below `gone` go anywhere at least 12 cells away along x."""
    g = torch.Generator("cuda").manual_seed(seed)
    to = torch.rand(R.shape, device="cuda", generator=g) * torch.tensor(M, device="cuda").float() * 0.999
    to[:, 0] = torch.remainder(R[:, 0] + 12 + torch.rand(len(R), device="cuda", generator=g) * (M[0] - 24.0),
                               float(M[0]))
    to[:, 0].clamp_(max=M[0] * (1 - 1e-6))
    return torch.where((tag < gone)[:, None], to, R)


CASES = [("many_small_bricks", (96, 96, 88), {i: 3000 for i in (7, 800, 1583)}, 7000, 30000),
         ("one_brick", (64, 64, 64), {77: 300000}, 300000, 9000),
         ("at_the_limit", (64, 72, 64), {5: LONG + 1, 60: LONG, 61: LONG - 1}, 3 * LONG, 2000),
         ("few_bricks", (40, 33, 40), {3: 20000, 9: 2500}, 22500, 100),
         ("more_than_named", (64, 64, 64), {i: 2100 for i in range(100, 150)}, 50 * 2100, 50000),
         ("part_of_a_brick", (128, 64, 64), {i: 9000 for i in (0, 511, 512, 1000, 1023)}, 30000, 20000)]


@pytest.mark.parametrize("M,fill,gone,extra", [c[1:] for c in CASES], ids=[c[0] for c in CASES])
def test_long_lists_are_counted_once(M, fill, gone, extra):
    s = _placed(fill, M, 2, len(fill), extra)
    st = engine.HpfState.from_system(s, sort_brick=8, halo=1)
    st.sort()
    st.R.copy_(_moved(st.R, st.tag, gone, M, 3))
    want = torch.zeros_like(st.counts)
    hpf.hpf_density_scatter(st.R, st.T, st.mesh, st.K, want)
    for fillv in (0, 255):                        # whatever the workspace held
        st.scatter_work.fill_(fillv)
        st.counts.fill_(-1)
        for _ in range(2):
            hpf.hpf_density_scatter_cells(st.R, st.T, st.mesh, st.K, st.cell_start, 8, 1, st.counts,
                                          st.scatter_work)
        assert torch.equal(st.counts, want)
    assert hpf.hpf_get_device_status(clear=True) == 0


def test_long_lists_of_a_batch():
    """Strays of a replica between two others; the first step's scatter, which follows the sort,
    has none, so the positions move between hpf_batch_start and hpf_batch_density."""
    Ms = [(24, 32, 24), (64, 32, 40), (16, 24, 16)]
    fills = [{0: 3000}, {9: 70000, 11: 2500, 100: 2049}, {1: 200}]
    systems = [_placed(f, M, 2, i + 1, 3000) for i, (f, M) in enumerate(zip(fills, Ms))]
    b = engine.BatchState(systems, sort_every=100, brick=8, halo=1, fuse_deposit=False)
    b.start()
    R, tag = b._current("R"), b._current("tag")
    for r, s in enumerate(systems):
        o, e = int(b.offsets[r]), int(b.offsets[r + 1])
        if r < 2:
            R[o:e] = _moved(R[o:e], tag[o:e] - o, sum(fills[r].values()), Ms[r], r)
    out = b.density()
    T = b._current("T")
    at = 0
    for r, s in enumerate(systems):
        o, e = int(b.offsets[r]), int(b.offsets[r + 1])
        mesh = hpf.hpf_mesh_make(s.L, s.M, s.N)
        want = torch.zeros(b.K * b.nm[r], dtype=torch.int64, device="cuda")
        hpf.hpf_density_scatter(R[o:e].contiguous(), T[o:e].contiguous(), mesh, b.K, want.view(b.K, -1))
        assert torch.equal(out[at:at + len(want)], want), r
        at += len(want)
    assert hpf.hpf_get_device_status(clear=True) == 0
