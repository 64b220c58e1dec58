"""GPU: the full counting sort at the sizes where its launches differ -- one column block or
several, the key range looked up or not, four, two and one wavefronts per placement
workgroup, key matching by rounds, few and many distinct keys per wavefront -- against the
oracle's (brick, tag) permutation, with the bond table renumbered and every key start."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle  # noqa: E402
from gpu_util import host  # noqa: E402
from paper_1310_2041_amd import engine, hpf  # noqa: E402
from synth import workloads as wl  # noqa: E402

CASES = [
    ("one_chunk", 3, 9, 3, 14, 16),             # 27 + beads, one chunk, a part-filled row
    ("small_columns", 3276, 20, 8, 20, 16),     # 65,520 beads: 64 chunks of 1024
    ("block_columns", 3300, 20, 8, 20, 80),     # 66,080 beads: 65 chunks
    ("solvent", 50, 12, 4, 40, 90000),          # 64 distinct keys per wavefront
    ("range", 4000, 20, 3, 40, 5),              # 2744 + 1 keys: above the range limit
    ("two_rows", 9000, 12, 2, 46, 3),           # 12,167 + 1 keys: two wavefronts a workgroup
    ("one_row", 9000, 12, 2, 58, 3),            # 24,389 + 1 keys: one
    ("rounds", 4000, 50, 16, 45, 7),            # 7400 beads a key: matching by rounds
]


@pytest.mark.parametrize("n_chains,chain_len,B,M,n_solvent", [c[1:] for c in CASES], ids=[c[0] for c in CASES])
def test_full_sort_paths_match_the_oracle(n_chains, chain_len, B, M, n_solvent):
    s = wl.small_system(n_chains, chain_len, 1.13 * M, M, seed=31, n_solvent=n_solvent)
    s, _ = wl.permuted(s, seed=32)
    perm, keys = oracle.sort_perm(s.R, s.tag, s.L, s.M, B)
    inv = np.empty(s.N, dtype=np.int64)
    inv[perm] = np.arange(s.N)
    st = engine.HpfState.from_system(s, sort_brick=B, halo=0)
    st.sort()
    assert np.array_equal(host(st.tag), s.tag[perm])
    assert np.array_equal(host(st.R), s.R[perm])
    assert np.array_equal(host(st.Vel), s.V[perm])
    assert np.array_equal(host(st.T), s.T[perm])
    moved = s.bonds[:, perm]
    assert np.array_equal(host(st.bonds), np.where(moved >= 0, inv[np.maximum(moved, 0)], -1))
    nk = hpf.sort_key_count(st.mesh, B)
    assert np.array_equal(host(st.cell_start), np.searchsorted(np.sort(keys), np.arange(nk + 2), side="left"))
    assert hpf.hpf_get_device_status(clear=True) == 0


@pytest.mark.parametrize("N,M,B,into", [(40, 12, 4, 40), (700, 24, 8, 64), (700, 24, 8, 65), (3000, 24, 8, 513),
                                        (6000, 24, 8, 2048), (6000, 24, 8, 2049), (9000, 45, 3, 0)])
def test_resort_movers_match_the_oracle(N, M, B, into):
    """`into` beads of a sorted system move into one brick (the runs of 64, the LDS capacity of
    2048 movers); into = 0: every bead leaves one brick for more bricks than the LDS table of
    destinations holds."""
    rng = np.random.default_rng(into + N)
    L = 1.0 * M
    R = (rng.random((N, 3)) * (L if into else B)).astype(np.float32)
    s = wl.small_system(N // 10, 10, L, M, seed=2)
    s.R[:] = R[: s.N]
    st = engine.HpfState.from_system(s, sort_brick=B, halo=0)
    st.sort()
    pos = st.R.cpu().numpy().copy()
    if into:
        pick = rng.permutation(s.N)[:into]
        pos[pick] = (B + rng.random((into, 3)) * B).astype(np.float32)
    else:
        pos = (rng.random((s.N, 3)) * L).astype(np.float32)
    st.R.copy_(torch.from_numpy(pos))
    st.resort = True
    tag = host(st.tag)
    perm, keys = oracle.sort_perm(pos, tag, s.L, s.M, B)
    bonds = host(st.bonds)[:, perm]
    inv = np.empty(s.N, dtype=np.int64)
    inv[perm] = np.arange(s.N)
    st.sort()
    assert np.array_equal(host(st.tag), tag[perm])
    assert np.array_equal(host(st.R), pos[perm])
    assert np.array_equal(host(st.bonds), np.where(bonds >= 0, inv[np.maximum(bonds, 0)], -1))
    nk = hpf.sort_key_count(st.mesh, B)
    assert np.array_equal(host(st.cell_start), np.searchsorted(np.sort(keys), np.arange(nk + 2), side="left"))
    assert hpf.hpf_get_device_status(clear=True) == 0
