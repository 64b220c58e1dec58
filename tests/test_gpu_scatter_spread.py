"""GPU: the any-order density scatter where a chunk's beads spread over the whole mesh (direct
global atomics, two lanes per bead): bit-exact against the oracle, at part-filled wavefronts and
chunks, across the periodic seam and with beads that must be skipped."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle  # noqa: E402
from gpu_util import counts_np, dev  # noqa: E402
from paper_1310_2041_amd import hpf  # noqa: E402


@pytest.mark.parametrize("N,M,K,bad", [(2, (32, 31, 33), 1, 0), (31, (40, 40, 40), 2, 0), (33, (40, 40, 40), 2, 3),
                                       (65, (17, 64, 25), 3, 0), (2049, (32, 31, 33), 8, 7), (5000, (64, 20, 41), 2, 50)])
def test_spread_chunk_matches_the_oracle(N, M, K, bad):
    rng = np.random.default_rng(N)
    L = tuple(1.07 * m for m in M)
    R = (rng.random((N, 3)) * np.asarray(L)).astype(np.float32)
    R[0], R[-1] = 0.0, np.nextafter(np.asarray(L, dtype=np.float32), np.float32(0))   # the two ends of the seam
    T = rng.integers(0, K, N).astype(np.uint8)
    skip = rng.choice(np.arange(1, N - 1), bad, replace=False) if bad else np.zeros(0, dtype=int)
    T[skip[::2]] = K
    R[skip[1::2], 1] = np.nan
    mesh = hpf.hpf_mesh_make(L, M, N)
    counts = torch.zeros((K, int(np.prod(M))), dtype=torch.int64, device="cuda")
    hpf.hpf_density_scatter(dev(R, torch.float32), dev(T, torch.uint8), mesh, K, counts)
    keep = np.setdiff1d(np.arange(N), skip)
    expect, _ = oracle.density(R[keep], T[keep], L, M, K)
    assert np.array_equal(counts_np(counts, K, M), expect)
    assert hpf.hpf_get_device_status(clear=True) == (hpf.HPF_FLAG_BAD_BEAD if bad else 0)
