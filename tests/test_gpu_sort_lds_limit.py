"""GPU: batches whose key totals (bricks + 1 of every replica) are the last and the first that
four and two slot rows fit a CU's LDS at -- 10,239 to 10,241 and 20,479 to 20,481 -- step as
their replicas do alone, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1310_2041_amd import engine, hpf  # noqa: E402
from synth import workloads as wl  # noqa: E402

# meshes of 4096, 256, 9 and 13 keys (bricks of 8 cells + 1), and how many of each
BIG, MID, EIGHT, NINE = (104, 120, 168), (24, 40, 136), (16, 16, 16), (16, 16, 24)
TOTALS = {10239: [(MID, 39), (EIGHT, 11), (NINE, 12)],
          10240: [((24, 24, 56), 160)],
          10241: [(MID, 39), (EIGHT, 4), (NINE, 17)],
          20479: [(BIG, 4), (MID, 15), (EIGHT, 11), (NINE, 12)],
          20480: [(BIG, 5)],
          20481: [(BIG, 4), (MID, 15), (EIGHT, 4), (NINE, 17)]}


@pytest.mark.parametrize("total", TOTALS)
def test_batch_with_a_key_total_at_the_lds_limit(total):
    systems = [wl.small_system(7 + i % 5, 10, tuple(1.07 * m for m in M), M, seed=i)
               for i, M in enumerate(M for M, n in TOTALS[total] for _ in range(n))]
    assert sum(1 + int(np.prod([-(-m // 8) for m in s.M])) for s in systems) == total
    hpf.hpf_get_device_status(clear=True)
    b = engine.BatchState(systems, sort_every=3, brick=8)
    b.start()
    b.step(7)
    first = {tuple(s.M): r for r, s in reversed(list(enumerate(systems)))}
    for r in sorted({*first.values(), len(systems) // 2, len(systems) - 1}):
        st = engine.HpfState.from_system(systems[r], sort_brick=8)
        st.start(sort=True)
        st.prime()
        st.run_fused(7, sort_every=3)
        for x, y in zip(b.replica_beads(r), st.host_beads()):
            assert np.array_equal(x, y), f"replica {r}"
    assert hpf.hpf_get_device_status(clear=True) == 0
