"""GPU: what HpfState.step keeps between steps besides the beads -- the streams it enqueues on and
its mesh counts -- in the states that a program can leave it in."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1310_2041_amd import engine, hpf  # noqa: E402
from synth import workloads as wl  # noqa: E402


def _states(n=2, **kw):
    s = wl.small_system(300, 10, (15.0, 17.5, 16.1), (15, 17, 16), seed=3, n_solvent=700)
    out = []
    for _ in range(n):
        st = engine.HpfState.from_system(s, **kw)
        st.start(sort=True)
        out.append(st)
    return out


def _assert_same(a, b):
    torch.cuda.synchronize()
    for x, y in zip(a.host_beads(), b.host_beads()):
        assert np.array_equal(x, y)


def test_stream_handle_zero_is_the_default_stream():
    side = torch.cuda.Stream()
    with torch.cuda.stream(side), engine._on(0):
        assert torch.cuda.current_stream().cuda_stream == 0
    with engine._on(side.cuda_stream):
        assert torch.cuda.current_stream().cuda_stream == side.cuda_stream
    a, b = _states()
    for st in (a, b):
        st.set_thermostat(5.0, seed=4)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        a.run(6, sort_every=4, stream=0)
    b.run(6, sort_every=4)
    _assert_same(a, b)


@pytest.mark.parametrize("left_by", ["scatter", "prime"])
def test_step_leaves_no_counts_behind(left_by):
    """Counts that a density read-out or a deposit never finished left in the buffer are gone
    after a step that rebuilds the field, so that a depositing pass may follow."""
    a, b = _states()
    if left_by == "scatter":
        a.scatter()
        assert not a.counts_clear and bool(a.counts.any())
    else:
        for st in (a, b):                          # strays: the halo is one cell, the beads move eight
            st.prime()
            st.Vel *= 200.0
            st.step_fused()
        assert bool(a.counts.any())
        for st in (a, b):
            st.density_pending = False
            st.Vel *= 0.005
        b.rebuild()
    a.step(report=True)
    b.step(report=True)
    assert not bool(a.counts.any()) and a.counts_clear
    for st in (a, b):
        st.prime()
        st.advance()                               # deposits, from the last gradient
        st.step_fused(report=True)
        st.run(2)
    _assert_same(a, b)
    assert a.energies()["W"] == b.energies()["W"]


def test_deposit_after_replayed_steps_and_a_read_out():
    a, b = _states()
    for st in (a, b):
        st.step()                                  # the strays' buffer is there before the capture
    torch.cuda.synchronize()
    g = engine.Graph(lambda: [a.step() for _ in range(2)])
    a.scatter()
    g.launch(torch.cuda.current_stream())
    b.step()
    b.step()
    for st in (a, b):
        st.prime()
        st.advance()                               # deposits, from the last gradient
        st.step_fused(report=True)
    _assert_same(a, b)
    assert a.energies()["W"] == b.energies()["W"]


def test_step_goes_on_without_memory_for_its_strays(monkeypatch):
    a, b = _states()
    tried = []

    def no_memory(*args, **kw):
        tried.append(args)
        raise torch.OutOfMemoryError("no memory")

    with monkeypatch.context() as m:
        m.setattr(engine.torch, "zeros", no_memory)
        a.run(5, sort_every=3)
    b.run(5, sort_every=3)
    assert len(tried) == 1 and a.strays is None and b.strays is not None
    _assert_same(a, b)


def test_step_after_one_that_was_broken_off(monkeypatch):
    """The calls of a step raise after its deposit; the program starts again from the positions
    it is left with, as it could when a step's scatter overwrote what an earlier one had left."""
    a, b = _states()
    for st in (a, b):
        st.run(3, sort_every=0)
        st.Vel *= 200.0                            # strays: the halo is one cell, the beads move eight
    with monkeypatch.context() as m:
        def broken(*args, **kw):
            raise RuntimeError("broken off")

        m.setattr(hpf, "hpf_field_potential_cells", broken)
        with pytest.raises(RuntimeError, match="broken off"):
            a.step()
    assert bool(a.strays.any())
    hpf.verlet_step(b.R, b.Vel, b.F, b.dt, b.box, 1)
    for st in (a, b):
        st.Vel *= 0.005
        st.start(sort=False)
        st.run(4, sort_every=0)
    assert not bool(a.strays.any())
    _assert_same(a, b)
