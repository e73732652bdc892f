"""Two CHE-only steps per launch (large periodic lattices, four steps or more at
a time) against single steps of the marching kernels, bit for bit: populations,
history and fields do not depend on the split, and the marches are compared
with the oracle elsewhere."""
import numpy as np
import pytest

from paper_1507_07294_amd import mplb
from paper_1507_07294_amd import workloads as wl

pytestmark = pytest.mark.gpu

# Beyond the bricks' 4.45 M nodes (FP32) and 7.12 M (16-bit populations): ragged
# tiles, full ones, a single segment of few planes, x axes of one and two nodes
# under a frame of three, last segments of two planes and where an even split
# would leave one.
BOXES = {"f32": [(170, 163, 165), (64, 272, 260), (600, 700, 11), (1, 2200, 2100), (2, 1500, 1520),
                 (64, 64, 1100), (64, 64, 1261)],
         "f16": [(193, 190, 197), (2, 1900, 1900), (66, 340, 330)],
         "bf16": [(193, 190, 197), (130, 131, 430)]}


def _workload(shape, kind, seed):
    """Random phi, so that no two nodes agree, in the interval that it stays in."""
    w = wl.deformation_flow(n=16)
    w.shape = shape
    w.phi0 = np.random.default_rng(seed).uniform(-0.5, 0.5, shape[::-1])
    # (the rotation's speed grows with the distance over nx)
    w.velocity = {"kind": kind, "U": 0.02 * min(1.0, 2.0 * shape[0] / max(shape[1:])), "T": 3.0}
    return w


def _state(lt):
    return {"phi": lt.read("phi"), "mu": lt.read("mu"), "uz": lt.read("uz")}


def _same(a, b, what):
    for k in a:
        assert np.array_equal(a[k], b[k]), (what, k, int((a[k] != b[k]).sum()))


@pytest.mark.parametrize("precision,i", [(p, i) for p in BOXES for i in range(len(BOXES[p]))])
def test_pairs_equal_single_steps(precision, i):
    shape = BOXES[precision][i]
    kind = ("deformation", "zalesak", "zero")[i % 3]
    w = _workload(shape, kind, 7 * i)
    lt, one = mplb.from_workload(w, precision), mplb.from_workload(w, precision)
    one.force_tile_rows(8)
    lt.poison()
    lt.step(6)
    one.step(6)
    _same(_state(lt), _state(one), (shape, kind))
    lt.step(1)  # the history that the pairs left
    lt.step(5)
    one.step(6)
    assert lt.step_count == one.step_count == 12
    _same(_state(lt), _state(one), (shape, kind, "again"))
    assert np.array_equal(lt.totals(), one.totals())
    lt.destroy()
    one.destroy()


def test_pairs_between_checks_batches_and_restores():
    """Checks at odd intervals, a batch, and a checkpoint taken between pairs."""
    w = _workload((170, 163, 165), "deformation", 3)
    one = mplb.from_workload(w, "f32")
    one.force_tile_rows(8)
    one.step(23)
    lt = mplb.from_workload(w, "f32")
    lt.set_check_interval(7)
    lt.step(4)
    saved = lt.checkpoint()
    lt.step(19)
    _same(_state(lt), _state(one), "checks")
    back = mplb.from_workload(w, "f32")
    back.restore(saved)
    small = mplb.from_workload(wl.deformation_flow(n=16), "f32")
    mplb.mplb_step_many([back, small], 19)
    assert back.step_count == 23
    _same(_state(back), _state(one), "restored, in a batch")
    for x in (one, lt, back, small):
        x.destroy()


def test_a_pair_reports_the_non_finite():
    w = _workload((170, 163, 165), "zalesak", 4)
    lt = mplb.from_workload(w, "f32")
    lt.set_check_interval(4)
    lt.step(8)
    lt.poke(0, 3, lt.N - 1, float("nan"))
    rc, msg = lt.try_step(8)
    assert rc == mplb.MPLB_E_NONFINITE and "after step 12" in msg
    lt.destroy()


def test_captured_steps_replay_as_the_program_goes_on():
    """Two steps and four, captured into graphs and replayed between eager ones
    (the velocity does not depend on time): each finds the state where it lay."""
    import torch

    w = _workload((170, 163, 165), "zalesak", 5)
    stream = torch.cuda.Stream()
    lt = mplb.from_workload(w, "f32")
    lt.set_stream(stream.cuda_stream)
    lt.set_check_interval(0)
    lt.step(5)
    one = mplb.from_workload(w, "f32")
    one.force_tile_rows(8)
    one.step(5)
    graphs = {}
    for n in (2, 4):
        graphs[n] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graphs[n], stream=stream):
            lt.step(n)
    for n in (4, 2, 4, 2, 2):
        with torch.cuda.stream(stream):
            graphs[n].replay()
        lt.step(4)
        lt.step(2)
        stream.synchronize()
        one.step(n + 6)
        assert np.array_equal(lt.read("phi"), one.read("phi")), n
    lt.destroy()
    one.destroy()
