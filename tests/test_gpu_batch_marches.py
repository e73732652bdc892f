"""The batched marching kernel in every form it is built in (storage, walls on x
or y, collision form, streaming stores), against each lattice's march alone, bit
for bit; and the march on the splits that a lattice of a few hundred blocks
takes, against the oracle.  mplb_step and mplb_step_many step most lattices of
these sizes in bricks; the kinds are asserted before the steps."""
import numpy as np
import pytest

import helpers
from paper_1507_07294_amd import mplb
from paper_1507_07294_amd import workloads as wl
from test_gpu_parity import F32_TOL, _two_block_count

pytestmark = pytest.mark.gpu

FORMS = [(False, False), (False, True), (True, False), (True, True)]
FIELDS = ("phi", "mu", "ux", "uz", "p")


def _case(shape, bc, seed, unit):
    w = wl.perturbed_case(shape, bc, seed, sigma=1e-3)
    if unit:
        w.params = w.params.replace(lambda_g=(1.0,) * 15)
    return w


def _batch_equals_alone(ws, precision, steps, poison=False):
    batch = [mplb.from_workload(w, precision) for w in ws]
    assert mplb.mplb_step_many_kinds(batch, steps) == [0] * len(ws)
    for b in batch:
        if poison:
            b.poison()
    mplb.mplb_step_many(batch, steps)
    mplb.mplb_step_many_noalloc(batch, steps)
    for w, b in zip(ws, batch):
        alone = mplb.from_workload(w, precision)
        alone.force_tile_rows(8)
        alone.step(2 * steps)
        assert b.step_count == alone.step_count
        for k in FIELDS:
            assert np.array_equal(b.read(k), alone.read(k)), (precision, w.shape, w.bc, k)
        alone.destroy()
        b.destroy()


@pytest.mark.parametrize("walls,unit", FORMS)
@pytest.mark.parametrize("precision", ["f64", "f32", "f16", "bf16"])
def test_flat_batches(precision, walls, unit):
    """Many lattices of one or two layers, ragged in x and y; their LDS and
    what a step must not read start as NaN."""
    shapes = [(61, 37, 1), (64, 64, 1), (17, 40, 1), (66, 8, 1), (130, 33, 1), (48, 48, 2)] * 9
    ws = [_case(s, (i % 2, i // 2 % 2, i // 4 % 2) if walls else (0, 0, i % 2), 20 + i, unit)
          for i, s in enumerate(shapes)]
    for steps in (3, 10):
        _batch_equals_alone(ws, precision, steps, poison=True)


# nodes enough that three lattices move more than 512 MB a step
LARGE = {"f64": [(70, 81, 80), (96, 61, 77), (130, 40, 88)], "f32": [(130, 81, 85), (96, 95, 100), (70, 130, 99)],
         "f16": [(130, 121, 100), (96, 130, 125), (190, 90, 91)]}
LARGE["bf16"] = LARGE["f16"]


@pytest.mark.parametrize("walls,unit", FORMS)
@pytest.mark.parametrize("precision", ["f64", "f32", "f16", "bf16"])
def test_streaming_batches(precision, walls, unit):
    """Batches beyond the cache in calls of too few steps for groups."""
    bcs = [(1, 0, 0), (0, 1, 1), (1, 1, 1)] if walls else [(0, 0, 0), (0, 0, 1), (0, 0, 0)]
    ws = [_case(s, bc, 90 + i, unit) for i, (s, bc) in enumerate(zip(LARGE[precision], bcs))]
    per = {"f64": 400, "f32": 200}.get(precision, 116)
    assert per * sum(w.nodes for w in ws) > 512 << 20
    _batch_equals_alone(ws, precision, 3)


@pytest.mark.parametrize("dims,bc,prec,coupled", [((70, 77, 69), (0, 0, 1), "f32", True),
                                                 ((72, 72, 72), (1, 1, 1), "f16", True),
                                                 ((70, 75, 80), (0, 1, 0), "f32", False),
                                                 ((80, 80, 80), (0, 0, 0), "f16", False)])
def test_one_block_per_cu_march_matches_oracle(dims, bc, prec, coupled):
    """Lattices whose march takes one block per CU because two would load the
    CUs unevenly, marching (they would step in bricks by themselves)."""
    mode = mplb.MPLB_COUPLED if coupled else mplb.MPLB_CHE_ONLY
    shape = mplb.mplb_step_shape(*dims, bc, mplb.PRECISIONS[prec], mode, rows=8)
    assert shape["kind"] == (0 if coupled else 2) and shape["blocks"] <= 256 < _two_block_count(dims, 5), shape
    w = wl.perturbed_case(dims, bc, 77 + dims[0], coupled=coupled)
    if not coupled:
        w.velocity = {"kind": "deformation", "U": 0.02, "T": 0.05}
    o, g = helpers.oracle_for(w), helpers.gpu_for(w, prec)
    g.force_tile_rows(8)
    done = 0
    for n in (1, 6):
        o.step(n - done)
        g.step(n - done)
        done = n
        errs = helpers.rel_errors(helpers.fields_of(g, coupled), helpers.fields_of(o, coupled))
        for k, e in errs.items():
            assert e <= (F32_TOL[k] if prec == "f32" else 5e-3), (k, n, e)
    g.destroy()
