"""The brick kernels (small lattices) against the marching ones, bit for bit: a
node's arithmetic does not depend on the kernel that does it, and the marches
are compared with the oracle elsewhere.  Boxes at the edges of the 16 x 4 x 4,
16 x 8 x 4 and 32 x 4 x 4 bricks, axes of one to three nodes, walls on every
axis."""
import numpy as np
import pytest

from paper_1507_07294_amd import mplb
from paper_1507_07294_amd import workloads as wl

pytestmark = pytest.mark.gpu

# nx at the brick widths and their remainders, ny and nz at 4 and 8 and theirs;
# the last four have 100 k nodes and more: 32 x 4 x 4 bricks, the 48-wide box
# 16 x 8 x 4
BOXES = [((1, 1, 1), (0, 0, 0)), ((1, 5, 2), (1, 0, 0)), ((2, 3, 9), (0, 1, 1)), ((15, 4, 4), (0, 0, 0)),
         ((16, 8, 5), (0, 0, 1)), ((17, 3, 13), (1, 1, 1)), ((33, 9, 6), (0, 1, 0)), ((31, 61, 62), (0, 0, 1)),
         ((64, 41, 43), (1, 1, 1)), ((96, 35, 34), (0, 0, 0)), ((48, 46, 49), (0, 1, 1))]


def _fields(w, precision, steps, rows, one_by_one):
    lt = mplb.from_workload(w, precision)
    lt.force_tile_rows(rows)
    for k in [1] * steps if one_by_one else [steps]:
        lt.step(k)
    out = {k: lt.read(k) for k in ("phi", "mu", "ux", "uy", "uz", "p")}
    lt.destroy()
    return out


@pytest.mark.parametrize("precision", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("kind", ["coupled", "unit", "q19", "field", "zalesak", "deformation"])
def test_bricks_equal_the_march(kind, precision):
    for i, (shape, bc) in enumerate(BOXES):
        coupled = kind in ("coupled", "unit", "q19")
        w = wl.perturbed_case(shape, bc, 40 + i, coupled=coupled, sigma=1e-3)
        if kind == "unit":
            w.params = w.params.replace(lambda_g=(1.0,) * 15)
        w.nse_q = 19 if kind == "q19" else 15
        if not coupled:
            w.velocity = {"kind": kind, "U": 0.02, "T": 3.0, "field": w.u0}
        bricks = _fields(w, precision, 5, 0, False)
        march = _fields(w, precision, 5, 8, True)
        for k in march:
            assert np.array_equal(bricks[k], march[k], equal_nan=True), (kind, precision, shape, bc, k)


@pytest.mark.parametrize("precision", ["f64", "f32", "f16"])
def test_small_batches_equal_their_lattices_alone(precision):
    """A batch that steps in bricks (narrow, and larger from 100 k nodes), with
    and without walls, both collision forms, odd and even step counts."""
    for unit in (False, True):
        for boxes in (BOXES[:7], BOXES[7:], BOXES[10:], [b for b in BOXES if b[1] == (0, 0, 0)]):
            ws = [wl.perturbed_case(s, bc, 70 + i, sigma=1e-3) for i, (s, bc) in enumerate(boxes)]
            if unit:
                for w in ws:
                    w.params = w.params.replace(lambda_g=(1.0,) * 15)
            batch = [mplb.from_workload(w, precision) for w in ws]
            mplb.mplb_step_many(batch, 3)
            mplb.mplb_step_many_noalloc(batch, 2)
            for w, b in zip(ws, batch):
                alone = _fields(w, precision, 5, 8, False)
                for k in alone:
                    assert np.array_equal(b.read(k), alone[k], equal_nan=True), (precision, unit, w.shape, w.bc, k)
                b.destroy()


def _droplet(shape, seed, bc=(0, 0, 0)):
    w = wl.static_droplet(n=8)
    w.shape, w.bc = shape, bc
    w.phi0 = wl.droplet_phi(*shape, 0.25 * min(shape) + seed, 4.0)
    return w


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("precision,steps", [("f32", 9), ("f16", 33), ("f64", 8)])
def test_batches_in_groups_equal_their_lattices_alone(precision, steps, noalloc):
    """Batches too large for the cache, whose lattices step in several groups:
    brick groups that fill up, lattices too large for bricks (one, which steps
    alone, and three, which march together), small ones between them."""
    big = (136, 130, 100)
    for sizes in ([(96, 96, 96), (33, 20, 17), (96, 96, 90), big, (20, 9, 40), (96, 40, 64)],
                  [big, (33, 20, 17), big, (96, 96, 96), (64, 64, 64), big]):
        ws = [_droplet(s, i, (0, 0, i % 2)) for i, s in enumerate(sizes)]
        batch = [mplb.from_workload(w, precision) for w in ws]
        (mplb.mplb_step_many_noalloc if noalloc else mplb.mplb_step_many)(batch, steps)
        for w, b in zip(ws, batch):
            lt = mplb.from_workload(w, precision)
            lt.step(steps)
            assert b.step_count == lt.step_count == steps
            for k in ("phi", "uz"):
                assert np.array_equal(b.read(k), lt.read(k)), (precision, w.shape, k)
            lt.destroy()
            b.destroy()


@pytest.mark.parametrize("precision", ["f64", "f32", "bf16"])
def test_flat_lattices_equal_the_march(precision):
    """Lattices of few layers on both sides of the limit from which they march,
    alone and with a cube in a batch."""
    for shape, count in (((256, 250, 1), 1), ((512, 510, 1), 1), ((130, 128, 5), 2), ((130, 128, 5), 9)):
        ws = [_droplet(shape, i, (0, 0, i % 2)) for i in range(count)] + [_droplet((40, 40, 40), 1)]
        batch = [mplb.from_workload(w, precision) for w in ws]
        mplb.mplb_step_many(batch, 9)
        for w, b in zip(ws, batch):
            for rows in (0, 8):
                alone = _fields(w, precision, 9, rows, False)
                for k in alone:
                    assert np.array_equal(b.read(k), alone[k], equal_nan=True), (precision, w.shape, count, rows, k)
            b.destroy()
