"""Which kernel a step takes (mplb_step_shape, a host computation from the rules
that the launches follow: no GPU needed).  The kernels give the same bits, so a
rule that moved would show in no comparison of fields; these tests hold both
sides of each line, and that the boxes of the bitwise tests still lie on the
side that those tests are named for."""
import numpy as np
import pytest

import test_gpu_bricks as bricks
import test_gpu_che_pairs as pairs
from paper_1507_07294_amd import mplb

P = mplb.PRECISIONS
COUPLED, CHE, Q19 = mplb.MPLB_COUPLED, mplb.MPLB_CHE_ONLY, mplb.MPLB_COUPLED_Q19
NARROW, MID, WIDE, PAIR = 4, 5, 6, 7


def kind(dims, prec, mode=COUPLED, nsteps=1, bc=(0, 0, 0), **kw):
    return mplb.mplb_step_shape(*dims, bc, P[prec], mode, nsteps=nsteps, **kw)["kind"]


@pytest.mark.parametrize("dims,prec,mode,want", [
    # below 100 k nodes, from there on, and FP64 coupled
    ((32, 32, 32), "f32", COUPLED, NARROW), ((64, 64, 64), "f32", COUPLED, WIDE), ((72, 72, 72), "f64", COUPLED, NARROW),
    ((64, 64, 64), "f64", CHE, WIDE),
    # wide bricks that cover 1.33 times the nodes of mid ones
    ((48, 48, 192), "f32", COUPLED, MID), ((48, 48, 192), "bf16", COUPLED, MID),
    # 285 MB a step (coupled FP32 200 B per node), FP64 CHE-only 240 MB
    ((112, 112, 112), "f32", COUPLED, WIDE), ((128, 128, 88), "f32", COUPLED, 0), ((64, 64, 256), "f32", Q19, WIDE),
    ((100, 100, 100), "f64", CHE, WIDE), ((128, 128, 128), "f64", CHE, 2),
    # 16-bit populations: full marching tiles from 1.2 M nodes on
    ((64, 64, 292), "f16", COUPLED, WIDE), ((64, 64, 293), "f16", COUPLED, 0),
    # CHE-only: 64 B per node in FP32, 40 with 16-bit populations
    ((128, 128, 271), "f32", CHE, WIDE), ((128, 128, 272), "f32", CHE, 2), ((192, 192, 192), "f16", CHE, WIDE),
    ((200, 200, 200), "f16", CHE, 3),
    # flat: idle work of bricks up to 1 M nodes
    ((256, 256, 1), "f32", COUPLED, NARROW), ((512, 512, 1), "f32", COUPLED, 0),
])
def test_bricks(dims, prec, mode, want):
    assert kind(dims, prec, mode) == want


def test_pairs():
    big = (256, 256, 256)
    for prec in ("f32", "f16", "bf16"):
        for velocity in ("zero", "zalesak", "deformation"):
            assert kind(big, prec, CHE, 4, velocity=velocity) == PAIR
            assert kind(big, prec, CHE, 3, velocity=velocity) == 3
        assert kind(big, prec, CHE, 4, velocity="field") == 3
        assert kind(big, prec, CHE, 4, rows=8) == 2
        for a in range(3):
            assert kind(big, prec, CHE, 4, bc=tuple(int(a == b) for b in range(3))) == 3
    assert kind(big, "f64", CHE, 4) == 2 and kind(big, "f32", CHE, 4, study=1) == 3
    assert kind((128, 128, 128), "f32", CHE, 4) == WIDE  # bricks come first
    # tiles that leave half idle (FP32) or 30 % (16-bit populations)
    assert kind((1024, 1024, 8), "f32", CHE, 4) == PAIR and kind((1024, 1024, 8), "f16", CHE, 4) == 3
    assert kind((1000, 1000, 6), "f32", CHE, 4) == 3 and kind((200, 200, 200), "f16", CHE, 4) == 3


def test_the_split_of_a_pair():
    """The cheapest of all splits, found without trying all of a long column's."""
    import time
    rng = np.random.default_rng(5)
    checked = 0
    while checked < 150:
        dims = tuple(int(v) for v in np.exp(rng.uniform(0, np.log(3000), 3)).astype(int) + 1)
        if not 5e6 < np.prod(dims, dtype=float) < 5e8:
            continue
        s = mplb.mplb_step_shape(*dims, (0, 0, 0), P["f32"], CHE, nsteps=4)
        if s["kind"] != PAIR:
            continue
        nz, cols, best = dims[2], -(-dims[0] // 64) * -(-dims[1] // 16), None
        for want in range(1, max(1, nz // 15) + 1):
            lz = -(-nz // want)
            nseg = -(-nz // lz)
            if (want > 1 and lz < 16) or nz - (nseg - 1) * lz < 2:
                continue
            cost = -(-cols * nseg // 256) * (lz + 6)
            if best is None or cost < best[0]:
                best = (cost, lz, nseg)
        assert (s["lz"], s["segments"]) == best[1:], (dims, s, best)
        checked += 1
    t0 = time.perf_counter()
    kind((1, 1, 1 << 30), "f32", CHE, 4), kind((1, 16, 60000000), "f32", CHE, 4)
    assert time.perf_counter() - t0 < 0.15  # 0.4 s with every split


def test_a_march_is_the_one_that_the_launch_shape_names():
    rng = np.random.default_rng(7)
    seen = set()
    for _ in range(2000):
        dims = tuple(int(v) for v in np.exp(rng.uniform(0, np.log(600), 3)).astype(int) + 1)
        prec = ("f64", "f32", "f16", "bf16")[int(rng.integers(0, 4))]
        mode = (COUPLED, CHE, Q19)[int(rng.integers(0, 3))]
        bc = tuple(int(v) for v in rng.integers(0, 2, 3))
        s = mplb.mplb_step_shape(*dims, bc, P[prec], mode, nsteps=int(rng.integers(1, 9)))
        seen.add(s["kind"])
        tw, th = s["tile"]
        assert s["blocks"] == -(-dims[0] // tw) * -(-dims[1] // th) * s["segments"]
        assert s["segments"] * s["lz"] >= dims[2] > (s["segments"] - 1) * s["lz"]
        if s["kind"] < NARROW:
            assert s == mplb.mplb_launch_shape(*dims, P[prec], mode)
        for rows in (8, 16):
            if rows == 16 and (prec == "f64" if mode == CHE else prec != "f32"):
                continue
            assert mplb.mplb_step_shape(*dims, bc, P[prec], mode, rows=rows, nsteps=4) == mplb.mplb_launch_shape(
                *dims, P[prec], mode, rows)
        if prec in ("f64", "f32"):  # a study switch
            assert mplb.mplb_step_shape(*dims, bc, P[prec], mode, study=1)["kind"] < NARROW
    assert {0, 2, 3, NARROW, MID, WIDE} <= seen, seen


def test_refusals():
    for args, kw in ((((0, 4, 4), (0, 0, 0), 1, 0), {}), (((4, 4, 4), (0, 0, 2), 1, 0), {}),
                     (((4, 4, 4), (0, 0, 0), 9, 0), {}), (((4, 4, 4), (0, 0, 0), 1, 0), {"rows": 12}),
                     (((4, 4, 4), (0, 0, 0), 0, 0), {"rows": 16}), (((4, 4, 4), (0, 0, 0), 1, 0), {"nsteps": 0}),
                     (((4, 4, 4), (0, 0, 0), 1, 0), {"study": 4})):
        dims, bc, prec, mode = args
        with pytest.raises(mplb.MplbError):
            mplb.mplb_step_shape(*dims, bc, prec, mode, **kw)


def test_the_boxes_of_the_bitwise_tests():
    kinds = {p: [kind(s, p, COUPLED, bc=bc) for s, bc in bricks.BOXES] for p in ("f64", "f32", "f16", "bf16")}
    assert set(kinds["f64"]) == {NARROW}
    for p in ("f32", "f16", "bf16"):
        assert set(kinds[p][:7]) == {NARROW} and kinds[p][10] == MID and WIDE in kinds[p][7:10], (p, kinds[p])
    for mode, p in ((CHE, "f64"), (CHE, "f32"), (CHE, "f16"), (Q19, "f32")):
        assert all(k >= NARROW for k in [kind(s, p, mode, 5, bc=bc) for s, bc in bricks.BOXES])
    for p, boxes in pairs.BOXES.items():
        assert [kind(s, p, CHE, 4) for s in boxes] == [PAIR] * len(boxes), p


def test_fp64_coupled_bricks_are_built_in_the_one_size_they_step_in():
    """FP64 coupled lattices take 16 x 4 x 4 bricks at every size, so the library
    carries no other coupled FP64 brick kernel."""
    import re
    import subprocess
    out = subprocess.run(["nm", "-C", mplb.LIB_PATH], capture_output=True, text=True, check=True).stdout
    built = {(m[1], m[2]) for m in re.finditer(r"__device_stub__(k_brick|k_brick_many)<0, [^>]*?(\d+, \d+, \d+)>", out)}
    assert built == {("k_brick", "16, 4, 4"), ("k_brick_many", "16, 4, 4")}
    rng = np.random.default_rng(11)
    for _ in range(500):
        dims = tuple(int(v) for v in np.exp(rng.uniform(0, np.log(100), 3)).astype(int) + 1)
        for mode in (COUPLED, Q19):
            assert kind(dims, "f64", mode) in (0, NARROW)
