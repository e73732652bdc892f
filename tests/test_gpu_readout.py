"""Read-outs through the pinned staging: sizes around its chunk and thread
thresholds, several threads at once on streams of their own, and the field
kernels against the totals and against a checkpoint."""
import threading

import numpy as np
import pytest

from paper_1507_07294_amd import mplb
from paper_1507_07294_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _lattice(shape, precision="f64", seed=3, mode=mplb.MPLB_CHE_ONLY):
    phi = np.random.default_rng(seed).uniform(-1, 1, shape[::-1])
    lt = mplb.Lattice(shape, (0, 0, 0), precision, mode, wl.static_droplet(n=8).params)
    if mode == mplb.MPLB_CHE_ONLY:
        lt.set_velocity("zero")
    lt.init(phi)
    return lt, phi


# 8 bytes a node: one node, just under and over 1 MiB chunks, 6 MiB (threads)
# and several rounds of the eight 4 MiB slots
@pytest.mark.parametrize("shape", [(1, 1, 1), (131071, 1, 1), (64, 64, 32), (131, 1001, 1), (1024, 768, 1),
                                   (1023, 769, 1), (1024, 769, 1), (257, 129, 300)])
def test_read_returns_every_node(shape):
    """At step 0 phi is the sum of the seven f^eq, phi itself up to its rounding
    (the terms of mu cancel); the same values come out of a checkpoint."""
    lt, phi = _lattice(shape)
    got = lt.read("phi")
    assert np.abs(got - phi).max() < 1e-14 * 64
    assert np.array_equal(lt.read("phi"), got)
    p = lt._params
    assert np.array_equal(lt.read("rho"), (1 + got) / 2 * p.rho_l + (1 - got) / 2 * p.rho_g) or np.allclose(
        lt.read("rho"), (1 + got) / 2 * p.rho_l + (1 - got) / 2 * p.rho_g, rtol=1e-15, atol=0)
    other, _ = _lattice(shape, seed=4)
    other.restore(lt.checkpoint())
    assert np.array_equal(other.read("phi"), got)
    assert abs(lt.totals()[0] - got.sum()) < 1e-12 * got.size
    lt.destroy()
    other.destroy()


def test_mu_and_front_of_a_layer():
    """mu through its own kernel is mu of the momentum balance's macro kernel
    (FP64 against the FP32 of the same box within FP32 rounding), and the front
    of a tilted layer is found whatever run of layers it falls in."""
    w = wl.rayleigh_taylor(W=16, Re=64.0, sigma=1e-2)
    fine, coarse = mplb.from_workload(w, "f64"), mplb.from_workload(w, "f32")
    # |delta mu| <= 2 [(8 beta + 12 kappa) |delta phi| + eps (12 beta + 12 kappa)], |delta phi| <= 8 eps
    eps, beta, kappa = 2.0 ** -24, 3 * 1e-2 / 16, 3 * 4 * 1e-2 / 8
    bound = 2 * ((8 * beta + 12 * kappa) * 8 * eps + eps * (12 * beta + 12 * kappa))
    assert np.abs(fine.read("mu") - coarse.read("mu")).max() < bound
    phi = fine.read("phi")
    a, b = phi[:-1], phi[1:]
    cross = (a < 0) != (b < 0)
    z = (np.arange(phi.shape[0] - 1)[:, None, None] + 0.5 + a / np.where(cross, a - b, 1.0))[cross]
    assert np.allclose(fine.front(), [z.min(), z.max()], rtol=1e-14, atol=0)
    for k in (0, 14, 15, 16, 17, 31, 32, 46):  # one crossing, between layers k and k + 1
        lt, _ = _lattice((3, 2, 48), mode=mplb.MPLB_COUPLED)
        phi0 = np.where(np.arange(48) <= k, -0.5, 0.5)[:, None, None] * np.ones((48, 2, 3))
        lt.init(phi0)
        assert np.allclose(lt.front(), [k + 1.0, k + 1.0], atol=1e-12), k
        lt.destroy()
    fine.destroy()
    coarse.destroy()


def test_reads_from_several_threads():
    """More threads than staging buffers, each with its own lattice and stream."""
    import torch
    made = [_lattice((200, 200, 30), seed=10 + i) for i in range(6)]
    streams = [torch.cuda.Stream() for _ in made]
    torch.cuda.synchronize()
    for (lt, _), s in zip(made, streams):
        lt.set_stream(s.cuda_stream)
    wrong = []

    def reader(i):
        lt, phi = made[i]
        for _ in range(5):
            if np.abs(lt.read("phi") - phi).max() > 1e-12:
                wrong.append(i)

    threads = [threading.Thread(target=reader, args=(i,)) for i in range(len(made))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    for lt, _ in made:
        lt.destroy()
