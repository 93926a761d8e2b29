"""GPU parity of the 3D gathers of more particles than one lane per support node
is used for (640 to 1024, by the lattice's size), beside the small cases of
the other files: the moments pass on the node rows that the stencils reach,
tiles with bins of one and two dual cells, and the gather of one particle by a
group of lanes with bins of four; delta and Lagrange weights, on odd extents
and with particles on the band's edges, against the FP64 oracle; and the same
bits for the same particles by lanes per node and by tiles.

Bounds: those of the free-particle tests (fields 1e-5 and 1e-6, 1e-3 and 1e-5
with 16-bit storage; velocities and displacements 1e-5).
"""
import numpy as np
import pytest

from tests import gpu_helpers as G
from tests.test_gpu_parity import _coupled_compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1407_6704_amd import pibm
    pibm.load()
    return pibm


def _spread_out(rng, lo, hi, np_, clear, edges):
    """np_ points of the box [lo, hi], `clear` apart from each other (a jittered grid, in random order); the first
    ones are moved to the band's edges along y and z."""
    pitch = clear + 0.12
    ax = [np.arange(lo[a] + 0.06, hi[a] - 0.06, pitch) for a in range(3)]
    p = np.stack(np.meshgrid(*ax, indexing="ij")).reshape(3, -1)
    assert p.shape[1] >= np_
    p = p[:, rng.permutation(p.shape[1])[:np_]] + rng.uniform(-0.05, 0.05, (3, np_))
    for a in (1, 2):
        for side, value in ((p[a] < ax[a][0] + 0.06, lo[a]), (p[a] > ax[a][-1] - 0.06, hi[a])):
            if edges:
                p[a, side] = value
    return p.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("lat,interp,bl,storage", [(19, "delta", 0, "fp32"), (15, "lagrange", 0, "fp32"),
                                                   (15, "delta", 1, "fp32"), (19, "lagrange", 1, "fp32"),
                                                   (15, "lagrange", 1, "fp32"), (19, "delta", 2, "fp32"),
                                                   (15, "lagrange", 2, "fp32"), (19, "lagrange", 0, "fp16")])
def test_gather_of_many_in_a_band(P, orc, lat, interp, bl, storage):
    from paper_1407_6704_amd import workloads as W

    print(f"gather of many {lat} {interp} {bl} {storage}", flush=True)
    rng = np.random.default_rng(77)
    n, np_ = (201, 17, 15), 1100
    X = _spread_out(rng, (0.6, 6.0, 8.0), (200.4, 9.6, 12.0), np_, 0.62, True)
    d = rng.uniform(0.3, 0.5, np_).astype(np.float32).astype(np.float64)
    U = (1e-4 * rng.standard_normal((3, np_))).astype(np.float32).astype(np.float64)
    rp = rng.uniform(1.5, 3.0, np_).astype(np.float32).astype(np.float64)
    cfg = P.make_config(lattice=lat, n=n, tau=0.7, gravity=(0, 0, -1e-5), n_sub=200, contact="lsd", interp=interp,
                        bin_log2=bl, storage=storage)
    sim0 = P.Sim(P.make_config(lattice=lat, n=n, tau=0.7, contact="none", storage=storage), 0)
    h0 = G.perturbed_state(orc, sim0, W.C0.replace(lattice=lat, n=n), seed=9, amp=1e-4)
    r = _coupled_compare(P, orc, cfg, X, U, d, rp, h0=h0, label="1 step")
    tu, tr = (1e-5, 1e-6) if storage == "fp32" else (1e-3, 1e-5)
    assert r["eu"] <= tu and r["er"] <= tr
    # (particles move by what they gathered: the stored populations are the oracle's start in either storage)
    assert r["ex"] <= 1e-5 and r["ev"] <= 1e-5 and r["efh"] <= 1e-5


@pytest.mark.parametrize("few", [1, 639, 640])
@pytest.mark.parametrize("lat,interp", [(19, "delta"), (15, "lagrange")])
def test_same_bits_by_both_gathers(P, orc, lat, interp, few):
    from paper_1407_6704_amd import workloads as W

    print(f"both gathers {lat} {interp} {few}", flush=True)
    rng = np.random.default_rng(78)
    n, many = (41, 33, 21), 1025
    X = _spread_out(rng, (0.3, 0.3, 0.3), (40.7, 32.7, 20.7), many, 0.62, False)
    U = (1e-4 * rng.standard_normal((3, many))).astype(np.float32).astype(np.float64)
    d, rp = np.full(many, 0.4), np.full(many, 2.0)
    sim0 = P.Sim(P.make_config(lattice=lat, n=n, tau=0.7, contact="none"), 0)
    h0 = G.perturbed_state(orc, sim0, W.C0.replace(lattice=lat, n=n), seed=9, amp=1e-4)
    out = []
    for np_ in (few, many):
        sim = P.Sim(P.make_config(lattice=lat, n=n, tau=0.7, gravity=(0, 0, -1e-5), n_sub=20, contact="none",
                                  interp=interp), np_)
        sim.write_populations(h0)
        sim.set_particles(X[:, :np_], U[:, :np_], d[:np_], rp[:np_])
        sim.step(1)
        sim.synchronize()
        out.append(sim.read_particles())
    for k in ("x", "v", "f_hydro"):
        assert np.array_equal(out[0][k], out[1][k][:, :few]), k
