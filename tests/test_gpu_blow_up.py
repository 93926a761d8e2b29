"""States that the spreading meets at its limits: particles that have left the
box by far, more of them in the corner tiles than are staged in LDS, on steps
that were queued behind the one that lost them (the library reports E_UNSTABLE
or E_SKIN at the next synchronising call and goes on with new particles and
fluid); and more particles around a tile than 16 bits count, against the FP64
oracle.

Bounds: those of the free-particle tests (1e-5 for fields, velocities and
displacements).
"""
import numpy as np
import pytest

from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1407_6704_amd import pibm
    pibm.load()
    return pibm


def _works_as_before(P, orc, sim, lat, X, rng):
    """New fluid and particles on the same context: one step against the oracle."""
    D, np_ = X.shape
    U = (1e-4 * rng.standard_normal((D, np_))).astype(np.float32).astype(np.float64)
    d, rp = np.full(np_, np.float32(0.4)).astype(np.float64), np.full(np_, 2.0)
    sim.init_equilibrium()
    sim.set_particles(X, U, d, rp)
    f0 = G.to_oracle_f(orc, lat, sim.read_populations())
    out = orc.step(G.oracle_cfg(orc, sim.cfg), f0, X.copy(), U.copy(), d, rp)
    sim.step(1)
    sim.synchronize()
    got = sim.read_particles()
    eu, er, _ = G.field_errors(orc, lat, sim.read_populations(), out["f"], sim.N)
    ex = np.abs(got["x"] - out["X"]).max() / np.abs(out["X"] - X).max()
    ev = np.linalg.norm(got["v"] - out["U"]) / np.linalg.norm(out["U"])
    print(f"  afterwards eps_u={eu:.2e} eps_rho={er:.2e} dX={ex:.2e} dU={ev:.2e}", flush=True)
    assert eu <= 1e-5 and er <= 1e-6 and ex <= 1e-5 and ev <= 1e-5


@pytest.mark.parametrize("speed", [30.0, 1e4, 1e9, 3e38])
@pytest.mark.parametrize("lat,n,np_,bin_log2", [(9, (60, 50, 1), 1500, 0), (19, (20, 18, 16), 1500, 0),
                                                (15, (20, 18, 16), 900, 0), (9, (60, 50, 1), 400, 0),
                                                (19, (20, 18, 16), 1500, 2)])
def test_particles_far_outside_the_box(P, orc, lat, n, np_, bin_log2, speed):
    print(f"far outside the box {lat} {np_} {bin_log2} {speed}", flush=True)
    D = 2 if lat == 9 else 3
    rng = np.random.default_rng(3)
    X = np.stack([rng.uniform(1.0, n[a] - 1.0, np_) for a in range(D)]).astype(np.float32).astype(np.float64)
    U = speed * np.sign(rng.standard_normal((D, np_)))             # to every corner
    sim = P.Sim(P.make_config(lattice=lat, n=n, tau=0.8, n_sub=20, contact="none", bin_log2=bin_log2,
                              gravity=(0, -1e-5, 0)), np_)
    sim.set_particles(X, U, np.full(np_, 0.4), np.full(np_, 2.0))
    sim.step(4)
    with pytest.raises(P.PibmError) as e:
        sim.synchronize()
    assert e.value.name in ("E_UNSTABLE", "E_SKIN")
    _works_as_before(P, orc, sim, lat, X, rng)


@pytest.mark.parametrize("lat,n", [(9, (60, 50, 1)), (19, (20, 18, 16))])
def test_overlapping_particles_blow_up(P, orc, lat, n):
    """Spring-dashpot particles that overlap by up to their size fly apart, out of the box, and take the fluid along."""
    print(f"blow-up {lat}", flush=True)
    D, np_ = (2 if lat == 9 else 3), 1500
    rng = np.random.default_rng(5)
    X = np.stack([rng.uniform(1.0, n[a] - 1.0, np_) for a in range(D)]).astype(np.float32).astype(np.float64)
    sim = P.Sim(P.make_config(lattice=lat, n=n, tau=0.8, n_sub=100, contact="lsd", max_candidates=64), np_)
    sim.set_particles(X, None, np.full(np_, 0.5), np.full(np_, 2.5))
    sim.step(12)
    with pytest.raises(P.PibmError) as e:
        sim.synchronize()
    assert e.value.name in ("E_UNSTABLE", "E_SKIN", "E_CAPACITY")
    # apart from each other: free particles
    k = np.arange(1500)
    side = int(np.ceil(1500 ** (1 / D)))
    p = np.stack([k % side, (k // side) % side, k // side ** 2])[:D]
    X = np.stack([1.0 + p[a] * (n[a] - 2.0) / side for a in range(D)]).astype(np.float32).astype(np.float64)
    _works_as_before(P, orc, sim, lat, X, rng)


@pytest.mark.parametrize("lat", [9, 19])
def test_more_particles_around_a_tile_than_16_bits_count(P, orc, lat):
    print(f"crowded tile {lat}", flush=True)
    D, np_ = (2 if lat == 9 else 3), (70_000 if lat == 9 else 120_000)
    n = (40, 24, 1) if D == 2 else (36, 10, 9)
    rng = np.random.default_rng(4)
    X = np.stack([rng.uniform(0.3 if a else 2.0, n[a] - 0.3 if a else 30.0, np_) for a in range(D)])
    X[1] = rng.uniform(2.0, 9.0, np_)
    if D == 3:
        X[2] = rng.uniform(2.0, 7.0, np_)
    X = X.astype(np.float32).astype(np.float64)
    U = (1e-4 * rng.standard_normal((D, np_))).astype(np.float32).astype(np.float64)
    d, rp = np.full(np_, np.float32(0.02)).astype(np.float64), np.full(np_, 2.0)
    g = [0.0, 0.0, 0.0]
    g[D - 1] = -1e-5
    cfg = P.make_config(lattice=lat, n=n, tau=0.8, gravity=g, n_sub=2000, contact="none")
    sim = P.Sim(cfg, np_)
    sim.set_particles(X, U, d, rp)
    f0 = G.to_oracle_f(orc, lat, sim.read_populations())
    out = orc.step(G.oracle_cfg(orc, cfg), f0, X.copy(), U.copy(), d, rp)
    sim.step(1)
    sim.synchronize()
    got = sim.read_particles()
    eu, er, _ = G.field_errors(orc, lat, sim.read_populations(), out["f"], sim.N)
    ex = np.abs(got["x"] - out["X"]).max() / np.abs(out["X"] - X).max()
    ev = np.linalg.norm(got["v"] - out["U"]) / np.linalg.norm(out["U"])
    print(f"  eps_u={eu:.2e} eps_rho={er:.2e} dX={ex:.2e} dU={ev:.2e}", flush=True)
    assert eu <= 1e-5 and er <= 1e-6 and ex <= 1e-5 and ev <= 1e-5
