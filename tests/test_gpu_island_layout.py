"""GPU parity of the layout of the touching islands: more touching pairs and
more particles touching a wall than compute units (several to a workgroup, the
last one partly filled), islands of three, a pair beside free particles, for
every contact law and both island set-ups, against the FP64 oracle.

Bounds of the other contact tests: particle positions (against the largest
displacement), velocities and spins 1e-5 relative.
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


def _touching(D, pairs, walls, triples):
    """Pairs one above the other, singles on the floor and rows of three, on a
    grid far enough apart to be islands of their own; all closing in."""
    nx = 128 if D == 2 else 28
    n = (nx, 80, 1) if D == 2 else (nx, nx, 24)
    rng = np.random.default_rng(5)
    X, U = [], []
    per = (nx - 6) // 2

    def base(i):
        if D == 2:
            return np.array([3.0 + 2.0 * (i % per), 3.0 + 2.5 * (i // per)])
        return np.array([3.0 + 2.0 * (i % per), 3.0 + 2.0 * ((i // per) % per), 3.0 + 2.5 * (i // (per * per))])

    up = np.eye(D)[D - 1]
    for i in range(pairs + triples):
        k = 2 if i < pairs else 3
        for m in range(k):
            X.append(base(i) + up * 0.4999 * m)
            U.append(1e-4 * rng.standard_normal(D) - up * 5e-4 * m)
    for i in range(walls):
        p = np.array([1.0 + (nx - 2.0) * i / walls, 0.0] if D == 2 else
                     [1.5 + 1.5 * (i % 17), 1.5 + 1.5 * (i // 17), 0.0])
        p[D - 1] = 0.2 - 1e-5
        X.append(p)
        U.append(1e-4 * rng.standard_normal(D))
    X = np.array(X).T.astype(np.float32).astype(np.float64)
    U = np.array(U).T.astype(np.float32).astype(np.float64)
    d = np.full(X.shape[1], 0.5)
    d[len(d) - walls:] = np.float32(0.4)      # the value both sides hold
    return n, X, U, d


@pytest.mark.parametrize("setup", [1, 2])
@pytest.mark.parametrize("lat,contact", [(9, "lsd"), (9, "hertz"), (9, "hertz_mindlin"), (19, "lsd"), (19, "hertz"),
                                         (19, "hertz_mindlin"), (19, "hertz_mindlin_microslip")])
def test_touching_islands_match_oracle(P, orc, lat, contact, setup):
    print(f"touching islands {lat} {contact} {setup}", flush=True)
    D = 2 if lat == 9 else 3
    # the walls' row of 2D holds about 120 singles 1 apart
    pairs, walls, triples = 300, (100 if D == 2 else 270), 20
    n, X, U, d = _touching(D, pairs, walls, triples)
    rp = np.full(X.shape[1], 2.5)
    g = [0.0, 0.0, 0.0]
    g[D - 1] = -1e-5
    cfg = P.make_config(lattice=lat, n=n, tau=0.8, gravity=g, n_sub=200, contact=contact, young=1e3,
                        island_setup=setup)
    sim = P.Sim(cfg, X.shape[1])
    sim.set_particles(X, U, d, rp)
    oc = G.oracle_cfg(orc, cfg)
    f = G.to_oracle_f(orc, lat, sim.read_populations())
    mindlin = contact.startswith("hertz_mindlin")
    Xo, Uo, Wo, hist = X.copy(), U.copy(), np.zeros((3, X.shape[1])), None
    for _ in range(2):
        out = orc.step_hm(oc, f, Xo, Uo, Wo, d, rp, hist) if mindlin else orc.step(oc, f, Xo, Uo, d, rp)
        f, Xo, Uo = out["f"], out["X"], out["U"]
        if mindlin:
            Wo, hist = out["W"], out["hist"]
    sim.step(1)
    assert sim.diagnostics()["active"] >= 2 * pairs + 3 * triples + walls
    sim.step(1)
    sim.synchronize()
    got = sim.read_particles()
    ex = np.abs(got["x"] - Xo).max() / np.abs(Xo - X).max()
    ev = np.linalg.norm(got["v"] - Uo) / np.linalg.norm(Uo)
    print(f"  dX={ex:.2e} dU={ev:.2e}", flush=True)
    assert ex <= 1e-5 and ev <= 1e-5
    if mindlin:
        w = sim.read_rotation()
        ref = Wo if D == 3 else Wo[2:3]
        assert np.linalg.norm(w - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("lat", [9, 19])
@pytest.mark.parametrize("lasting,closing,walls", [(1, 0, 0), (8, 1, 1), (9, 257, 3), (20, 7, 0)])
def test_lasting_and_closing_pairs_match_oracle(P, orc, lat, lasting, closing, walls):
    """Spring-dashpot pairs that overlap and move together (laid out eight to
    a workgroup) beside pairs that close in (one to a workgroup, two above
    256) and particles at a wall; the same bits by both island set-ups."""
    print(f"lasting and closing pairs {lat} {lasting} {closing} {walls}", flush=True)
    D = 2 if lat == 9 else 3
    n, X, U, d = _touching(D, lasting + closing, max(walls, 1), 0)
    if walls == 0:
        X, U, d = X[:, :-1], U[:, :-1], d[:-1]
    U[:, 1:2 * lasting:2] = U[:, 0:2 * lasting:2]
    rp = np.full(X.shape[1], 2.5)
    g = [0.0, 0.0, 0.0]
    g[D - 1] = -1e-5
    got = []
    for setup in (1, 2):
        cfg = P.make_config(lattice=lat, n=n, tau=0.8, gravity=g, n_sub=100, contact="lsd", island_setup=setup)
        sim = P.Sim(cfg, X.shape[1])
        sim.set_particles(X, U, d, rp)
        f = G.to_oracle_f(orc, lat, sim.read_populations())
        sim.step(1)
        sim.synchronize()
        got.append(sim.read_particles())
    out = orc.step(G.oracle_cfg(orc, cfg), f, X, U, d, rp)
    ex = np.abs(got[0]["x"] - out["X"]).max() / np.abs(out["X"] - X).max()
    ev = np.linalg.norm(got[0]["v"] - out["U"]) / np.linalg.norm(out["U"])
    print(f"  {X.shape[1]} particles dX={ex:.2e} dU={ev:.2e}", flush=True)
    assert ex <= 1e-5 and ev <= 1e-5
    for k in ("x", "v", "f_hydro", "f_contact"):
        assert np.array_equal(got[0][k], got[1][k]), k
