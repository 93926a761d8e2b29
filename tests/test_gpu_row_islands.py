"""GPU parity of touching islands of three and more particles without friction:
chains of 3 to 9 (up to eight run with a quad of lanes per contact where no
member has more than two candidates), triangles, a particle with four partners
(general loop), chains whose end rests on the floor, one and nine of each so
that they fill one and several workgroups' shares, for every contact law,
against the FP64 oracle.

Bounds of the other contact tests: positions (against the largest
displacement) and velocities 1e-5 relative.
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


def _shapes(D):
    s = 0.49995                                                  # of diameter 0.5: every neighbour touches
    out = [np.outer(np.arange(m) * s, [1.0, 0, 0]) for m in (3, 4, 5, 8, 9)]
    out.append(np.array([[0, 0, 0], [s, 0, 0], [0.5 * s, s * np.sqrt(0.75), 0]]))
    out.append(np.array([[0, 0, 0], [s, 0, 0], [-s, 0, 0], [0, s, 0], [0, -s, 0]]))
    return [o[:, :D] for o in out]


@pytest.mark.parametrize("setup", [1, 2])
@pytest.mark.parametrize("lat,copies,contact,n_sub", [(9, 1, "lsd", 200), (9, 9, "lsd", 200), (9, 9, "hertz", 100),
                                                      (9, 9, "soft", 50), (15, 1, "lsd", 200), (19, 9, "lsd", 200),
                                                      (19, 9, "hertz", 100)])
def test_row_islands_match_oracle(P, orc, lat, copies, contact, n_sub, setup):
    print(f"row islands {lat} {copies} {contact} {setup}", flush=True)
    D = 2 if lat == 9 else 3
    n = (24, 16 * copies + 10, 1) if D == 2 else (24, 3 * copies + 8, 20)
    X = []
    for k in range(copies):
        for i, o in enumerate(_shapes(D)):
            at = np.array([4.0 + 0.1 * k, 4.0 + 16.0 * k + 2.1 * i]) if D == 2 else \
                np.array([4.0 + 0.1 * k, 4.0 + 2.7 * k, 3.0 + 2.1 * i])
            X.append(at + o)
        # three standing on the floor (y in 2D, z in 3D)
        up = np.eye(D)[D - 1]
        foot = np.array([12.0 + k, 0.0] if D == 2 else [12.0, 4.0 + 2.7 * k, 0.0])
        X.append(np.array([foot + up * (0.24999 + 0.49995 * m) for m in range(3)]))
    X = np.concatenate(X).T.astype(np.float32).astype(np.float64)
    rng = np.random.default_rng(13)
    U = (1e-4 * rng.standard_normal(X.shape)).astype(np.float32).astype(np.float64)
    np_ = X.shape[1]
    d, rp = np.full(np_, 0.5), np.full(np_, 2.5)
    g = [0.0, 0.0, 0.0]
    g[D - 1] = -1e-5
    cfg = P.make_config(lattice=lat, n=n, tau=0.8, gravity=g, n_sub=n_sub, contact=contact, young=1e3,
                        island_setup=setup)
    sim = P.Sim(cfg, np_)
    sim.set_particles(X, U, d, rp)
    oc = G.oracle_cfg(orc, cfg)
    out = orc.step(oc, G.to_oracle_f(orc, lat, sim.read_populations()), X, U, d, rp)
    sim.step(1)
    sim.synchronize()
    got = sim.read_particles()
    ex = np.abs(got["x"] - out["X"]).max() / np.abs(out["X"] - X).max()
    ev = np.linalg.norm(got["v"] - out["U"]) / np.linalg.norm(out["U"])
    print(f"  {np_} particles dX={ex:.2e} dU={ev:.2e}", flush=True)
    assert ex <= 1e-5 and ev <= 1e-5
