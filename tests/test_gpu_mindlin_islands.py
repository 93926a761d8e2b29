"""GPU parity of Hertz-Mindlin islands of three and more particles, which run
with four lanes per member where every member has at most four candidates and
no wall in reach: chains of 3 to 17 (more than sixteen take the general loop),
triangles, a particle with four and with six partners, several of each so that
they fill more than one workgroup's share, beside pairs; two steps, so that
the tangential history is carried, against the FP64 oracle.

Bounds of the other Hertz-Mindlin tests: positions (against the largest
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


def _shapes(D):
    s = 0.4998                                                   # of diameter 0.5: every neighbour touches
    ax = np.eye(3)
    out = [np.outer(np.arange(m) * s, ax[0]) for m in (2, 3, 4, 5, 8, 16, 17)]
    out.append(np.array([[0, 0, 0], [s, 0, 0], [0.5 * s, s * np.sqrt(0.75), 0]]))
    out.append(np.array([[0, 0, 0], [s, 0, 0], [-s, 0, 0], [0, s, 0], [0, -s, 0]]))
    if D == 3:
        out.append(np.concatenate([[[0, 0, 0]], s * ax, -s * ax]))           # six partners
    else:
        t = np.arange(6) * np.pi / 3
        out.append(np.concatenate([[[0, 0, 0]], s * np.stack([np.cos(t), np.sin(t), 0 * t], 1)]))
    return [o[:, :D] for o in out]


@pytest.mark.parametrize("lat,copies,contact", [(9, 1, "hertz_mindlin"), (9, 9, "hertz_mindlin"),
                                                (19, 9, "hertz_mindlin"), (19, 2, "hertz_mindlin_microslip")])
def test_mindlin_islands_match_oracle(P, orc, lat, copies, contact):
    print(f"mindlin islands {lat} {copies} {contact}", flush=True)
    D = 2 if lat == 9 else 3
    shapes = _shapes(D)
    n = (28, 11 * copies + 10, 1) if D == 2 else (28, 4 * copies + 8, 24)
    if D == 2:
        n = (28, 22 * copies + 8, 1)
    X = []
    for k in range(copies):
        for i, o in enumerate(shapes):
            at = np.array([4.0 + 0.1 * k, 4.0 + 22.0 * k + 2.1 * i]) if D == 2 else \
                np.array([4.0 + 0.1 * k, 4.0 + 3.5 * k, 3.0 + 1.9 * i])
            X.append(at + o)
    X = np.concatenate(X).T.astype(np.float32).astype(np.float64)
    rng = np.random.default_rng(11)
    np_ = X.shape[1]
    U = (2e-4 * rng.standard_normal((D, np_))).astype(np.float32).astype(np.float64)
    nw = 3 if D == 3 else 1
    W = np.zeros((3, np_))
    W[3 - nw:] = (1e-3 * rng.standard_normal((nw, np_))).astype(np.float32)
    d, rp = np.full(np_, 0.5), np.full(np_, 2.5)
    g = [0.0, 0.0, 0.0]
    g[D - 1] = -1e-5
    cfg = P.make_config(lattice=lat, n=n, tau=0.8, gravity=g, n_sub=200, contact=contact, young=1e3)
    sim = P.Sim(cfg, np_)
    sim.set_particles(X, U, d, rp)
    sim.set_rotation(W if D == 3 else W[2:3])
    oc = G.oracle_cfg(orc, cfg)
    f = G.to_oracle_f(orc, lat, sim.read_populations())
    Xo, Uo, Wo, hist = X.copy(), U.copy(), W.copy(), None
    for _ in range(2):
        out = orc.step_hm(oc, f, Xo, Uo, Wo, d, rp, hist)
        f, Xo, Uo, Wo, hist = out["f"], out["X"], out["U"], out["W"], out["hist"]
    sim.step(2)
    sim.synchronize()
    got = sim.read_particles()
    w = sim.read_rotation()
    ref = Wo if D == 3 else Wo[2:3]
    ex = np.abs(got["x"] - Xo).max() / np.abs(Xo - X).max()
    ev = np.linalg.norm(got["v"] - Uo) / np.linalg.norm(Uo)
    ew = np.linalg.norm(w - ref) / np.linalg.norm(ref)
    print(f"  {np_} particles dX={ex:.2e} dU={ev:.2e} dW={ew:.2e}", flush=True)
    assert ex <= 1e-5 and ev <= 1e-5 and ew <= 1e-5


@pytest.mark.parametrize("contact", ["hertz_mindlin", "hertz_mindlin_microslip"])
def test_member_with_many_candidates(P, orc, contact):
    """Hubs of twelve equal spheres around one (the corners of an icosahedron), which all touch it and are in reach of
    each other."""
    print(f"many candidates {contact}", flush=True)
    rng = np.random.default_rng(12)
    n, t = (24, 14, 12), 0.5 * (1 + 5 ** 0.5)
    e = np.array([p for s in (1, -1) for u in (t, -t) for p in ((0, s, u), (s, u, 0), (u, 0, s))]) / np.sqrt(1 + t * t)
    hub = 0.4998 * np.concatenate([np.zeros((1, 3)), e])
    X = np.concatenate([np.array([5.1, 5.2, 5.3]) + hub, np.array([15.4, 7.3, 6.2]) + hub]).T
    X = X.astype(np.float32).astype(np.float64)
    np_ = X.shape[1]
    U = (2e-4 * rng.standard_normal((3, np_))).astype(np.float32).astype(np.float64)
    W = (1e-3 * rng.standard_normal((3, np_))).astype(np.float32).astype(np.float64)
    d, rp = np.full(np_, 0.5), np.full(np_, 2.5)
    cfg = P.make_config(lattice=19, n=n, tau=0.8, gravity=(0, 0, -1e-5), n_sub=200, contact=contact, young=1e3)
    sim = P.Sim(cfg, np_)
    sim.set_particles(X, U, d, rp)
    sim.set_rotation(W)
    oc = G.oracle_cfg(orc, cfg)
    f = G.to_oracle_f(orc, 19, sim.read_populations())
    Xo, Uo, Wo, hist = X.copy(), U.copy(), W.copy(), None
    for _ in range(2):
        out = orc.step_hm(oc, f, Xo, Uo, Wo, d, rp, hist)
        f, Xo, Uo, Wo, hist = out["f"], out["X"], out["U"], out["W"], out["hist"]
    sim.step(2)
    sim.synchronize()
    got, w = sim.read_particles(), sim.read_rotation()
    ex = np.abs(got["x"] - Xo).max() / np.abs(Xo - X).max()
    ev = np.linalg.norm(got["v"] - Uo) / np.linalg.norm(Uo)
    ew = np.linalg.norm(w - Wo) / np.linalg.norm(Wo)
    print(f"  dX={ex:.2e} dU={ev:.2e} dW={ew:.2e}", flush=True)
    assert ex <= 1e-5 and ev <= 1e-5 and ew <= 1e-5
