"""The cell list of few particles, built in one launch, on both sides of the
particle count up to which it is (512), with several particles in a bin and
more bins than one workgroup writes: keys, the order (bin, id) and the bins'
starts against numpy, over steps that move particles between bins, with
spins and fixed points carried along.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1407_6704_amd import pibm
    pibm.load()
    return pibm


@pytest.mark.parametrize("lat,n,np_,bin_log2", [(9, (40, 30, 1), 1, 0), (9, (63, 64, 1), 511, 0), (9, (64, 63, 1), 512, 1),
                                                (9, (300, 200, 1), 513, 0), (15, (10, 10, 50), 1, 0),
                                                (19, (17, 16, 15), 64, 0), (19, (16, 16, 16), 512, 2),
                                                (19, (60, 50, 40), 300, 0)])
def test_cells_of_few_particles(P, lat, n, np_, bin_log2):
    print(f"cells of few {lat} {n} {np_} {bin_log2}", flush=True)
    D = 2 if lat == 9 else 3
    rng = np.random.default_rng(np_ + n[0])
    X = rng.random((D, np_)) * (np.array(n[:D])[:, None] - 0.6) + 0.3       # (none leaves the box)
    if np_ > 100:
        X[:, 50:90] = np.array(n[:D])[:, None] * 0.5 + 0.2 * rng.random((D, 40))       # many in a bin
    X = X.astype(np.float32).astype(np.float64)
    U = (0.02 * rng.standard_normal((D, np_))).astype(np.float32).astype(np.float64)
    d = np.full(np_, 0.5)
    cfg = P.make_config(lattice=lat, n=n, tau=0.8, n_sub=8, contact="none", bin_log2=bin_log2, skin=1.0)
    sim = P.Sim(cfg, np_)
    sim.set_particles(X, U, d, np.full(np_, 2.5))
    for step in range(3):
        x = sim.read_particles()["x"]
        sim.step(1)
        keys, ids, start = sim.read_cell_list()
        nb = [(n[a] >> bin_log2) + 1 for a in range(D)]
        b = [np.clip((np.floor(x[a] - 0.5).astype(np.int64) + 1) >> bin_log2, 0, nb[a] - 1) for a in range(D)]
        key = b[0] + nb[0] * b[1] + (nb[0] * nb[1] * b[2] if D == 3 else 0)
        order = np.lexsort((np.arange(np_), key))
        assert np.array_equal(ids, order) and np.array_equal(keys, key[order])
        assert np.array_equal(start, np.searchsorted(key[order], np.arange(np.prod(nb) + 1)))
    sim.synchronize()


@pytest.mark.parametrize("lat,np_", [(9, 512), (19, 300), (9, 513)])
def test_spins_and_fixed_points_are_carried(P, orc, lat, np_):
    from tests import gpu_helpers as G

    print(f"spins and fixed points {lat} {np_}", flush=True)
    D = 2 if lat == 9 else 3
    side = int(np.ceil(np_ ** (1.0 / D)))
    n = (side + 4, side + 5, 1) if D == 2 else (side + 4, side + 5, side + 6)
    rng = np.random.default_rng(np_ + D)
    cells = np.stack(np.meshgrid(*[np.arange(side)] * D, indexing="ij")).reshape(D, -1)
    cells = cells[:, rng.permutation(cells.shape[1])[:np_]]            # ids in no spatial order
    X = (cells + 2.3 + 0.2 * rng.random((D, np_))).astype(np.float32).astype(np.float64)
    U = (1e-4 * rng.standard_normal((D, np_))).astype(np.float32).astype(np.float64)
    d, rp = rng.uniform(0.3, 0.6, np_).astype(np.float32).astype(np.float64), np.full(np_, 2.5)
    nw = 3 if D == 3 else 1
    W = np.zeros((3, np_))
    W[3 - nw:] = (1e-4 * rng.standard_normal((nw, np_))).astype(np.float32)
    fixed = np.zeros(np_, np.int32)
    fixed[rng.permutation(np_)[:np_ // 8]] = 1
    area = np.where(fixed == 1, np.float32(0.3), 0.0)
    U[:, fixed == 1] = 0.0
    cfg = P.make_config(lattice=lat, n=n, tau=0.8, gravity=(0, -1e-5, 0), n_sub=50, contact="hertz_mindlin", young=1e3,
                        bodies=1)
    sim = P.Sim(cfg, np_)
    sim.set_particles(X, U, d, rp)
    sim.set_rotation(W[3 - nw:])
    sim.set_bodies(np.where(fixed == 1, 0, -1), area=area)
    oc = G.oracle_cfg(orc, cfg)
    f, Xo, Uo = G.to_oracle_f(orc, lat, sim.read_populations()), X, U
    for step in range(2):
        out = orc.step_full(oc, f, Xo, Uo, d, rp, W=W, hist=None, fixed=fixed, area=area)
        f, Xo, Uo = out["f"], out["X"], out["U"]
    sim.step(2)
    sim.synchronize()
    got = sim.read_particles()
    ex = np.abs(got["x"] - Xo).max() / np.abs(Xo - X).max()
    ev = np.linalg.norm(got["v"] - Uo) / np.linalg.norm(Uo)
    print(f"  dX={ex:.2e} dU={ev:.2e}", flush=True)
    assert ex <= 1e-5 and ev <= 1e-5
    assert np.array_equal(got["x"][:, fixed == 1], X[:, fixed == 1])
    assert np.array_equal(sim.read_rotation(), W[3 - nw:])             # no contact: spins unchanged
