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
