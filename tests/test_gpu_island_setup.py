"""GPU parity of the island set-up in one workgroup on both sides of its
thread count (1024 active particles: one thread each, islands in LDS; more:
in turns), with pairs, rows of three and a chain longer than a wave, and of
the same scenes through the multi-kernel set-up, against the FP64 oracle.

Bounds of the other contact tests: positions (against the largest
displacement) and velocities 1e-5 relative.
"""
import numpy as np
import pytest

from tests import gpu_helpers as G
from tests.test_gpu_island_layout import _touching

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1407_6704_amd import pibm
    pibm.load()
    return pibm


@pytest.mark.parametrize("setup", [1, 2])
@pytest.mark.parametrize("pairs,walls,triples,chain,contact", [
    (1, 0, 0, 0, "lsd"), (482, 0, 20, 0, "lsd"), (482, 1, 20, 0, "lsd"), (440, 0, 20, 70, "hertz"),
    (440, 6, 20, 80, "hertz_mindlin"), (500, 40, 40, 150, "lsd")])
def test_island_setup_matches_oracle(P, orc, pairs, walls, triples, chain, contact, setup):
    print(f"island set-up {pairs} {walls} {triples} {chain} {contact} {setup}", flush=True)
    n, X, U, d = _touching(2, pairs, max(walls, 1), triples)
    if walls == 0:
        X, U, d = X[:, :-1], U[:, :-1], d[:-1]
    if chain:
        rng = np.random.default_rng(7)
        Xc = np.stack([20.0 + 0.4999 * np.arange(chain), 60.0 + 0.0 * np.arange(chain)])
        X = np.concatenate([X, Xc.astype(np.float32).astype(np.float64)], 1)
        U = np.concatenate([U, (1e-4 * rng.standard_normal(Xc.shape)).astype(np.float32).astype(np.float64)], 1)
        d = np.concatenate([d, np.full(chain, 0.5)])
    rp = np.full(X.shape[1], 2.5)
    cfg = P.make_config(lattice=9, n=n, tau=0.8, gravity=(0, -1e-5, 0), n_sub=100, contact=contact, young=1e3,
                        island_setup=setup)
    sim = P.Sim(cfg, X.shape[1])
    sim.set_particles(X, U, d, rp)
    oc = G.oracle_cfg(orc, cfg)
    f = G.to_oracle_f(orc, 9, sim.read_populations())
    if contact == "hertz_mindlin":
        out = orc.step_hm(oc, f, X, U, np.zeros((3, X.shape[1])), d, rp, None)
    else:
        out = orc.step(oc, f, X, U, d, rp)
    sim.step(1)
    sim.synchronize()
    assert sim.diagnostics()["active"] == X.shape[1]
    got = sim.read_particles()
    ex = np.abs(got["x"] - out["X"]).max() / np.abs(out["X"] - X).max()
    ev = np.linalg.norm(got["v"] - out["U"]) / np.linalg.norm(out["U"])
    print(f"  active {X.shape[1]} dX={ex:.2e} dU={ev:.2e}", flush=True)
    assert ex <= 1e-5 and ev <= 1e-5
