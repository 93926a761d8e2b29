"""GPU parity of the reverse pass of more than 512 particles, whose tape the
sort writes: several workgroups of the particle stage, many more bins than
particles, tiles and lanes per node; against autograd through the FP64
reference, and bitwise the same for every checkpoint interval; and from 65,536
particles on, where the first sort after a hand-over goes through records.

Bounds: those of the small adjoint tests (final positions 1e-5, gradients 1e-4
relative).
"""
import numpy as np
import pytest

from tests.test_gpu_adjoint import _gpu_grads, _ref_grads, _rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1407_6704_amd import pibm
    pibm.load()
    return pibm


def _dilute(lattice, n, np_, seed):
    """np_ particles of diameter 0.5 on a jittered grid in random order, every tenth beside its predecessor so that
    they touch (soft contacts), some of them near walls."""
    rng = np.random.default_rng(seed)
    D = 2 if lattice == 9 else 3
    ax = [np.arange(0.4, n[a] - 1.4, 1.6) for a in range(D)]
    p = np.stack(np.meshgrid(*ax, indexing="ij")).reshape(D, -1)
    assert p.shape[1] >= np_
    X = p[:, rng.permutation(p.shape[1])[:np_]] + rng.uniform(-0.1, 0.1, (D, np_))
    X[:, 1::10] = X[:, 0::10][:, :X[:, 1::10].shape[1]] + np.array([0.4, 0.15, 0.1])[:D, None]
    X = X.astype(np.float32).astype(np.float64)
    U = (1e-3 * rng.standard_normal((D, np_))).astype(np.float32).astype(np.float64)
    rp = rng.uniform(1.8, 3.0, np_) if D == 2 else rng.uniform(7.0, 9.0, np_)      # explicit drag stable with one sub-step
    return X, U, np.full(np_, 0.5), rp.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("lattice,n,np_", [(9, (90, 101, 1), 600), (19, (23, 21, 19), 600), (15, (27, 22, 21), 1100)])
def test_adjoint_of_many_matches_autograd(P, lattice, n, np_):
    print(f"adjoint of many {lattice} {n} {np_}", flush=True)
    X, U, d, rp = _dilute(lattice, n, np_, 3)
    D, tau, g, steps = X.shape[0], 0.7, 1e-3, 5
    runs = [_gpu_grads(P, lattice, n, X, U, d, rp, tau, g, steps, K) for K in (1, 3, 5)]
    for r in runs[1:]:
        assert r["dtau"] == runs[0]["dtau"] and r["dgravity"] == runs[0]["dgravity"]
        assert np.array_equal(r["dv0"], runs[0]["dv0"]) and np.array_equal(r["dx0"], runs[0]["dx0"])
    gpu, ref = runs[1], _ref_grads(lattice, n, X, U, d, rp, tau, g, steps)
    e = {"xT": np.abs(gpu["xT"] - ref["xT"]).max(), "dtau": _rel(gpu["dtau"], ref["dtau"]),
         "dg": _rel(gpu["dgravity"][:D], ref["dgravity"]), "dv0": _rel(gpu["dv0"], ref["dv0"]),
         "dx0": _rel(gpu["dx0"], ref["dx0"])}
    print("  " + " ".join(f"{k}={v:.2e}" for k, v in e.items()), flush=True)
    assert e["xT"] <= 1e-5
    assert e["dtau"] <= 1e-4 and e["dg"] <= 1e-4 and e["dv0"] <= 1e-4 and e["dx0"] <= 1e-4


@pytest.mark.parametrize("np_", [65535, 65536])
def test_reverse_pass_through_records(P, np_):
    print(f"reverse pass through records {np_}", flush=True)
    lattice, n = 9, (420, 431, 1)
    X, U, d, rp = _dilute(lattice, n, np_, 4)
    runs = [_gpu_grads(P, lattice, n, X, U, d, rp, 0.7, 1e-3, 4, K) for K in (1, 3, 4)]
    assert np.isfinite(runs[0]["dv0"]).all() and np.abs(runs[0]["dv0"]).max() > 0
    for r in runs[1:]:
        assert r["dtau"] == runs[0]["dtau"] and r["dgravity"] == runs[0]["dgravity"]
        assert np.array_equal(r["dv0"], runs[0]["dv0"]) and np.array_equal(r["dx0"], runs[0]["dx0"])


@pytest.mark.parametrize("lattice,n,np_,storage", [(9, (512, 512, 1), 10_000, "fp32"), (19, (61, 67, 72), 3000, "fp16")])
def test_a_taped_step_holds_particles_not_bins(P, lattice, n, np_, storage):
    """What a rollout's buffer grows by with each taped step: the populations, the force field and, per particle,
    positions (two parts), velocity, id and bin; nothing per bin."""
    D = 2 if lattice == 9 else 3
    sim = P.Sim(P.make_config(lattice=lattice, n=n, contact="soft", n_sub=1, storage=storage), np_)
    grown = [sim.lib.pibm_rollout_bytes(sim.ctx, t, t) for t in (200, 100)]
    per_step = (grown[0] - grown[1]) / 100
    N = n[0] * n[1] * n[2]
    held = N * (lattice * (2 if storage == "fp16" else 4) + 4 * D) + 4 * (3 * D + 2) * np_
    print(f"a taped step {lattice} {n}: {per_step / 1e6:.3f} MB", flush=True)
    assert per_step <= held + 256          # a step's share of the alignment


@pytest.mark.parametrize("np_,K", [(40, 3), (600, 3), (600, 7)])
def test_cell_list_after_the_reverse_pass(P, np_, K):
    """The keys and bins that are left after a backward pass are those of the first step, the last one reversed."""
    print(f"cell list after the reverse pass {np_} {K}", flush=True)
    n = (90, 101, 1)
    X, U, d, rp = _dilute(9, n, np_, 5)
    sim = _gpu_grads(P, 9, n, X, U, d, rp, 0.7, 1e-3, 7, K)["sim"]
    keys, _, start = sim.read_cell_list()
    plain = P.Sim(P.make_config(lattice=9, n=n, tau=0.7, gravity=(0, -1e-3, 0), contact="soft", k_soft=2e-3, n_sub=1), np_)
    plain.set_particles(X, U, d, rp)
    plain.step(1)
    ref = plain.read_cell_list()
    assert np.array_equal(keys, ref[0]) and np.array_equal(start, ref[2])
