"""An island's result depends on its own members only, not on the islands that
happen to share its wave or workgroup (their order of ranking is not fixed):
five touching islands (pairs, chains of three and four) run beside one more of
their size, which lies free, has a wall in reach, holds a fixed point, or (of
four) is a star with three candidates at its centre.  The fluid is not driven
(one-way coupling), so the five see nothing else of the sixth: their positions,
velocities, forces and spins after one and two steps are equal bit for bit.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

S = 0.4998                                                   # of diameter 0.5: every neighbour touches


@pytest.fixture(scope="module")
def P():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1407_6704_amd import pibm
    pibm.load()
    return pibm


def _chain(m):
    return np.outer(np.arange(m) * S, [1.0, 0.0, 0.0])


def _star():
    return S * np.array([[0.0, 0, 0], [1, 0, 0], [-1, 0, 0], [0, 1, 0]])


@pytest.mark.parametrize("setup", [1, 2])
@pytest.mark.parametrize("size", [2, 3, 4])
@pytest.mark.parametrize("lat,contact", [(9, "lsd"), (19, "lsd"), (19, "hertz"), (9, "hertz_mindlin"),
                                         (19, "hertz_mindlin"), (19, "hertz_mindlin_microslip")])
def test_island_does_not_depend_on_its_company(P, lat, contact, size, setup):
    D = 2 if lat == 9 else 3
    md = contact.startswith("hertz_mindlin")
    n = (20, 40, 1) if D == 2 else (20, 40, 12)
    rng = np.random.default_rng(5)
    up = 2e-4 * rng.standard_normal((6 * size, D))
    spin = 1e-3 * rng.standard_normal((6 * size, 3))

    def run(company):
        shapes = [_chain(size)] * 5 + [_star() if company == "star" else _chain(size)]
        x = np.concatenate([np.array([0.2505 if company == "wall" and k == 5 else 8.0, 5.0 + 6.0 * k, 5.7])[:D] +
                            o[:, :D] for k, o in enumerate(shapes)])
        x = x.T.astype(np.float32).astype(np.float64)
        np_ = x.shape[1]
        cfg = P.make_config(lattice=lat, n=n, tau=0.8, gravity=(0.0, -1e-5, 0.0), n_sub=200, contact=contact, young=1e3,
                            two_way=0, bodies=1, island_setup=setup)
        sim = P.Sim(cfg, np_)
        sim.set_particles(x, up.T, np.full(np_, 0.5), np.full(np_, 2.5))
        if md:
            sim.set_rotation(spin.T if D == 3 else spin.T[2:3])
        body = np.full(np_, -1, np.int32)
        if company == "fixed":
            body[5 * size] = 0
        sim.set_bodies(body)
        out = []
        for step in range(2):
            sim.step(1)
            sim.synchronize()
            got = sim.read_particles()
            out += [got[k][:, :5 * size].copy() for k in ("x", "v", "f_hydro", "f_contact")]
            if md:
                out.append(sim.read_rotation()[:, :5 * size].copy())
        assert np.abs(out[3]).min(axis=1).max() > 0.0           # every member is in contact during the first step
        return out

    alone = run("free")
    for company in ("wall", "fixed") + (("star",) if size == 4 else ()):
        print(f"island company {lat} {contact} {size} {setup} {company}", flush=True)
        for k, (a, b) in enumerate(zip(alone, run(company))):
            assert np.array_equal(a, b), (company, k)
