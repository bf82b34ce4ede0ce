"""Small D2Q9 lattices take several steps in one launch, in regions with a halo
of four cells per step: parity with the FP64 oracle (FP64 element by element
within 1e-12 of the largest population; FP32 rho, T, P rel-L2 1e-5 -- the
velocities here are a few 1e-3 c_s, where the FP32 pressure's rounding alone is
1e-5 of them, so u is held by the FP64 form of the same code) over the forms of a
region -- whole lattice, own columns with halos that wrap, end at a
zero-gradient wall or at a diffuse wall -- and independence of the split: one
call of n steps, n calls of one step and a restart in between agree bitwise."""
import sys

import numpy as np
import pytest

import oracle
from paper_2510_14712_amd import inputs

pytestmark = pytest.mark.gpu

ST = inputs.states()
KW = inputs.physics(ST)
RHOC, TC = ST["critical"]["rho"], ST["critical"]["T"]
WALLS = (((0.0, -0.04), 0.95 * TC), ((0.0, 0.08), 1.25 * TC))

# whole lattices (one row, one column, the largest of each type), then columns:
# a last region of one column, halos longer than the lattice's rest
CASES = [
    ((512, 1), (0, 0)), ((1, 37), (1, 1)), ((25, 12), (1, 0)), ((32, 16), (0, 1)), ((4, 5), (0, 0)),
    ((513, 4), (1, 0)), ((517, 3), (0, 0)), ((300, 9), (1, 1)), ((190, 12), (0, 0)), ((1000, 4), (0, 1)),
    ((23, 6), (2, 0)), ((64, 8), (2, 0)), ((1, 4), (2, 0)), ((203, 5), (2, 0)), ((2, 3), (2, 0)),
]


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("shape,bc", CASES)
def test_several_steps_per_launch_match_oracle(storage, shape, bc):
    from paper_2510_14712_amd import lbm
    lbm.load()
    steps = 19
    kw = dict(KW, walls=WALLS) if bc[0] == 2 else KW
    rho, u, T = inputs.random_state(2, shape, 57, RHOC, 1.1 * TC, drho=0.04, du=0.06, dT=0.03, white=0.005)
    print(f"case {storage} {shape} bc={bc}", flush=True)
    sys.stdout.flush()
    lats = [lbm.Lattice(2, shape, bc=bc + (0,), storage=storage, **kw) for _ in range(3)]
    try:
        one, many, again = lats
        one.init(rho, u, T).step(steps)
        many.init(rho, u, T)
        for _ in range(steps):
            many.step(1)
        again.init(rho, u, T).step(8)
        again.set_populations(*again.get_populations())
        again.step(steps - 8)
        pops = [[t.cpu().numpy() for t in lat.get_populations()] for lat in lats]
        mom = {k: v.cpu().numpy() for k, v in one.moments().items()}
        kinds = set(one.step_timed(3))
    finally:
        for lat in lats:
            lat.close()
    assert kinds == {"k_block2d"}
    for f, g in pops[1:]:
        assert np.array_equal(f, pops[0][0]) and np.array_equal(g, pops[0][1])
    p = oracle.Params(2, shape, bc=bc + (0,), **kw)
    fr, gr = oracle.run(p, *oracle.init(p, rho, u, T), steps)
    if storage == "f64":
        assert np.max(np.abs(pops[0][0] - fr)) <= 1e-12 * np.abs(fr).max()
        assert np.max(np.abs(pops[0][1] - gr)) <= 1e-12 * np.abs(gr).max()
    ref = oracle.fields(p, fr, gr)
    for k in ("rho", "T", "P") + (("u",) if storage == "f64" else ()):
        err = np.linalg.norm(mom[k] - ref[k]) / np.linalg.norm(ref[k])
        assert err <= (1e-12 if storage == "f64" else 1e-5), (k, err)


def test_larger_lattices_keep_the_step_of_one_launch_each():
    from paper_2510_14712_amd import lbm
    lbm.load()
    rho, u, T = inputs.random_state(2, (256, 65), 58, RHOC, 1.1 * TC)
    with lbm.Lattice(2, (256, 65), storage="f32", **KW) as lat:
        assert set(lat.init(rho, u, T).step_timed(2)) == {"k_fused", "k_fused_fixup"}  # 65 = 16 x 4 + 1 rows: one-cell tiles
    rho, u, T = inputs.random_state(2, (256, 66), 58, RHOC, 1.1 * TC)
    with lbm.Lattice(2, (256, 66), storage="f32", **KW) as lat:
        assert set(lat.init(rho, u, T).step_timed(2)) == {"k_fused"}


@pytest.mark.parametrize("shape,bc,steps", [((64, 4), (0, 0), 6), ((64, 8), (2, 0), 4), ((1000, 4), (0, 1), 10)])
def test_captured_even_step_counts_replay(shape, bc, steps):
    """A call of an even number of steps leaves the two buffers as it found
    them, whatever the steps per launch: its graph advances the state at every
    replay, bit for bit as the calls themselves do."""
    import torch
    from paper_2510_14712_amd import lbm
    lbm.load()
    kw = dict(KW, walls=WALLS) if bc[0] == 2 else KW
    rho, u, T = inputs.random_state(2, shape, 59, RHOC, 1.1 * TC, drho=0.04, du=0.06, dT=0.03)
    print(f"case {shape} bc={bc} steps {steps}", flush=True)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with lbm.Lattice(2, shape, bc=bc + (0,), storage="f64", stream=s, **kw) as a, \
            lbm.Lattice(2, shape, bc=bc + (0,), storage="f64", stream=s, **kw) as b, torch.cuda.stream(s):
        a.init(rho, u, T).step(2)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            a.step(steps)
        b.init(rho, u, T).step(2)
        for _ in range(3):
            graph.replay()
            b.step(steps)
            torch.cuda.synchronize()
            for p, q in zip(a.get_populations(), b.get_populations()):
                assert torch.equal(p, q)
