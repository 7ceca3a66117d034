"""Steps with the whole grid held on the chip (hjw_resident.h) against the launches per stage:
the same bits, for every boundary, family and precision, on ragged splits and at the edges of
the sizes that take it."""
import numpy as np
import pytest

import emulator as EM
import oracle as O
from paper_1909_13263_amd import workloads as W

TILES = [(4, 0), (8, 2), (16, 4), (16, 8)]
# one tile; one past a tile's side; narrow last tiles; tiles of three rows or more only
SHAPES = [(8, 8), (9, 65), (16, 64), (17, 129), (70, 150), (41, 200)]
FAMILIES = [(O.H_LINEAR, (0.7, -0.4), 0), (O.H_BURGERS, (1.0, 1.0, 1.0), 0),
            (O.H_NORM, (1.0, 0.0), 1), (O.H_NEGCOS, (1.0, 1.0, 0.3), 2),
            (O.H_CONTROL, (), (0, 1)), (O.H_TIMED, (0.8, -0.6, 5.0, 0.9), (1, 0)),
            (O.H_QUARTIC, (1.0, 0.5, 0.2), (2, 0))]


def _data(shape, seed):
    rng = np.random.default_rng(seed)
    return W.random_smooth_periodic(shape, seed=seed) + 0.02 * rng.normal(size=shape)


def _general(phi, h, ham, params, t_final, cfl, steps, bc, prec):
    t = 0.0
    for _ in range(steps):
        rc, phi, info = EM.rk3_step(phi, h, ham, params, t, t_final, cfl, bc, prec)
        assert rc == 0
        t = info[0]
    return phi, info


@pytest.mark.parametrize("tile", TILES, ids=lambda t: f"64x{t[0]}s{t[1]}")
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("family", range(len(FAMILIES)))
def test_emulated_resident_steps_are_the_stages_bits(tile, shape, family):
    ham, params, bc = FAMILIES[family]
    prec = (0, 1, 2)[(family + len(TILES)) % 3]
    h = (0.05, 0.06)
    phi = _data(shape, 10 * family + shape[0])
    EM.set_tile(16, 8)
    EM.set_scheme(family % 2)
    EM.set_dissipation(1 if family == 1 else 0)
    ref, ri = _general(phi, h, ham, params, 10.0, 0.4, 3, bc, prec)
    rc, got, gi = EM.resident_steps(phi, h, ham, params, 0.0, 10.0, 0.4, 3, tile, bc, prec)
    EM.set_scheme(0)
    EM.set_dissipation(0)
    assert rc == 0
    assert np.array_equal(gi, ri)
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("n", [8, 254, 255, 256, 257, 511, 700, 1030])
@pytest.mark.parametrize("bc", [0, 1, 2])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_emulated_resident_steps_1d(n, bc, prec):
    phi = _data((n,), n)
    EM.set_tile(16, 8)
    ref, ri = _general(phi, (0.05,), O.H_BURGERS, (1.0, 0.0, 1.0), 10.0, 0.4, 4, bc, prec)
    rc, got, gi = EM.resident_steps(phi, (0.05,), O.H_BURGERS, (1.0, 0.0, 1.0), 0.0, 10.0, 0.4, 4,
                                    (1, 1), bc, prec)
    assert rc == 0
    assert np.array_equal(gi, ri) and np.array_equal(got, ref)


# ------------------------------------------------------------------ on the GPU
GPU_CASES = [((8,), 0), ((160,), 0), ((257,), 2), ((5000,), 1), ((8, 8), 0), ((9, 65), 1),
             ((80, 80), 2), ((130, 100), 0), ((256, 256), 1), ((333, 517), 0), ((512, 512), 0),
             ((700, 1000), 1), ((777, 640), (0, 2)), ((1024, 1024), 0), ((1024, 1025), 0)]


def _grid(shape, bc, prec, ham, params, resident):
    from paper_1909_13263_amd import hjw
    dim = len(shape)
    g = hjw.Grid(shape, (0.0,) * dim, (4.0,) * dim, bc, prec)
    g.set_hamiltonian(ham, params)
    if not resident:
        g.set_option(hjw.OPT_USE_GRAPH, 0)   # launches per stage
    return g


@pytest.mark.gpu
@pytest.mark.parametrize("shape,bc", GPU_CASES, ids=str)
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_resident_solve_is_the_stages_bits(shape, bc, prec):
    """Whole solves with the grid on the chip against launches per stage: phi, steps, t, dt,
    alpha and the derivative box, in two calls (the second continues), and once more from a
    new phi on the same grid (the mailboxes hold the first solve's words)."""
    kinds = [(O.H_BURGERS, (1.0, 1.0 if len(shape) == 2 else 0.0, 1.0)), (O.H_NORM, (1.0, 0.0)),
             (O.H_NEGCOS, (1.0, 0.0, 0.3)), (O.H_TIMED, (0.8, -0.6 * (len(shape) - 1), 5.0, 0.9)),
             (O.H_QUARTIC, (1.0, 0.0, 0.2)), (O.H_CONTROL, ()) if len(shape) == 2 else
             (O.H_LINEAR, (0.7, 0.0))]
    ham, params = kinds[(sum(shape) + prec) % 6]
    print(f"resident {shape} bc={bc} prec={prec} ham={ham}", flush=True)
    out = []
    for resident in (True, False):
        g = _grid(shape, bc, prec, ham, params, resident)
        got = []
        for seed in (1, 2):
            phi = W.random_smooth_periodic(shape, seed=seed)
            g.set_phi(phi)
            a = g.step_to(100.0, 0.4, max_steps=5)
            b = g.step_to(a.t + 3.4 * a.last_dt, 0.4)
            got.append((g.get_phi(), a, b))
        g.close()
        out.append(got)
    for (pa, a, b), (pb, c, d) in zip(*out):
        assert a == c and b == d
        assert np.array_equal(pa, pb)


@pytest.mark.gpu
def test_two_threads_with_their_own_streams():
    """Two grids that each fill the GPU step at the same time from two threads on two streams:
    neither launch may keep the other from coming together for good, and both give the bits of
    a grid stepped alone (by either route)."""
    import threading

    import torch

    from paper_1909_13263_amd import hjw
    prs = [W.burgers2d(1024), W.negcos2d(900)]
    want = []
    for pr in prs:
        g = hjw.grid_for(pr, hjw.FP32_MIXED)
        g.set_phi(pr.phi0())
        g.step_to(1.0, 0.5, max_steps=60)
        want.append(g.get_phi())
        g.close()
    got = [None, None]

    def work(k):
        st = torch.cuda.Stream()
        g = hjw.grid_for(prs[k], hjw.FP32_MIXED, stream=st.cuda_stream)
        g.set_phi(prs[k].phi0())
        for n in (7, 13, 40):
            g.step_to(1.0, 0.5, max_steps=n)
        got[k] = g.get_phi()
        g.close()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k in range(2):
        assert np.array_equal(got[k], want[k])


@pytest.mark.gpu
@pytest.mark.parametrize("prec", [0, 1])
def test_non_finite_step_ends_the_launch_as_it_ends_the_stages(prec):
    """A solve that blows up mid-launch stops at the same step with the same record."""
    from paper_1909_13263_amd import hjw
    pr = W.burgers2d(96, 50.0)
    infos = []
    for resident in (True, False):
        g = hjw.grid_for(pr, prec)
        if not resident:
            g.set_option(hjw.OPT_USE_GRAPH, 0)
        g.set_phi(pr.phi0() * 1e3)
        with pytest.raises(hjw.HJWError) as e:
            g.step_to(pr.t_final, 40.0)
        assert e.value.code == hjw.ENONFINITE
        infos.append(g.info())
        with pytest.raises(hjw.HJWError):
            g.step_to(pr.t_final, 0.5)
        g.set_phi(pr.phi0())              # and the grid steps again
        infos.append(g.step_to(0.01, 0.5))
        infos.append(g.get_phi().tobytes())
        g.close()
    assert infos[0] == infos[3] and infos[1] == infos[4] and infos[2] == infos[5]
