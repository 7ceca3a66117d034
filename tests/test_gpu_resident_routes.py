"""Which route a grid's steps take on the GPU (one launch for many, or launches per stage), and the
ways from one to the other: the count of steps taken in one launch says that the kernel under test
ran, and every mixture gives the bits of the launches per stage."""
import numpy as np
import pytest

from paper_1909_13263_amd import workloads as W

hjw = pytest.importorskip("paper_1909_13263_amd.hjw")
pytestmark = pytest.mark.gpu

FP64, MIXED, FP32 = 0, 1, 2
# every instantiation: 1-D; 64 x 4, 64 x 8, 64 x 16 by 4 and by 8 nodes; three precisions
FITS = [((160,), 0), ((5000,), 1), ((80, 80), 0), ((256, 256), 1), ((256, 256), 0), ((256, 500), 2),
        ((512, 512), 1), ((512, 512), 0), ((640, 640), 0), ((1000, 1000), 2), ((1024, 1024), 1)]


def _grid(shape, prec, timed=False, **options):
    dim = len(shape)
    g = hjw.Grid(shape, (0.0,) * dim, (4.0,) * dim, 0, prec)
    if timed:
        g.set_hamiltonian(hjw.H_TIMED, (0.8, -0.6 * (dim - 1), 5.0, 0.9))
    else:
        g.set_hamiltonian(hjw.H_BURGERS, (1.0, 1.0 * (dim - 1), 1.0))
    for name, value in options.items():
        g.set_option(getattr(hjw, name), value)
    g.set_phi(W.random_smooth_periodic(shape, seed=3))
    return g


def _run(g, calls):
    for n in calls:
        info = g.step_to(100.0, 0.4, max_steps=n)
    return info, g.get_phi()


@pytest.mark.parametrize("shape,prec", FITS, ids=str)
@pytest.mark.parametrize("timed", [False, True])
def test_a_grid_that_fits_steps_in_one_launch(shape, prec, timed):
    print(f"one launch {shape} prec={prec} timed={timed}", flush=True)
    g = _grid(shape, prec, timed)
    info, phi = _run(g, (5, 6))
    assert info.steps == g.resident_steps() == 11
    s = _grid(shape, prec, timed, OPT_RESIDENT=0)
    ref, phi_s = _run(s, (5, 6))
    assert s.resident_steps() == 0
    assert info == ref and np.array_equal(phi, phi_s)


@pytest.mark.parametrize("shape,prec,options", [
    ((1024, 1025), MIXED, {}), ((800, 800), FP64, {}), ((1024 * 255 + 1,), FP64, {}),
    ((128, 128), MIXED, {"OPT_USE_GRAPH": 0}), ((128, 128), MIXED, {"OPT_SEGMENT": 8}),
    ((128, 128), MIXED, {"OPT_PLAN": 1}), ((128, 128), MIXED, {"OPT_TILE_ROWS": 32}),
    ((128, 128), MIXED, {"OPT_KERNEL_EVENTS": 1})], ids=str)
def test_a_grid_that_does_not_takes_launches_per_stage(shape, prec, options):
    g = _grid(shape, prec, **options)
    info, _ = _run(g, (5,))
    assert info.steps == 5 and g.resident_steps() == 0


@pytest.mark.parametrize("shape,prec", [((5000,), 0), ((256, 256), 1), ((512, 512), 0), ((1024, 1024), 2)],
                         ids=str)
def test_a_meeting_given_up_changes_nothing(shape, prec):
    """Launches that wait for a workgroup too many (option 2) leave without having changed
    anything, before, between and after launches that meet."""
    print(f"given up {shape} prec={prec}", flush=True)
    g = _grid(shape, prec, OPT_RESIDENT=2)
    calls = (5, 1, 20)
    _run(g, calls)
    assert g.resident_steps() == 0
    g.set_option(hjw.OPT_RESIDENT, 1)
    _run(g, (300,))
    taken = g.resident_steps()
    assert taken > 0                       # and it does not stay with the launches per stage
    g.set_option(hjw.OPT_RESIDENT, 2)
    info, phi = _run(g, (30, 7))
    assert g.resident_steps() == taken
    s = _grid(shape, prec, OPT_RESIDENT=0)
    ref, phi_s = _run(s, calls + (300, 30, 7))
    assert info == ref and np.array_equal(phi, phi_s)


@pytest.mark.parametrize("shape,prec", [((600,), 0), ((80, 80), 1), ((256, 256), 0), ((640, 640), 1)], ids=str)
def test_a_launch_whose_waits_run_out_fails_and_the_grid_recovers(shape, prec):
    """Option 3: no wait has a second look, so workgroups give up at different places and end;
    the call fails, the grid is failed until phi is set, and then its steps are right."""
    print(f"waits run out {shape} prec={prec}", flush=True)
    g = _grid(shape, prec, OPT_RESIDENT=3)
    for _ in range(3):
        with pytest.raises(hjw.HJWError) as e:
            g.step_to(100.0, 0.4, max_steps=50)
        assert e.value.code == hjw.EHIP
        with pytest.raises(hjw.HJWError) as e:
            g.step_to(100.0, 0.4, max_steps=50)
        assert e.value.code == hjw.ESTATE
        g.set_phi(W.random_smooth_periodic(shape, seed=3))
    g.set_option(hjw.OPT_RESIDENT, 1)
    info, phi = _run(g, (9, 3, 40))
    assert g.resident_steps() == 52
    s = _grid(shape, prec, OPT_RESIDENT=0)
    ref, phi_s = _run(s, (9, 3, 40))
    assert info == ref and np.array_equal(phi, phi_s)


@pytest.mark.parametrize("prec", [FP64, MIXED, FP32])
def test_graph_replays_at_both_parities_are_the_eager_launches(prec):
    """Replays of whole steps from a graph, captured at each parity of the step record (an odd
    number of eager steps between), with reads and eager work between them, every one against
    eager launches."""
    pr = W.burgers2d(192)
    grids = []
    for options in ({"OPT_RESIDENT": 0}, {"OPT_USE_GRAPH": 0}):
        g = hjw.grid_for(pr, prec)
        for name, value in options.items():
            g.set_option(getattr(hjw, name), value)
        g.set_phi(pr.phi0())
        grids.append(g)
    for n in (16, 3, 32, 16, 1, 48, 5, 16):
        infos = [g.step_to(100.0, 0.4, max_steps=n) for g in grids]
        assert infos[0] == infos[1]
        assert np.array_equal(grids[0].get_phi(), grids[1].get_phi())
        _ = grids[0].derivatives()
    assert grids[0].resident_steps() == grids[1].resident_steps() == 0


def test_a_server_and_a_grid_step_at_the_same_time():
    """A server drains a batch in one thread while a grid that fills the GPU steps in another:
    both give the bits that they give alone, whichever routes the grid takes."""
    import threading

    import torch
    problems = [W.burgers2d(200 + 40 * k, 0.02) for k in range(6)]
    pr = W.burgers2d(1024)

    def serve(out):
        st = torch.cuda.Stream()
        srv = hjw.Server(MIXED, pool_bytes=256 << 20, max_active=16, stream=st.cuda_stream)
        for _ in range(3):
            ids = [srv.submit(p) for p in problems]
            done = {r.rid: r.phi for r in srv.drain()}
            out.append([done[i] for i in ids])
        srv.close()

    def step(out):
        st = torch.cuda.Stream()
        g = hjw.grid_for(pr, MIXED, stream=st.cuda_stream)
        g.set_phi(pr.phi0())
        for n in (1, 70, 200, 2, 5):
            out.append((g.step_to(1.0, 0.5, max_steps=n), g.get_phi()))
        g.close()

    alone, together = ([], []), ([], [])
    serve(alone[0])
    step(alone[1])
    threads = [threading.Thread(target=serve, args=(together[0],)),
               threading.Thread(target=step, args=(together[1],))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(together[0]) == len(alone[0]) and len(together[1]) == len(alone[1])
    for a, b in zip(alone[0], together[0]):
        assert all(np.array_equal(x, y) for x, y in zip(a, b))
    for (ia, pa), (ib, pb) in zip(alone[1], together[1]):
        assert ia == ib and np.array_equal(pa, pb)
