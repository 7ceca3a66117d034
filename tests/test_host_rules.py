"""Where a grid's steps go and what its launches are given, by the library's own host code on a
stand-in HIP runtime (tests/host): no GPU, every case in a process of its own."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module", autouse=True)
def stub():
    from paper_1909_13263_amd import build
    if not os.path.exists(build.HIP_STUB):
        build.build_hip_stub()


def _run(body):
    code = "from rig import *\nsetup()\n" + textwrap.dedent(body)
    r = subprocess.run([sys.executable, "-c", code], cwd=os.path.join(HERE, "host"), timeout=120,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout


def test_rebind_to_another_device_moves_the_exchange_area():
    """After a bind to a second device every launch's mailboxes lie there, and the first
    device's have been given back."""
    _run("""
        g = Grid((256, 256))
        assert g.step(5)[0] == 0
        assert [r[4] for r in resident(log())] == [0]
        g.bind(1)
        lines = log()
        assert "free device=0" in lines and "malloc device=1" in lines, lines
        g.set_phi()
        assert g.step(5)[0] == 0
        lines = log()
        assert [r[4] for r in resident(lines)] == [1], lines
        S.hipSetDevice(0)              # whichever device is current at the call
        assert g.step(5)[0] == 0
        assert [r[4] for r in resident(log())] == [1]
        g.bind(1)                      # the same device again: the area is kept, and cleared
        assert log() == ["clear device=1"]
        g.close()
        assert "free device=1" in log()
    """)


def test_a_launch_that_stopped_answering_leaves_no_tags():
    """The words of a broken launch carry its tags: before the grid steps again in one launch,
    the mailboxes are cleared or the tags are others."""
    _run("""
        g = Grid((256, 256))
        S.stub_modes(b"2")
        assert g.step(40)[0] == EHIP
        before = log()
        broken = resident(before)[-1]
        S.stub_modes(b"0")
        assert g.step(5)[0] != 0       # failed until phi is set again
        g.set_phi()
        assert g.step(5)[0] == 0
        lines = log()
        (after,) = resident(lines)
        sent = next(k for k, l in enumerate(before) if "resident" in l)
        first = next(k for k, l in enumerate(lines) if "resident" in l)
        cleared = "clear device=0" in before[sent:] + lines[:first]
        assert cleared or after[2] > broken[2] + broken[3], (broken, lines)
    """)


def test_tiles_are_chosen_for_the_devices_own_units():
    """On 32 compute units a grid takes the tiles that fit there (16 rows, four a unit), and FP64
    grids of just over three tiles a unit, not of just over 768, the dense kernels."""
    _run("""
        setup(cus=32)
        g = Grid((512, 256))
        assert g.step(5)[0] == 0
        assert [r[:2] for r in resident(log())] == [(128, 256)]
        for shape, dense in (((1024, 1024), False), ((448, 256), True), ((512, 384), False)):
            g = Grid(shape, FP64)
            assert g.step(3)[0] == 0
            lines = [l for l in log() if l.startswith("step")]
            assert len(lines) == 3 and all(l.endswith("dense") == dense for l in lines), lines
        setup(cus=256)
        g = Grid((512, 256))
        assert g.step(5)[0] == 0
        assert [r[:2] for r in resident(log())] == [(256, 512)]   # 8 rows
        g = Grid((1024, 1024), FP64)
        assert g.step(3)[0] == 0
        assert sum(l.endswith("dense") for l in log()) == 3
    """)


def test_grids_that_do_not_fit_together_keep_to_launches_per_stage():
    """A call that begins while another grid of the process is stepping on the device takes the
    resident launch only where both fit at once."""
    _run("""
        for shape, fits in (((1024, 1024), False), ((128, 128), True), ((512, 512), False)):
            a, b = Grid(shape), Grid(shape)
            setup(per_cu=4 if shape[0] == 1024 else 2)
            seen = []
            @HOOK
            def beside():
                if not seen:
                    seen.append(None)
                    log()
                    assert b.step(100)[0] == 0
                    seen.append(log())
            S.stub_hook(beside)
            rc, info = a.step(100)
            S.stub_hook(HOOK(0))
            assert rc == 0 and info.steps == 100
            assert bool(resident(seen[1])) == fits, (shape, seen)
            assert staged(seen[1]) == (0 if fits else 100)
            log()
            assert b.step(100)[0] == 0            # alone again
            lines = log()
            assert staged(lines) == 0 and resident(lines)
            other = Grid((1024, 1024), device=1)  # another device's calls are no company
            seen.clear()
            def elsewhere():
                if not seen:
                    seen.append(None)
                    log()
                    assert other.step(100)[0] == 0
                    seen.append(log())
            keep = HOOK(elsewhere)
            S.stub_hook(keep)
            assert a.step(100)[0] == 0
            S.stub_hook(HOOK(0))
            if shape[0] == 1024:
                assert resident(seen[1])
    """)


def test_a_meeting_given_up_is_not_tried_again_at_once():
    """After a meeting that was given up the next 64 steps go by stages, whatever the calls they
    come in, then 128, and so on; one that is kept starts the count anew."""
    _run("""
        g = Grid((256, 256))
        S.stub_modes(b"1")
        tries, steps = [], 0
        for k in range(500):
            rc, info = g.step(1)
            steps += 1
            assert rc == 0 and info.steps == steps
            if resident(log()):
                tries.append(steps)
        assert tries == [1, 65, 193, 449], tries
        S.stub_modes(b"0")
        assert g.step(2000)[0] == 0           # the pause runs out in it, and the meeting is kept
        assert resident(log())
        S.stub_modes(b"1")
        tries, start = [], steps + 2000
        for k in range(200):
            rc, info = g.step(1)
            if resident(log()):
                tries.append(info.steps - start)
        assert tries == [1, 65, 193], tries
    """)


def test_a_launch_that_fills_the_gpu_is_short():
    """Launches that fill more than half of the GPU end after 64 steps, others after 256; the tags
    of launches that follow each other are apart."""
    _run("""
        for shape, prec, most in (((1024, 1024), FP32_MIXED, 64), ((256, 256), FP32_MIXED, 256),
                                  ((640, 640), FP64, 64), ((160,), FP64, 256)):
            setup(per_cu=2 if prec == FP64 else 4)
            log()
            g = Grid(shape, prec)
            assert g.step(7)[0] == 0
            rc, info = g.step(1000)
            assert rc == 0 and info.steps == 1007
            lines = log()
            assert not staged(lines)
            launches = resident(lines)
            assert max(r[3] for r in launches) == most
            for x, y in zip(launches, launches[1:]):
                assert y[2] > x[2] + x[3]
            rc, info = g.step(t=info.t + 99.5 * STEP)     # by time: a step to spare at most
            assert rc == 0 and info.steps == 1107
    """)


def test_a_chain_of_launches_stops_at_the_first_that_does_not_meet():
    """Launches queued behind one that gave up, or that stopped answering, do nothing."""
    _run("""
        g = Grid((1024, 1024))
        assert g.step(10)[0] == 0
        S.stub_modes(b"010")
        rc, info = g.step(256)
        assert rc == 0 and info.steps == 266
        lines = log()
        assert staged(lines) >= 64            # then by stages, and by launches again
        taken = i64()
        assert L.hjw_resident_steps(g.h, ctypes.byref(taken)) == 0
        assert taken.value + staged(lines) == 266
        S.stub_modes(b"020")
        assert g.step(256)[0] == EHIP
        lines = log()
        assert lines[-1] == "clear device=0"
        S.stub_modes(b"0")
        g.set_phi()
        rc, info = g.step(256)
        assert rc == 0 and info.steps == 256
    """)


def test_few_steps_of_a_full_grid_take_launches_per_stage():
    _run("""
        for shape, few in (((1024, 1024), True), ((256, 256), False)):
            g = Grid(shape)
            for n, by_stages in ((1, few), (2, few), (3, False)):
                log()
                assert g.step(n)[0] == 0
                assert staged(log()) == (n if by_stages else 0), (shape, n)
            rc, info = g.step(t=6 * STEP + 1.5 * STEP)      # two steps by time
            assert rc == 0 and info.steps == 8
    """)


def test_the_no_allocation_solves_array_holds_every_exchange_area_and_little_more():
    """The largest grids of each precision, tile and dimension that step in one launch do so on the
    library's own array, which is as large as the header says."""
    _run("""
        S.stub_variables.restype = ctypes.c_size_t
        assert 54 << 20 < S.stub_variables() < 56 << 20
        for n, prec, count in (((1024, 1024), FP32_MIXED, 1024), ((1024, 1024), FP32, 1024),
                               ((64, 16384), FP32_MIXED, 1024), ((1024, 512), FP64, 512),
                               ((256, 256), FP64, 256), ((255 * 1024,), FP64, 1024)):
            dim = len(n)
            phi = S.stub_malloc(8 * n[0] * (n[1] if dim == 2 else 1), 0)
            info = Info()
            rc = L.hjw_solve_noalloc(
                dim, (i64 * dim)(*n), (dbl * dim)(*[0.0] * dim), (dbl * dim)(*[1.0] * dim),
                (ctypes.c_int * dim)(*[0] * dim), prec, 1, (dbl * 3)(1.0, 1.0, 1.0), 3, vp(phi),
                dbl(1e9), dbl(0.5), i64(50), ctypes.byref(info), vp())
            assert rc == 0 and info.steps == 50, L.hjw_last_error()
            lines = log()
            assert [r[0] for r in resident(lines)] == [count] and resident(lines)[0][4] == 0, (n, lines)
    """)


def test_a_launch_that_stopped_answering_reports_the_record_before_it():
    _run("""
        g = Grid((256, 256))
        rc, good = g.step(5)
        assert rc == 0
        S.stub_modes(b"2")
        assert g.step(40)[0] == EHIP
        info, taken = Info(), i64()
        assert L.hjw_get_info(g.h, ctypes.byref(info)) == 0
        assert L.hjw_resident_steps(g.h, ctypes.byref(taken)) == 0
        assert info.steps == good.steps == taken.value == 5 and info.t == good.t
    """)
