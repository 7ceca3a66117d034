"""The library's host code on the stand-in runtime (hip_stub.hip), without a GPU: run in a process
of its own, so that libhjw.so binds to it.  Test support."""
import ctypes
import os
import re

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))

S = ctypes.CDLL(os.path.join(HERE, "libhip_stub.so"), mode=ctypes.RTLD_GLOBAL)
L = ctypes.CDLL(os.environ.get("HJW_HOST_TEST_LIB") or
                os.path.join(ROOT, "paper_1909_13263_amd", "libhjw.so"))
vp, i64, dbl = ctypes.c_void_p, ctypes.c_int64, ctypes.c_double
S.stub_log.restype = ctypes.c_char_p
S.stub_malloc.restype = vp
S.stub_malloc.argtypes = [ctypes.c_size_t, ctypes.c_int]
HOOK = ctypes.CFUNCTYPE(None)
L.hjw_step_to.argtypes = [vp, dbl, dbl, i64, vp]
L.hjw_set_option.argtypes = [vp, ctypes.c_int, i64]
L.hjw_bind.argtypes = [vp, vp, ctypes.c_size_t, vp]
L.hjw_set_phi.argtypes = [vp, vp, ctypes.c_int]
L.hjw_grid_destroy.argtypes = [vp]
L.hjw_last_error.restype = ctypes.c_char_p
FP64, FP32_MIXED, FP32 = 0, 1, 2
STEP = 1.0 / 1024   # the stub's time step
EHIP = -3


def setup(devices=2, cus=256, per_cu=4):
    S.stub_setup(devices, cus, per_cu)


def log():
    """The launches since the last call, and forget them."""
    out = S.stub_log().decode().splitlines()
    S.stub_clear_log()
    return out


def resident(lines):
    """[(workgroups, threads, first tag, most steps, device of the mailboxes)]."""
    out = []
    for line in lines:
        m = re.match(r"resident count=(\d+) block=(\d+) epoch=(\d+) steps=(\d+) mail_device=(-?\d+)", line)
        if m:
            out.append(tuple(int(v) for v in m.groups()))
    return out


def staged(lines):
    """Steps taken by launches per stage."""
    return sum(line.startswith("step ") for line in lines)


class Info(ctypes.Structure):
    _fields_ = [("steps", i64), ("t", dbl), ("dt", dbl), ("ax", dbl), ("ay", dbl),
                ("range", dbl * 4)]


class Grid:
    def __init__(self, shape, prec=FP32_MIXED, device=0):
        dim = len(shape)
        self.h = vp()
        rc = L.hjw_grid_create(dim, (i64 * dim)(*shape[::-1]), (dbl * dim)(*[0.0] * dim),
                               (dbl * dim)(*[1.0] * dim), (ctypes.c_int * dim)(*[0] * dim), prec,
                               ctypes.byref(self.h))
        assert rc == 0
        nb = ctypes.c_size_t()
        assert L.hjw_workspace_bytes(self.h, ctypes.byref(nb)) == 0
        self.bytes = nb.value
        self.phi = (dbl * (shape[0] * (shape[1] if dim == 2 else 1)))()
        self.bind(device)
        assert L.hjw_set_hamiltonian(self.h, 1, (dbl * 3)(1.0, 1.0, 1.0), 3) == 0
        self.set_phi()

    def bind(self, device=0):
        assert S.hipSetDevice(device) == 0
        assert L.hjw_bind(self.h, S.stub_malloc(self.bytes, device), self.bytes, None) == 0

    def set_phi(self):
        assert L.hjw_set_phi(self.h, self.phi, 0) == 0

    def step(self, n=0, t=1e9):
        """(status, info) of hjw_step_to over n steps."""
        info = Info()
        rc = L.hjw_step_to(self.h, t, 0.5, n, ctypes.byref(info))
        return rc, info

    def option(self, o, v):
        return L.hjw_set_option(self.h, o, v)

    def close(self):
        L.hjw_grid_destroy(self.h)
