"""The host side of the library against a stand-in for the GPU in host memory
(host_device.hip): the work lists of a handle as its cavities retire and come
back, with device memory exhausted after creation, and what the autotuner
keeps.  Every launch, and every launch of a replayed graph, is checked against
the live allocations."""
import ctypes
import os
import random
import subprocess

import numpy as np
import pytest

import paper_2306_07603_amd as M
from paper_2306_07603_amd import _build

PRECISIONS = ["fp64", "fp32", "fp16dev", "fp32x", "fp32sr", "fp32srf"]
TOL = 1e-6


class Host:
    """api.hip on the stand-in: the C ABI, called as the binding calls it."""

    def __init__(self, path):
        self.L = L = ctypes.CDLL(path)
        L.ifdlbm_create.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_void_p, ctypes.POINTER(ctypes.c_void_p)]
        L.ifdlbm_step.argtypes = [ctypes.c_void_p, ctypes.c_int64]
        L.ifdlbm_run_to_steady.argtypes = [ctypes.c_void_p, ctypes.c_double, ctypes.c_int64] + [ctypes.c_void_p] * 3
        L.ifdlbm_get_residuals.argtypes = [ctypes.c_void_p] * 3
        L.ifdlbm_set_state.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p]
        L.ifdlbm_autotune.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.POINTER(ctypes.c_int32),
                                      ctypes.POINTER(ctypes.c_double)]
        L.ifdlbm_adjoint.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_int32,
                                     ctypes.c_void_p, ctypes.c_void_p]
        L.host_peak_bytes.restype = L.host_live_bytes.restype = ctypes.c_long
        L.ifdlbm_destroy.argtypes = [ctypes.c_void_p]
        L.ifdlbm_destroy.restype = None
        L.host_reset.argtypes = [ctypes.c_long, ctypes.c_long]
        L.host_reset.restype = None
        L.host_converge.argtypes = [ctypes.c_void_p, ctypes.c_int]
        L.host_converge.restype = None

    def create(self, sizes, **opt):
        self.L.host_reset(-1, -1)
        self.sizes = sizes
        arr = (M.ifdlbm.ifdlbm_cavity * len(sizes))(*[M.Cavity(a, b, 400.0, 0.8, 60.0).c() for a, b in sizes])
        o = M.ifdlbm_default_options(**opt)
        h = ctypes.c_void_p()
        assert self.L.ifdlbm_create(arr, len(sizes), ctypes.byref(o), ctypes.byref(h)) == 0
        return h

    def exhaust(self):
        """No device allocation succeeds from here on."""
        self.L.host_reset(0, -1)

    def converge(self, flags):
        a = np.ascontiguousarray(flags, dtype=np.int32)
        self.L.host_converge(a.ctypes.data, a.size)

    def restart(self, h, c):
        nx, ny = self.sizes[c]
        F, lam = np.zeros((9, ny, nx)), np.ones((ny, nx))
        return self.L.ifdlbm_set_state(h, c, F.ctypes.data, lam.ctypes.data)

    def faults(self):
        text = ctypes.create_string_buffer(200)
        n = self.L.host_faults(text, 200)
        return n, text.value.decode()

    def last_kernel(self):
        text = ctypes.create_string_buffer(20)
        self.L.host_last_kernel(text, 20)
        return text.value.decode()


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("host")
    objs = []
    for src in (os.path.join(_build.CSRC, "api.hip"), os.path.join(os.path.dirname(__file__), "host_device.hip")):
        objs.append(str(d / (os.path.basename(src) + ".o")))
        subprocess.run([_build.HIPCC, "--offload-host-only", "-x", "hip", "-O1", "-std=c++17", "-fPIC", "-I", _build.INCLUDE,
                        "-I", _build.CSRC, '-DIFD_SOURCE_DIGEST="host"', "-c", src, "-o", objs[-1]], check=True)
    lib = str(d / "libhost.so")
    # the stand-in's runtime, also where the process has loaded the GPU's
    subprocess.run(["g++", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-o", lib, *objs], check=True)
    return Host(lib)


# (batch, cavities left, kernel before, kernel after): the tiles of those left are more items than the march of all
RETIRE = [("fp32srf", 64, 15, (513, 513), "march", "tile"), ("fp64", 40, 10, (129, 129), "block", "tile")]


@pytest.mark.parametrize("case", RETIRE, ids=lambda c: c[0])
@pytest.mark.parametrize("graph", [0, 4])
def test_retirement_needs_no_memory(host, case, graph):
    precision, n, left, size, before, after = case
    h = host.create([size] * n, precision=precision, graph_steps=graph, residual_every=2)
    host.exhaust()
    host.converge([0] * n)
    assert host.L.ifdlbm_step(h, 8) == 0 and host.last_kernel() == before
    host.converge([0] * left + [1] * (n - left))
    assert host.L.ifdlbm_run_to_steady(h, TOL, 2, None, None, None) == M.IFDLBM_ENOTCONVERGED
    assert host.L.ifdlbm_step(h, 9) == 0 and host.last_kernel() == after
    assert host.faults() == (0, "")
    # and back: every cavity restarted
    for c in range(left, n):
        assert host.restart(h, c) == 0
    assert host.L.ifdlbm_step(h, 9) == 0 and host.last_kernel() == before
    assert host.faults() == (0, "")
    host.L.ifdlbm_destroy(h)


@pytest.mark.parametrize("batched", [1, 0])
@pytest.mark.parametrize("precision", PRECISIONS)
def test_lists_hold_any_running_set(host, precision, batched):
    """Batches of every size class, with random sets of cavities stopped and restarted."""
    rng = random.Random(7)
    for trial in range(12):
        count = rng.choice((1, 2, 7, 30, 120))
        side = rng.choice((5, 9, 25, 60, 130, 300, 700)) if count < 100 else rng.choice((5, 25, 60, 130))
        sizes = [(max(5, int(side * rng.uniform(0.4, 2.0))), max(5, int(side * rng.uniform(0.4, 2.0)))) for _ in range(count)]
        h = host.create(sizes, precision=precision, batched=batched, residual_every=1)
        host.exhaust()
        stopped = []
        for _ in range(4):
            flags = [int(rng.random() < 0.6) for _ in range(count)]
            host.converge(flags)
            rc = host.L.ifdlbm_run_to_steady(h, TOL, 1, None, None, None)
            assert rc in (M.IFDLBM_OK, M.IFDLBM_ENOTCONVERGED), (trial, rc)
            stopped = sorted(set(stopped) | {c for c in range(count) if flags[c]})
            host.converge([0] * count)
            assert host.L.ifdlbm_step(h, 2) == 0
            assert host.faults() == (0, ""), (trial, sizes[:3], count)
            for c in rng.sample(stopped, len(stopped) // 2):
                assert host.restart(h, c) == 0
                stopped.remove(c)
        host.L.ifdlbm_destroy(h)


@pytest.mark.parametrize("batched", [1, 0])
@pytest.mark.parametrize("precision", PRECISIONS)
def test_autotune_keeps_a_faster_automatic_choice(host, precision, batched):
    """Small cavities, on a stand-in whose tiles are faster than any march and whose fastest march has 40 rows to an item:
    the tuned handle steps on tiles, as the untuned one does, in one launch or one per cavity; the rows it reports are a
    length of the march, the fastest one, for another handle."""
    sizes = [(33, 240), (65, 240)]   # 6 segments at 40 rows, 5 at 48
    h = host.create(sizes, precision=precision, batched=batched)
    rows, ms = ctypes.c_int32(), ctypes.c_double()
    host.L.host_cheap_rows(40)
    assert host.L.ifdlbm_autotune(h, 3, ctypes.byref(rows), ctypes.byref(ms)) == 0
    assert host.L.ifdlbm_step(h, 1) == 0 and host.last_kernel() == "tile"
    assert host.faults() == (0, "")
    host.L.ifdlbm_destroy(h)
    assert rows.value == 40 and ms.value == (1.0 if batched else 2.0)
    h = host.create(sizes, precision=precision, batched=batched, segment_rows=rows.value)
    assert host.L.ifdlbm_step(h, 1) == 0 and host.last_kernel() == ("block" if precision in ("fp64", "fp32x", "fp32sr") else "march")
    host.L.ifdlbm_destroy(h)


def test_residuals_without_pinned_memory(host):
    """Where no host memory can be pinned, residuals are read into pageable memory, and the steps after go on."""
    h = host.create([(33, 33)] * 3)
    host.L.host_reset(-1, 0)
    host.converge([0, 1, 0])
    assert host.L.ifdlbm_step(h, 1) == 0
    res = np.zeros(3)
    for _ in range(2):
        assert host.L.ifdlbm_get_residuals(h, res.ctypes.data, None) == 0
        assert list(res) == [1.0, 0.0, 1.0]
        assert host.L.ifdlbm_step(h, 1) == 0
    assert host.faults() == (0, "")
    host.L.ifdlbm_destroy(h)


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("size", [(17, 400), (129, 129), (16, 64)])
def test_adjoint_memory(host, size, precision):
    """A trajectory takes no more device memory than one FP64 value per population and node and step, whatever the pitch:
    the states of a segment and the checkpoints (100 steps in segments of 50), and at most 60 doubles per node of work
    arrays and two padded states of the handle beside its scratch and lists."""
    nx, ny = size
    nodes, padded = nx * ny, -(-nx // 16) * 16 * ny
    J, grad = np.zeros(1), np.zeros(3)
    cav, o = M.Cavity(nx, ny, 400.0, 0.8, 60.0).c(), M.ifdlbm_default_options(precision=precision)
    host.L.host_reset(-1, -1)
    before = host.L.host_live_bytes()
    assert host.L.ifdlbm_adjoint(ctypes.byref(cav), ctypes.byref(o), 100, 50, 0, J.ctypes.data, grad.ctypes.data) == 0
    peak = host.L.host_peak_bytes() - before
    limit = 80 * nodes * (50 + 1) + 2 * 80 * padded + 60 * 8 * nodes + 2 * 80 * padded + 80 * nodes + 300 * nodes // 8 + 100000
    print(size, precision, peak, limit)
    assert peak <= limit
    assert host.L.host_live_bytes() == before and host.faults() == (0, "")
