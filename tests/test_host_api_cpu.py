"""The host side of the library (csrc/lbm_api.cpp) without a GPU: built with tests/hip_stub.cpp, whose
HIP calls and launchers only keep a log."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads
from paper_1708_07525_amd.lbm import OK, Obs, make_params

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
VP, D = ctypes.c_void_p, ctypes.POINTER(ctypes.c_double)


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("host") / "libhost.so")
    csrc = os.path.join(ROOT, "paper_1708_07525_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-w", "-pthread",
                    "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(csrc, "lbm_api.cpp"), os.path.join(HERE, "hip_stub.cpp"), "-Wl,-z,defs", "-o", so],
                   check=True)
    lib = ctypes.CDLL(so)
    lib.lbm_create.argtypes = [VP, ctypes.POINTER(VP)]
    lib.lbm_set_fields.argtypes = [VP, D, D, D, D, D]
    lib.lbm_step.argtypes = [VP, ctypes.c_int64]
    lib.lbm_observables.argtypes = [VP, VP, D]
    lib.lbm_observables_static.argtypes = [VP, VP, D]
    lib.lbm_get_fields.argtypes = [VP, D]
    lib.lbm_destroy.argtypes = [VP]
    lib.lbm_destroy.restype = None
    lib.stub_calls.argtypes = [ctypes.c_char_p]
    lib.stub_calls.restype = ctypes.c_longlong
    lib.stub_fail.argtypes = [ctypes.c_char_p, ctypes.c_int]
    lib.stub_launches.restype = ctypes.c_char_p
    return lib


@pytest.fixture()
def lib(built):
    built.stub_reset()
    return built


class Context:
    """A context of the stub library; ready: with its initial fields."""

    def __init__(self, lib, nx, ny, prec="fp32", ready=False, **kw):
        self.lib, self.nx, self.ny, self.h = lib, nx, ny, VP()
        p = make_params(workloads.cavity_params(nx=nx, ny=ny, **kw), prec)
        assert lib.lbm_create(ctypes.byref(p), ctypes.byref(self.h)) == OK
        if ready:
            assert lib.lbm_set_fields(self.h, None, None, None, None, None) == OK

    def fields(self):
        f = np.empty((5, self.ny, self.nx))
        return self.lib.lbm_get_fields(self.h, f.ctypes.data_as(D))

    def look(self, fields=False, static=False):
        f = np.empty((5, self.ny, self.nx)) if fields else None
        o = Obs()
        fn = self.lib.lbm_observables_static if static else self.lib.lbm_observables
        return fn(self.h, ctypes.byref(o), f.ctypes.data_as(D) if fields else None)

    def close(self):
        self.lib.lbm_destroy(self.h)


@pytest.mark.parametrize("n,call", [(200, b"hipMalloc"), (200, b"launch_export"), (64, b"launch_observables")])
def test_a_failed_look_leaves_nothing_in_flight(lib, n, call):
    """The observables' kernels write into the context's pinned block, which goes to another context
    once this one is destroyed: a look that fails after their launch waits for them."""
    c = Context(lib, n, n, ready=True)
    lib.lbm_step(c.h, 3)
    lib.stub_fail(call, 1)
    assert c.look(fields=True) != OK
    assert lib.stub_pending() == 0
    assert c.look(fields=True) == OK
    c.close()


NODE = ("nee_hot", "nee_robin", "nee_adiabatic", "nee_cold")


@pytest.mark.parametrize("nx,ny,prec", [(128, 7200, "fp32"), (135, 7300, "fp32"), (139, 7194, "fp32")])
def test_one_launch_in_effect(lib, nx, ny, prec):
    """Narrow lattices between node walls that the region launch's rule and the march's both take: one
    of the two is in effect, for the getters, plain launches and graph replays alike."""
    c = Context(lib, nx, ny, prec, ready=True, sides=NODE, Bi_T=1.0, Bi_C=1.0)
    region, march = lib.lbm_get_region_steps(c.h), lib.lbm_get_march_steps(c.h)
    assert region == 0 or march == 0
    lib.stub_reset()
    assert lib.lbm_step(c.h, 64 + 12) == OK     # a replay (what it leaves of 64) and plain launches
    log = lib.stub_launches().decode().split()
    assert log.index("]") > 1
    for k in log:
        if k not in ("[", "]", "graph"):
            assert k.startswith("region" if region else ("march", "packed") if march else "step"), log
            if region:
                assert int(k.split("/")[1]) <= region, log
    c.close()


def test_pinned_memory_is_for_contexts_that_look_often(lib):
    """One context at a time: creating, stepping, three looks and destroying allocate no pinned memory;
    the fourth look does.  Others take what lies idle, and the last one gives everything back."""
    for _ in range(2):
        c = Context(lib, 64, 64, ready=True)
        for fields in (False, True, False):
            assert c.look(fields=fields) == OK
        c.close()
    assert lib.stub_calls(b"hipHostMalloc") == 0 and lib.stub_calls(b"hipHostFree") == 0
    c = Context(lib, 64, 64, ready=True)
    for _ in range(4):
        assert c.look(fields=True) == OK
    assert lib.stub_calls(b"hipHostMalloc") == 1
    d = Context(lib, 60, 60, ready=True)        # of the same size class: its first look finds an idle block
    mallocs, copies = lib.stub_calls(b"hipMalloc"), lib.stub_calls(b"hipMemcpyAsync")
    assert d.look(fields=True) == OK
    assert lib.stub_calls(b"hipMalloc") == mallocs and lib.stub_calls(b"hipMemcpyAsync") == copies
    assert lib.stub_calls(b"hipHostMalloc") == 1
    c.close()
    assert lib.stub_calls(b"hipHostFree") == 0
    d.close()
    assert lib.stub_calls(b"hipHostFree") == 1


def test_contexts_share_what_they_have_gone_without(lib):
    """The looks and exports of contexts that live together add up: a block is theirs in turn."""
    c = [Context(lib, 64, 64, ready=True) for _ in range(5)] + [Context(lib, 512, 512, ready=True) for _ in range(4)]
    for k, x in enumerate(c[:5]):
        assert x.look() == OK and lib.stub_calls(b"hipHostMalloc") == (k >= 3)
    for k, x in enumerate(c[5:]):
        assert x.fields() == OK and lib.stub_calls(b"hipHostMalloc") == 1 + (k >= 3)
    for x in c:
        x.close()
    assert lib.stub_calls(b"hipHostFree") == 2
    d = Context(lib, 64, 64, ready=True)        # alone again: the count starts anew
    assert d.look() == OK and lib.stub_calls(b"hipHostMalloc") == 2
    d.close()


def test_static_looks_allocate_nothing(lib):
    c = Context(lib, 64, 64, ready=True)
    lib.stub_reset()
    for _ in range(8):
        assert c.look(fields=True, static=True) == OK
    assert lib.stub_calls(b"hipHostMalloc") == 0 and lib.stub_calls(b"hipMalloc") == 0
    c.close()


def test_looks_without_pinned_memory(lib):
    """No pinned memory to be had: looks and exports take the way through device memory."""
    lib.stub_fail(b"hipHostMalloc", 1000)
    c, big = Context(lib, 64, 64, ready=True), Context(lib, 520, 500, ready=True)
    for _ in range(6):
        assert c.look(fields=True) == OK and c.fields() == OK and big.look(fields=True) == OK and big.fields() == OK
    c.close()
    big.close()


def test_exports_allocate_their_block_once_it_pays(lib):
    """512 x 512 fields (10.5 MB): through device memory until 40 MB have been exported; an idle
    block is taken at once."""
    c = Context(lib, 512, 512, ready=True)
    for k in range(4):
        assert lib.stub_calls(b"hipHostMalloc") == 0
        assert c.fields() == OK
    assert lib.stub_calls(b"hipHostMalloc") == 1
    d = Context(lib, 300, 400, ready=True)
    mallocs = lib.stub_calls(b"hipMalloc")
    assert d.fields() == OK
    assert lib.stub_calls(b"hipMalloc") == mallocs and lib.stub_calls(b"hipHostMalloc") == 1
    c.close()
    d.close()


@pytest.mark.parametrize("nx,ny,blocks", [(52429, 21, 1), (60000, 20, 1), (200000, 6, 1), (250000, 5, 0)])
def test_exports_of_wide_rows_keep_their_block(lib, nx, ny, blocks):
    """Rows above 2 MB: the slots fit the block that the pool keeps, which a second export finds idle; rows
    above 8 MB go through device memory."""
    c = Context(lib, nx, ny, ready=True)
    lib.stub_reset()
    for _ in range(3):
        assert c.fields() == OK
    assert lib.stub_calls(b"hipHostMalloc") == blocks
    assert lib.stub_calls(b"pinned bytes") == blocks * (16 << 20)
    c.close()


@pytest.mark.parametrize("n,threads", [(256, 2), (400, 6), (512, 8)])
def test_exports_start_a_thread_per_mb(lib, n, threads):
    """256 x 256 fields are 2.6 MB: five threads cost more to start than they save."""
    keep, c = Context(lib, 1100, 1000, ready=True), Context(lib, n, n, ready=True)
    assert keep.fields() == OK                  # leaves an idle block
    lib.stub_reset()
    assert c.fields() == OK
    assert lib.stub_calls(b"hipMalloc") == 0
    assert lib.stub_calls(b"hipSetDevice") == min(threads, len(os.sched_getaffinity(0)))
    c.close()
    keep.close()


HALF = ("hot", "cold", "adiabatic", "adiabatic")


@pytest.mark.parametrize("prec,sides,nx,ny,launch", [
    ("fp32", HALF, 2048, 2048, "march/19"), ("fp64", HALF, 2048, 2048, "march/37"),
    ("fp32", NODE, 2048, 2048, "march/19"),
    ("fp32", HALF, 128, 8000, "step3"), ("fp32", HALF, 128, 20000, "step3"), ("fp32", HALF, 233, 4200, "step3"),
    ("fp32", HALF, 233, 9000, "packed/11"), ("fp32", HALF, 300, 4200, "step3"), ("fp32", HALF, 300, 6007, "packed/9"),
    ("fp32", HALF, 465, 3000, "step3"), ("fp32", HALF, 1100, 1600, "march/8"), ("fp32", HALF, 180, 30000, "march/30"),
    ("fp64", HALF, 128, 20000, "step3"), ("fp64", HALF, 233, 9000, "step3"), ("fp64", HALF, 300, 4200, "step3"),
    ("fp64", HALF, 465, 3000, "step3"), ("fp64", HALF, 233, 30000, "packed/74"), ("fp64", HALF, 1000, 1000, "packed/9"),
    ("fp64", HALF, 200, 5001, "march/10"), ("fp32", NODE, 300, 4200, "step2"), ("fp32", NODE, 300, 6007, "packed/9"),
    ("fp32", NODE, 760, 2000, "march/8"), ("fp64", NODE, 465, 3000, "packed/14"),
    ("fp32", HALF, 140, 8000, "step3"), ("fp32", HALF, 140, 11000, "march/11"), ("fp64", HALF, 64000, 200, "march/40"),
    ("fp32", HALF, 125000, 100, "march/20"), ("fp64", HALF, 100000, 128, "march/128"),
    ("fp64", NODE, 20000, 100, "march/14"), ("fp32", NODE, 20000, 100, "march/10"), ("fp64", NODE, 64000, 64, "step2")])
def test_march_where_its_strips_are_filled(lib, prec, sides, nx, ny, launch):
    """Lattices of few columns or few rows: the march only where its strips, its work-groups and the chip's
    slots are filled."""
    c = Context(lib, nx, ny, prec, ready=True, sides=sides, Bi_T=1.0, Bi_C=1.0)
    lib.stub_reset()
    assert lib.lbm_step(c.h, 4 if launch[0] in "mp" else int(launch[-1])) == OK
    assert lib.stub_launches().decode().split() == [launch]
    assert (lib.lbm_get_march_steps(c.h) == 4) == (launch[0] in "mp")
    c.close()


@pytest.mark.parametrize("prec,sides,nx,ny,steps", [
    ("fp32", HALF, 384, 384, 3), ("fp32", HALF, 400, 400, 3), ("fp32", HALF, 8000, 20, 3), ("fp32", HALF, 12000, 13, 0),
    ("fp32", HALF, 50000, 3, 0), ("fp32", HALF, 3, 50000, 3), ("fp32", HALF, 4000, 13, 4), ("fp32", HALF, 10000, 5, 3),
    ("fp16s", HALF, 8000, 20, 0), ("fp16s", HALF, 64, 2500, 3), ("fp16s", HALF, 400, 400, 3), ("fp64", HALF, 400, 400, 0),
    ("fp64", HALF, 380, 380, 3), ("fp64", HALF, 340, 340, 0), ("fp64", HALF, 100, 1600, 3), ("fp64", HALF, 12000, 13, 0),
    ("fp32", NODE, 20000, 24, 0), ("fp32", NODE, 24, 20000, 3), ("fp32", NODE, 6000, 30, 3), ("fp32", NODE, 700, 690, 3),
    ("fp32", NODE, 128, 4000, 0), ("fp16s", NODE, 20000, 24, 0), ("fp16s", NODE, 2000, 200, 3),
    ("fp16s", NODE, 3000, 24, 3)])
def test_region_launch_where_its_regions_are_filled(lib, prec, sides, nx, ny, steps):
    """Low and narrow lattices: several regions per CU only where they are not many more than the tiles."""
    c = Context(lib, nx, ny, prec, ready=True, sides=sides, Bi_T=1.0, Bi_C=1.0)
    assert lib.lbm_get_region_steps(c.h) == steps
    c.close()


def test_no_memory_while_a_batch_is_captured(lib):
    """A batch whose capture finds no host memory: an error, the capture ended, and the next call works."""
    lib.lbm_batch_create.argtypes = [ctypes.c_int32, ctypes.c_int32, VP, ctypes.POINTER(VP)]
    lib.lbm_batch_attach.argtypes = [VP, VP]
    lib.lbm_batch_step.argtypes = [VP, ctypes.c_int64]
    lib.lbm_batch_destroy.argtypes = [VP]
    c, b = Context(lib, 64, 64, ready=True), VP()
    assert lib.lbm_batch_create(4, 24, None, ctypes.byref(b)) == OK
    assert lib.lbm_batch_attach(b, c.h) == OK
    lib.stub_new_fails(1)
    assert lib.lbm_batch_step(b, 24) != OK
    lib.stub_new_fails(0)
    assert not lib.stub_in_capture()
    assert lib.lbm_batch_step(b, 24) == OK
    lib.lbm_batch_destroy(b)
    c.close()
