"""The library's host code against a stand-in for the HIP runtime (tests/stub).
uad_set_prefix_kv: which sources are read in place, what is refused before
anything is written, and what an error on the way leaves behind.  Steps: what is
refused before any work is enqueued, and the memory that the adaptive norms keep."""
import concurrent.futures as cf
import ctypes
import os
import subprocess

import numpy as np
import pytest

import paper_2609_37772_amd as U

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
OK, STATE, HIP = 0, 3, 5
L, B, P, HKV, HD = 2, 2, 70, 2, 64
BYTES = L * B * P * HKV * HD * 4


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = str(tmp_path_factory.mktemp("stub"))
    srcs = [os.path.join(ROOT, p) for p in ("paper_2609_37772_amd/csrc/uad_api.cpp",
                                            "paper_2609_37772_amd/csrc/schedule.cpp", "tests/stub/hip_stub.cpp")]

    def compile_one(src):
        obj = os.path.join(d, os.path.basename(src) + ".o")
        subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-fPIC", "-std=c++17",
                        "-c", src, "-o", obj], check=True)
        return obj
    with cf.ThreadPoolExecutor(3) as ex:
        objs = list(ex.map(compile_one, srcs))
    # the device code that host-only objects refer to does not exist
    names = subprocess.run(["nm", "-u", *objs], capture_output=True, text=True, check=True).stdout.split()
    fat = ["-Wl,--defsym,%s=0" % n for n in names if n.startswith("__hip_fatbin")]
    so = os.path.join(d, "libstub.so")
    subprocess.run(["g++", "-shared", "-o", so, *objs, "-Wl,-z,defs", "-Wl,-Bsymbolic", *fat], check=True)
    lib = ctypes.CDLL(so)
    lib.stub_log.restype = lib.uad_last_error.restype = ctypes.c_char_p
    lib.stub_shift_bytes.restype = lib.stub_shift_end.restype = ctypes.c_size_t
    lib.stub_map.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
    return lib


def create(lib, batch=B, chunk=8, flags=0):
    cfg = U._binding.uad_model_config(L, 128, 2, HKV, HD, 256, 7, batch, chunk, P + 10, 1e-6, flags)
    c = ctypes.c_void_p()
    assert lib.uad_create(ctypes.byref(cfg), 0, None, ctypes.byref(c)) == OK
    return c


@pytest.fixture
def ctx(lib):
    c = create(lib)
    yield c
    lib.uad_destroy(c)


class Memory:
    """`n` bytes in the middle of nothing: the runtime knows only what was mapped."""

    def __init__(self, lib, n):
        self.lib, self.a, self.maps = lib, np.zeros(n, np.uint8), []
        self.p = self.a.ctypes.data

    def map(self, at, n):
        self.lib.stub_map(self.p + at, n)
        self.maps.append(self.p + at)
        return self

    def unmap(self):
        for p in self.maps:
            self.lib.stub_map(p, 0)


def set_prefix(lib, c, k, v, on_device, fail_in=-1):
    lib.stub_reset(fail_in)
    st = lib.uad_set_prefix_kv(c, ctypes.c_void_p(k), ctypes.c_void_p(v), 0, B, P, on_device)
    return st, lib.stub_log().decode().split()


@pytest.mark.parametrize("pieces", [[BYTES], [BYTES + 100], [4096, BYTES - 4096], [BYTES // 2, 64, BYTES]])
def test_covered_device_source_is_read_in_place(lib, ctx, pieces):
    k, v = Memory(lib, BYTES + 8192), Memory(lib, 3 * BYTES)
    k.map(0, BYTES)
    at = 0
    for n in pieces:
        v.map(at, n)
        at += n
    st, log = set_prefix(lib, ctx, k.p, v.p, 1)
    assert st == OK and "copy" not in log and log.count("pack") == 1
    k.unmap(), v.unmap()


@pytest.mark.parametrize("short", [1, 4, BYTES // 2 + 4, BYTES // L])
def test_device_source_shorter_than_the_prefix_is_refused(lib, ctx, short):
    """The device kernel would read past the allocation; the copies that it took
    the place of were refused."""
    k, v = Memory(lib, BYTES).map(0, BYTES), Memory(lib, BYTES).map(0, BYTES - short)
    for pair in ((k.p, v.p), (v.p, k.p)):
        st, log = set_prefix(lib, ctx, *pair, 1)
        assert st == HIP and not {"copy", "pack"} & set(log)
    k.unmap(), v.unmap()


@pytest.mark.parametrize("on_device,fail_in", [(0, 0), (0, 1), (0, 2), (0, 4), (1, 0)])
def test_error_on_the_way_waits_and_leaves_no_prefix(lib, ctx, on_device, fail_in):
    """An error after copies or kernels were queued: they still use the caller's
    memory until the wait, and the stores hold parts of two prefixes."""
    k, v = Memory(lib, BYTES), Memory(lib, BYTES)
    if on_device:
        k.map(0, BYTES), v.map(0, BYTES)
    assert set_prefix(lib, ctx, k.p, v.p, on_device)[0] == OK
    st, log = set_prefix(lib, ctx, k.p, v.p, on_device, fail_in)
    assert st == HIP and log[-1] == "sync" and len(log) == fail_in + 3  # the stream's wait, the calls, the wait
    assert b"stub error" in lib.uad_last_error(ctx)
    assert lib.stub_prefix_set(ctx) == 0
    assert set_prefix(lib, ctx, k.p, v.p, on_device)[0] == OK and lib.stub_prefix_set(ctx) == 1
    k.unmap(), v.unmap()


@pytest.mark.parametrize("batch,chunk", [(3, 8), (20, 16)])  # below and from the row count of the by-class norms
def test_compacted_adaptive_norm_step_is_refused_before_any_work(lib, batch, chunk):
    c = create(lib, batch, chunk, flags=1)
    lib.stub_ready(c)
    x, bud = np.zeros((batch, chunk, 7), np.float32), np.full((batch, chunk), 2, np.int32)
    args = (c, ctypes.c_void_p(x.ctypes.data), ctypes.c_void_p(bud.ctypes.data), batch, chunk, None, None, None)
    assert lib.uad_denoise_budgets(*args) == OK  # every environment at every step
    lib.stub_set_active(c, 0, batch - 1)
    lib.stub_reset(-1)
    assert lib.uad_denoise_budgets(*args) == STATE
    assert lib.stub_log() == b""
    lib.uad_destroy(c)


@pytest.mark.parametrize("batch,chunk,by_token", [(1, 9, True), (15, 17, True), (16, 16, True), (17, 16, False),
                                                  (64, 50, False)])
def test_shift_operands_are_kept_for_steps_by_token_only(lib, batch, chunk, by_token):
    """They take rows up to 256: larger steps go by flow-time class without them."""
    c = create(lib, batch, chunk, flags=1)
    lib.stub_ready(c)
    lib.stub_reset(-1)
    x = np.zeros((batch, chunk, 7), np.float32)
    p = ctypes.c_void_p(x.ctypes.data)
    assert lib.uad_denoise_step(c, p, p, p, p, None, batch, chunk) == OK
    M, row = batch * chunk, 128 * 2
    kept = min((M + 63) // 64 * 64, 256)
    assert lib.stub_shift_bytes(c) == 2 * L * kept * row
    assert lib.stub_shift_end(c) == (((2 * L - 1) * kept + (M + 15) // 16 * 16) * row if by_token else 0)
    lib.uad_destroy(c)
