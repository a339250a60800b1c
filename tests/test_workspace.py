"""Growth of the device workspace on the host: bellman_api.cpp linked with an
allocator of limited memory (tests/native/workspace_shim.cpp).  A block is
taken with room to grow; where that cannot be had, one of the call's own size
must do, prompt attention runs with its keys uncut where the cut's pieces do
not fit, and only a call that does not fit at all is refused."""
from __future__ import annotations

import ctypes
import os
import subprocess

import pytest

from paper_2510_15330_amd import _binding as b

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MIB = 1 << 20
OK, OOM = 0, -4


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("workspace") / "libws.so")
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    subprocess.check_call([hipcc, "-x", "hip", "--offload-host-only", "-no-hip-rt", "-O1", "-std=c++17", "-shared",
                           "-fPIC", os.path.join(ROOT, "tests", "native", "workspace_shim.cpp"),
                           os.path.join(ROOT, "paper_2510_15330_amd", "csrc", "bellman_api.cpp"), "-o", out,
                           "-Wl,-z,lazy", "-Wl,-Bsymbolic"])
    L = ctypes.CDLL(out, mode=os.RTLD_LAZY)
    L.ws_device.argtypes = [ctypes.c_size_t]
    L.ws_device.restype = None
    L.bellman_reserve_workspace.argtypes = [ctypes.c_int64]
    L.bellman_last_error.restype = ctypes.c_char_p
    return L


def _asked(lib):
    sizes = (ctypes.c_size_t * 8)()
    n = lib.ws_calls(sizes)
    return list(sizes[:n])


@pytest.mark.parametrize("mib", [1, 3, 100, 300, 2000])
def test_reservation_near_a_full_device(lib, mib):
    need = mib * MIB - 5
    # all the memory there is: some room to grow
    lib.bellman_shutdown()
    lib.ws_device(1 << 40)
    assert lib.bellman_reserve_workspace(need) == OK
    room, = _asked(lib)
    assert need * 5 // 4 <= room <= max(4 * need, need + need // 4) + MIB
    # no room to grow: the size asked for, to the next MiB
    lib.bellman_shutdown()
    lib.ws_device(mib * MIB)
    assert lib.bellman_reserve_workspace(need) == OK, lib.bellman_last_error()
    assert _asked(lib) == [room, mib * MIB]
    assert lib.bellman_reserve_workspace(need) == OK and _asked(lib) == []
    assert lib.bellman_reserve_workspace(mib * MIB) == OK and _asked(lib) == []
    # not even that: refused
    lib.bellman_shutdown()
    lib.ws_device(mib * MIB - 1)
    assert lib.bellman_reserve_workspace(need) == OOM
    assert b"hipMalloc" in lib.bellman_last_error()
    lib.bellman_shutdown()


def _desc(dtype, *shape):
    d = b.Tensor()
    d.data, d.dtype, d.ndim = 1 << 20, dtype, len(shape)     # (an address that nothing reads)
    stride = 1
    for i in reversed(range(len(shape))):
        d.shape[i], d.stride[i] = shape[i], stride
        stride *= shape[i]
    return d


def test_prompt_attention_near_a_full_device(lib):
    # one 512-token chunk of 4/2 heads over 2000 cached ones: 16 tiles + 2 of
    # 128 rows, cut into 512 units of 128 (4 D + 8) bytes
    T, H_q, H_kv, D, maxP, NP = 512, 4, 2, 128, 160, 200
    steps = maxP // 4
    uncut = 256 + 256 + 256 * -(-4 * steps * H_kv // 256) + steps * H_kv * 128 * D
    pieces = 512 * 128 * (4 * D + 8)

    def call():
        return lib.bellman_prefill_attention(
            ctypes.byref(_desc(b.BF16, T, H_q, D)), ctypes.byref(_desc(b.BF16, NP, H_kv, D // 8, 16, 8)),
            ctypes.byref(_desc(b.BF16, NP, H_kv, D, 16)), ctypes.byref(_desc(b.INT32, 1, maxP)),
            ctypes.byref(_desc(b.INT32, 1)), ctypes.byref(_desc(b.INT32, 2)), ctypes.c_float(0.1),
            ctypes.byref(_desc(b.BF16, T, H_q, D)), None)

    for limit, rc, split in ((1 << 40, OK, 1), (uncut + pieces + 4 * MIB, OK, 1), (uncut + 4 * MIB, OK, 0),
                             (uncut - MIB, OOM, -1)):
        lib.bellman_shutdown()
        lib.ws_device(limit)
        assert call() == rc, (limit, lib.bellman_last_error())
        assert lib.ws_split() == split, limit
    lib.bellman_shutdown()
