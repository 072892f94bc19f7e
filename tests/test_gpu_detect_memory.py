"""Detection of long texts into managed and pinned host memory.

Sequences of more than 64 chunks are split over several workgroups, whose counts meet in the
sequence's z slot by 64-bit atomic adds.  The outputs may be any memory the device can write:
device memory, hipMallocManaged, hipHostMalloc.  Each kind in turn for all three outputs,
through the C ABI, twice over the same buffers, against the oracle.
"""
import ctypes
import os

import numpy as np
import pytest

import oracle
from test_gpu_detect_ex import assert_ex_equal
from test_gpu_parity import WIDE, env, say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hip(env):
    """The HIP runtime that torch and libsbw already use."""
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64.so" in line)
    return ctypes.CDLL(os.path.realpath(path))


@pytest.mark.parametrize("kind", ["managed", "pinned"])
@pytest.mark.parametrize("seeding,width", [("context", 1), ("self_salt", 4)])
def test_outputs_in_host_visible_memory(env, hip, kind, seeding, width):
    torch, sbw, dev = env
    N, L = 5, 20011                                   # split over several workgroups
    rng = np.random.default_rng(31 + width)
    tok = rng.integers(0, 128256, (N, L)).astype(np.int32)
    lengths = np.array([L, width, 16384, 9000, 0], dtype=np.int32)
    t, lens = torch.from_numpy(tok).to(dev), torch.from_numpy(lengths).to(dev)
    expect = oracle.detect_ex(tok, width, WIDE, 0.25, seeding, lengths=lengths)
    bytes_ = 16 * N                                   # z, then counts, then scored
    base = ctypes.c_void_p()
    allocate = hip.hipMallocManaged if kind == "managed" else hip.hipHostMalloc
    assert allocate(ctypes.byref(base), ctypes.c_size_t(bytes_),
                    ctypes.c_uint(1 if kind == "managed" else 0)) == 0
    try:
        host = (ctypes.c_char * bytes_).from_address(base.value)
        z = np.frombuffer(host, dtype=np.float64, count=N)
        counts = np.frombuffer(host, dtype=np.int32, count=N, offset=8 * N)
        scored = np.frombuffer(host, dtype=np.int32, count=N, offset=12 * N)
        say(f"detect into {kind} memory {seeding} h={width}")
        for _ in range(2):
            status = sbw.raw().sbw_detect_ex(
                t.data_ptr(), N, L, L, lens.data_ptr(), width, WIDE, 0.25,
                sbw.SEED_CONTEXT if seeding == "context" else sbw.SEED_SELF_SALT, 0,
                base.value + 8 * N, base.value + 12 * N, base.value,
                torch.cuda.current_stream().cuda_stream)
            assert status == 0
            torch.cuda.synchronize()
            assert_ex_equal((counts.copy(), scored.copy(), z.copy()), expect, f"{kind} {seeding}/{width}")
    finally:
        torch.cuda.synchronize()
        (hip.hipFree if kind == "managed" else hip.hipHostFree)(base)
