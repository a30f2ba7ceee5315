"""Reductions and CU copies beside a kernel that holds most of the LDS.

A bounded spin kernel (tests/native/occupy.hip) keeps two blocks of one wave
and 64 KiB of LDS on every CU of its stream, which leaves 30 KiB of 160 and
nearly all wave slots.  A launch that asks for no LDS finishes beside it; one
that asks for 40 KiB or more starts only when the spin ends.  Large all-reduces
of three to five ranks and wide gathers ask for LDS where they have the whole
chip and choose their own workgroups; everything else must not."""
import ctypes
import os
import time
import types

import numpy as np
import pytest
import torch

import oracle
import paper_2609_34334_amd as hc
import workloads as W
from gpu_util import assert_bitwise, from_dev, to_dev

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
SPIN_MS = 40.0
HIP = ctypes.CDLL("libamdhip64.so.7")          # the HIP runtime torch has loaded
_SPIN = {}


@pytest.fixture(autouse=True)
def _fresh_config():
    saved = hc.get_config()
    yield
    hc.set_config(**saved)


def masked(cus):
    """A stream on the first `cus` CUs with a hardware queue of its own."""
    h = ctypes.c_void_p()
    words = [0xFFFFFFFF if 32 * (i + 1) <= cus else 0 for i in range(8)]
    assert HIP.hipExtStreamCreateWithCUMask(ctypes.byref(h), 8, (ctypes.c_uint32 * 8)(*words)) == 0
    return torch.cuda.ExternalStream(h.value)


def spin(cus):
    if "lib" not in _SPIN:
        lib = ctypes.CDLL(os.path.join(HERE, "native", "liboccupy.so"))
        lib.occupy_lds_launch.argtypes = [ctypes.c_int, ctypes.c_uint64, ctypes.c_uint, ctypes.c_void_p]
        _SPIN["lib"] = lib
    if cus not in _SPIN:
        _SPIN[cus] = (masked(cus), masked(cus))
    return _SPIN["lib"], *_SPIN[cus]


def ends_beside_the_spin(run, cus=256):
    """Milliseconds from the spin's start to the end of `run`, issued 5 ms
    into it on a stream of the same CUs."""
    lib, hold, s = spin(cus)
    run(s)
    torch.cuda.synchronize()
    t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    t0.record(hold)
    assert lib.occupy_lds_launch(2 * cus, int(SPIN_MS * 1e5), 64 << 10, ctypes.c_void_p(hold.cuda_stream)) == 0
    time.sleep(5e-3)
    run(s)
    t1.record(s)
    torch.cuda.synchronize()
    return t0.elapsed_time(t1)


@pytest.mark.parametrize("R, n, cus, cfg", [
    (8, 1 << 20, 256, {}),                               # the bound gained nothing at eight ranks
    (4, 1 << 18, 256, {}),                               # nor in small calls
    (4, 5 << 20, 256, dict(workgroups_per_step=64)),     # a budget bounds by itself
    (4, 5 << 20, 32, {}),                                # a part of the CUs
], ids=["eight", "small", "budget", "masked"])
def test_allreduce_leaves_the_lds_to_others(R, n, cus, cfg):
    hc.set_config(reduce_algo="direct", **cfg)
    x = [W.random_values("fp32", 1000 + R, r, n) for r in range(R)]
    send = [to_dev(a, hc.FP32) for a in x]
    out = [torch.empty_like(t) for t in send]
    ms = ends_beside_the_spin(lambda s: hc.allreduce(send, out, stream=s), cus)
    assert ms < SPIN_MS - 10, f"ended {ms:.1f} ms after the spin began: it waited for the LDS"
    ref = oracle.allreduce_new(x, hc.FP32)
    for r in range(R):
        assert_bitwise(from_dev(out[r], hc.FP32), ref[r], f"r={r}")


@pytest.mark.parametrize("n, cus, cfg", [
    (1 << 16, 256, {}), (1 << 20, 256, dict(workgroups_per_step=64)), (1 << 20, 32, {}),
], ids=["small", "budget", "masked"])
def test_gather_leaves_the_lds_to_others(n, cus, cfg):
    hc.set_config(copy_path="kernel", **cfg)
    R = 8
    x = [W.random_bits(1010, r, n, 1) for r in range(R)]
    send = [to_dev(a, hc.UINT8) for a in x]
    out = [torch.empty(R * n, dtype=torch.uint8, device="cuda") for _ in range(R)]
    ms = ends_beside_the_spin(lambda s: hc.allgather(send, out, stream=s), cus)
    assert ms < SPIN_MS - 10, f"ended {ms:.1f} ms after the spin began: it waited for the LDS"
    whole = np.concatenate(x)
    for r in range(R):
        assert_bitwise(from_dev(out[r], hc.UINT8), whole, f"r={r}")


@pytest.mark.parametrize("cus", [256, 32])
def test_bounded_launches_on_whole_and_masked_streams(cus):
    """The sizes that ask for LDS on the whole chip, and the same calls on a
    part of it."""
    s = spin(cus)[1]
    R, n = 3, (4 << 20) + 3
    x = [W.random_values("fp32", 1020, r, n) for r in range(R)]
    send = [to_dev(a, hc.FP32) for a in x]
    out = [torch.empty_like(t) for t in send]
    hc.set_config(reduce_algo="direct", copy_path="kernel")
    torch.cuda.synchronize()
    hc.allreduce(send, out, stream=s)
    torch.cuda.synchronize()
    ref = oracle.allreduce_new(x, hc.FP32)
    for r in range(R):
        assert_bitwise(from_dev(out[r], hc.FP32), ref[r], f"AR r={r}")
    shards = [W.random_bits(1030, r, (3 << 20) + 7, 1) for r in range(6)]
    send = [to_dev(a, hc.UINT8) for a in shards]
    out = [torch.empty(6 * shards[0].size, dtype=torch.uint8, device="cuda") for _ in range(6)]
    torch.cuda.synchronize()
    hc.allgather(send, out, stream=s)
    torch.cuda.synchronize()
    whole = np.concatenate(shards)
    for r in range(6):
        assert_bitwise(from_dev(out[r], hc.UINT8), whole, f"AG r={r}")


def test_bounded_launch_on_the_per_thread_stream():
    """The handle 2 (hipStreamPerThread) is no pointer: asking for its mask must
    not follow it."""
    R, n = 3, (4 << 20) + 3
    x = [W.random_values("fp32", 1040, r, n) for r in range(R)]
    send = [to_dev(a, hc.FP32) for a in x]
    out = [torch.empty_like(t) for t in send]
    hc.set_config(reduce_algo="direct")
    torch.cuda.synchronize()
    hc.allreduce(send, out, stream=types.SimpleNamespace(cuda_stream=2))
    torch.cuda.synchronize()
    ref = oracle.allreduce_new(x, hc.FP32)
    for r in range(R):
        assert_bitwise(from_dev(out[r], hc.FP32), ref[r], f"AR r={r}")
