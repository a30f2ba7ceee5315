"""The CU copy kernel's launches: what the statistics report of them, which
copies share one, and results bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_34334_amd as hc
import workloads as W
from gpu_util import assert_bitwise, check_canaries, from_dev, padded, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _fresh_config():
    saved = hc.get_config()
    yield
    hc.set_config(**saved)


@pytest.mark.parametrize("nbytes, budget", [(100, 0), (1 << 20, 0), ((64 << 20) + 5, 0), (1 << 20, 3)])
def test_statistics_hold_the_workgroups_launched(nbytes, budget):
    """A message of one tile takes one workgroup and one CU at most, a large
    one as many as it has tiles (of at least one 16-byte vector per thread)
    and every CU; a budget is what is launched."""
    hc.set_config(copy_path="kernel", workgroups_per_step=budget)
    x = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    hc.sendrecv([x, x], [None, torch.empty_like(x)], [1, -1])
    torch.cuda.synchronize()
    s = hc.last_stats()
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    most = -(-nbytes // (256 * 16))
    assert s["copy_kernel_launches"] == 1
    if budget:
        assert s["workgroups_per_step"] == budget and s["cus_used_max"] == budget
    else:
        assert 1 <= s["workgroups_per_step"] <= most, s
        assert s["cus_used_max"] == min(s["workgroups_per_step"], ncu)
    if nbytes > 64 << 20:
        assert s["cus_used_max"] == ncu


def gather(R, n, lead=3):
    """An all-gather of byte shards into windows at odd offsets, checked with
    canaries; returns the call's statistics."""
    x = [W.random_bits(1100 + R, r, n, 1) for r in range(R)]
    pads = [padded(R * n, hc.UINT8, lead=lead + r) for r in range(R)]
    hc.allgather([to_dev(a, hc.UINT8) for a in x], [w for _, w in pads])
    torch.cuda.synchronize()
    whole = np.concatenate(x)
    for r, (full, win) in enumerate(pads):
        check_canaries(full, lead + r, R * n, hc.UINT8)
        assert_bitwise(from_dev(win, hc.UINT8), whole, f"AG R={R} n={n} r={r}")
    return hc.last_stats()


@pytest.mark.parametrize("R", [2, 5, 8])
@pytest.mark.parametrize("chunk", [4096, 5000, 65_537])
def test_pieces_of_a_copy_share_its_launch(R, chunk):
    """chunk_bytes cuts copies for the engines; the kernel joins the pieces, so
    that a gather is one launch and reads a shard once."""
    hc.set_config(copy_path="kernel", chunk_bytes=chunk)
    assert gather(R, 131_075)["copy_kernel_launches"] == 1


@pytest.mark.parametrize("cfg", [dict(a2a_schedule=1), dict(a2a_schedule=0)], ids=["staged", "direct"])
def test_pieces_in_the_schedulers_order(cfg):
    """The scheduler deals the pieces of several flows in turn: those of one
    flow mostly don't follow each other."""
    hc.set_config(copy_path="kernel", chunk_bytes=4096, **cfg)
    R, n = 4, 20_001
    x = [W.random_bits(1120, r, R * n, 1) for r in range(R)]
    ref = [np.zeros(R * n, np.uint8) for _ in range(R)]
    oracle.alltoall(x, ref, n, hc.UINT8)
    out = hc.alltoall([to_dev(a, hc.UINT8) for a in x])
    torch.cuda.synchronize()
    for r in range(R):
        assert_bitwise(from_dev(out[r], hc.UINT8), ref[r], f"A2A r={r}")


def test_pieces_of_a_forwarding_gather():
    hc.set_config(copy_path="kernel", chunk_bytes=4096, allgather_direct=0)
    gather(5, 30_001)


@pytest.mark.parametrize("R, launches", [(8, 1), (9, 1), (10, 1), (16, 1), (17, 2), (25, 4)])
def test_no_destination_is_left_for_a_launch_of_its_own(R, launches):
    """Segments of up to eight destinations, 32 to a launch: nine and 17 ranks
    split their destinations evenly."""
    hc.set_config(copy_path="kernel")
    assert gather(R, 1003)["copy_kernel_launches"] == launches
