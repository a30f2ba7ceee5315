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


def test_statistics_count_a_shared_read_once():
    """Nine ranks read every shard twice (for five destinations and four) and
    write it nine times; a copy of its own per destination reads it nine times."""
    R, n = 9, 4096
    send = [torch.zeros(n, dtype=torch.uint8, device="cuda") for _ in range(R)]
    recv = [torch.empty(R * n, dtype=torch.uint8, device="cuda") for _ in range(R)]
    for path, reads in (("kernel", 2), ("hip", R)):
        hc.set_config(copy_path=path)
        hc.allgather(send, recv)
        torch.cuda.synchronize()
        s = hc.last_stats()
        assert s["hbm_bytes_algorithmic"] == R * n * (reads + R), path
        assert s["copy_bytes"] == R * R * n
    hc.set_config(copy_path="kernel")
    hc.sendrecv(send, recv=[torch.empty_like(t) for t in send], peers=[(r + 1) % R for r in range(R)])
    torch.cuda.synchronize()
    assert hc.last_stats()["hbm_bytes_algorithmic"] == 2 * R * n


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


def random_bytes(n, seed, lead=0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(0, 256, (lead + n,), generator=g, device="cuda", dtype=torch.uint8)[lead:]


def same(full, lead, n, parts, what):
    """The window holds `parts` one after another and the canaries around it
    stand (compared on the device: these buffers are large)."""
    assert bool((full[:lead] == 0x5A).all()) and bool((full[lead + n:] == 0x5A).all()), f"{what}: canary overwritten"
    at = lead
    for p in parts:
        assert torch.equal(full[at:at + p.numel()], p), what
        at += p.numel()
    assert at == lead + n


# Which form a copy launch takes goes by its bytes, the evenness of its segments
# and the workgroup budget: each form at odd lengths and offsets, below and
# above every limit.
@pytest.mark.parametrize("wg", [0, 5, 300])
@pytest.mark.parametrize("R, n", [(2, 4_000_037), (2, (9 << 20) + 3), (2, (25 << 20) + 1), (3, (5 << 20) + 7)])
def test_messages_in_every_form(R, n, wg):
    hc.set_config(copy_path="kernel", workgroups_per_step=wg)
    send = [random_bytes(n, 1200 + r, lead=5 * r + 1) for r in range(R)]
    pads = [padded(n, hc.UINT8, lead=3 + r) for r in range(R)]
    hc.sendrecv(send, [w for _, w in pads], [(r + 1) % R for r in range(R)])
    torch.cuda.synchronize()
    for r, (full, _) in enumerate(pads):
        same(full, 3 + r, n, [send[(r - 1) % R]], f"SR R={R} n={n} r={r}")


@pytest.mark.parametrize("wg", [0, 5, 64, 300])
@pytest.mark.parametrize("R, n, skew", [(8, 70_001, 0), (8, (1 << 20) - 5, 0), (8, (1 << 20) + 3, 0),
                                        (8, 200_000, 1), (6, 900_000, 1), (12, 3000, 1)])
def test_all_to_all_in_every_form(R, n, skew, wg):
    hc.set_config(copy_path="kernel", workgroups_per_step=wg)
    rng = np.random.default_rng(1210 + R)
    counts = [int(n * (4 * rng.random() ** 6 if skew else 1)) for _ in range(R * R)]
    sd = [sum(counts[s * R:s * R + d]) for s in range(R) for d in range(R)]
    rd = [sum(counts[q * R + d] for q in range(s)) for s in range(R) for d in range(R)]
    send = [random_bytes(sum(counts[s * R:(s + 1) * R]), 1220 + s, lead=s) for s in range(R)]
    sizes = [sum(counts[s * R + d] for s in range(R)) for d in range(R)]
    pads = [padded(m, hc.UINT8, lead=1 + d) for d, m in enumerate(sizes)]
    hc.alltoallv(send, counts, sd, [w for _, w in pads], rd)
    torch.cuda.synchronize()
    for d, (full, _) in enumerate(pads):
        parts = [send[s][sd[s * R + d]:sd[s * R + d] + counts[s * R + d]] for s in range(R)]
        same(full, 1 + d, sizes[d], parts, f"A2AV R={R} n={n} d={d}")


@pytest.mark.parametrize("wg", [0, 5, 300])
@pytest.mark.parametrize("R, n", [(3, 100_003), (3, (3 << 20) + 1), (4, (2 << 20) - 1), (5, (1 << 20) + 9),
                                  (8, 262_143), (8, 262_147), (9, 1_000_003)])
def test_gathers_in_every_form(R, n, wg):
    hc.set_config(copy_path="kernel", workgroups_per_step=wg)
    send = [random_bytes(n, 1230 + r, lead=7 * r + 1) for r in range(R)]
    pads = [padded(R * n, hc.UINT8, lead=2 + r) for r in range(R)]
    hc.allgather(send, [w for _, w in pads])
    torch.cuda.synchronize()
    for r, (full, _) in enumerate(pads):
        same(full, 2 + r, R * n, send, f"AG R={R} n={n} r={r}")


@pytest.mark.parametrize("wg", [0, 300])
def test_launches_beyond_the_last_level_cache(wg):
    """More than 256 MiB in one launch: read past the caches without a budget,
    by equal and by unequal segments at odd lengths and offsets."""
    hc.set_config(copy_path="kernel", workgroups_per_step=wg)
    n = (129 << 20) + 5
    send = [random_bytes(n, 1240 + r, lead=3 + 2 * r) for r in range(2)]
    pads = [padded(n, hc.UINT8, lead=1 + r) for r in range(2)]
    hc.sendrecv(send, [w for _, w in pads], [1, 0])
    torch.cuda.synchronize()
    assert hc.last_stats()["copy_kernel_launches"] == 1
    for r, (full, _) in enumerate(pads):
        same(full, 1 + r, n, [send[1 - r]], f"SR r={r}")
    del send, pads
    R = 8
    rng = np.random.default_rng(1250)
    counts = [int(v) for v in rng.integers(4_000_001, 5_000_000, R * R)]
    sd = [sum(counts[s * R:s * R + d]) for s in range(R) for d in range(R)]
    rd = [sum(counts[q * R + d] for q in range(s)) for s in range(R) for d in range(R)]
    send = [random_bytes(sum(counts[s * R:(s + 1) * R]), 1260 + s, lead=s) for s in range(R)]
    sizes = [sum(counts[s * R + d] for s in range(R)) for d in range(R)]
    assert sum(sizes) > 256 << 20
    pads = [padded(m, hc.UINT8, lead=1 + d) for d, m in enumerate(sizes)]
    hc.alltoallv(send, counts, sd, [w for _, w in pads], rd)
    torch.cuda.synchronize()
    for d, (full, _) in enumerate(pads):
        parts = [send[s][sd[s * R + d]:sd[s * R + d] + counts[s * R + d]] for s in range(R)]
        same(full, 1 + d, sizes[d], parts, f"A2AV d={d}")
