"""Vector paths on operands that share no alignment, against the oracle bit
for bit: every rank's input and output starts at an element offset of its
own, at lengths around one vector, one workgroup's tile and several tiles,
for the fold, the ring, fused hops and one hop, with canaries around every
output."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_34334_amd as hc
import workloads as W
from gpu_util import NAME, assert_bitwise, check_canaries, from_dev, padded, to_dev

pytestmark = pytest.mark.gpu

DTS = [hc.INT32, hc.FP32, hc.BF16]
# Below, at and beyond one vector; a workgroup's tile of 256 threads (one
# vector each of 4 or 8 elements, or several) less one, itself and one more.
LENGTHS = [1, 3, 8, 17, 1023, 1025, 2047, 4097, 40_961]


@pytest.fixture(autouse=True)
def _fresh_config():
    saved = hc.get_config()
    yield
    hc.set_config(**saved)


def shifted(a, dt, lead):
    return to_dev(np.concatenate([np.zeros(lead, a.dtype), a]), dt)[lead:]


def outputs(R, n, dt, step):
    return [padded(n, dt, lead=(step * r + 1) % 9) for r in range(R)]


def finish(outs, n, dt, ref, step, what):
    torch.cuda.synchronize()
    for r, (full, win) in enumerate(outs):
        check_canaries(full, (step * r + 1) % 9, n, dt)
        assert_bitwise(from_dev(win, dt), ref[r], f"{what} r={r}")


@pytest.mark.parametrize("cfg", [dict(reduce_algo="direct"), dict(reduce_algo="ring"),
                                 dict(reduce_algo="ring", fused_hops=3)],
                         ids=["fold", "ring", "fused"])
@pytest.mark.parametrize("R", [2, 5, 8, 17])
@pytest.mark.parametrize("dt", DTS, ids=NAME.get)
def test_reductions_where_no_two_buffers_share_alignment(dt, R, cfg):
    hc.set_config(copy_path="kernel", **cfg)
    for n in LENGTHS:
        x = [W.random_values(NAME[dt], 900 + R, r, R * n) for r in range(R)]
        outs = outputs(R, n, dt, 5)
        hc.reduce_scatter([shifted(x[r], dt, (3 * r + 1) % 9) for r in range(R)], [o[1] for o in outs])
        finish(outs, n, dt, oracle.reduce_scatter_new(x, dt), 5, f"RS n={n}")
        xa = [W.random_values(NAME[dt], 910 + R, r, n) for r in range(R)]
        outs = outputs(R, n, dt, 2)
        hc.allreduce([shifted(xa[r], dt, (5 * r + 2) % 9) for r in range(R)], [o[1] for o in outs])
        finish(outs, n, dt, oracle.allreduce_new(xa, dt), 2, f"AR n={n}")


@pytest.mark.parametrize("partials", [0, 1])
@pytest.mark.parametrize("R", [6, 7, 9, 10, 16, 18, 24, 33])
def test_fold_at_every_remainder_of_its_batches(R, partials):
    """The fold keeps up to 8 ranks in registers and takes more in batches
    of 8: R - 1 one batch exactly, one rank over, one short, and several."""
    hc.set_config(reduce_algo="direct", bf16_partials=partials)
    for dt in DTS:
        hops = partials and dt == hc.BF16
        for n in (5, 2049):
            x = [W.random_values(NAME[dt], 920 + R, r, R * n) for r in range(R)]
            outs = outputs(R, n, dt, 5)
            hc.reduce_scatter([to_dev(a, dt) for a in x], [o[1] for o in outs])
            ref = oracle.reduce_scatter_bf16_hops_new(x) if hops else oracle.reduce_scatter_new(x, dt)
            finish(outs, n, dt, ref, 5, f"RS {NAME[dt]} n={n}")
            xa = [W.random_values(NAME[dt], 930 + R, r, R * n + 1) for r in range(R)]
            send = [to_dev(a, dt) for a in xa]
            hc.allreduce(send)                        # in place
            torch.cuda.synchronize()
            ref = oracle.allreduce_bf16_hops_new(xa) if hops else oracle.allreduce_new(xa, dt)
            for r in range(R):
                assert_bitwise(from_dev(send[r], dt), ref[r], f"AR {NAME[dt]} n={R * n + 1} r={r}")


# Bytes around one vector, one lane's leftovers and a copy tile (256 threads
# of one or of four 16-byte vectors).
COPY_BYTES = [1, 15, 16, 33, 4095, 4097, 16_383, 16_385, 100_003]


@pytest.mark.parametrize("wg", [0, 1, 7])
@pytest.mark.parametrize("R", [2, 3, 4, 9, 17])
def test_gathered_shards_share_their_source_reads(R, wg):
    """The CU copy reads a shard once for up to eight destinations; every
    rank's output starts at its own offset, and 9 and 17 ranks leave a
    segment of a single destination."""
    hc.set_config(copy_path="kernel", workgroups_per_step=wg)
    for n in COPY_BYTES:
        x = [W.random_bits(940 + R, r, n, 1) for r in range(R)]
        ref = oracle.allgather_new(x, hc.UINT8)
        outs = outputs(R, R * n, hc.UINT8, 5)
        hc.allgather([shifted(x[r], hc.UINT8, (7 * r + 1) % 17) for r in range(R)], [o[1] for o in outs])
        finish(outs, R * n, hc.UINT8, ref, 5, f"AG n={n}")
        full = [to_dev(np.concatenate([x[r] if q == r else np.zeros(n, np.uint8) for q in range(R)]), hc.UINT8)
                for r in range(R)]
        hc.allgather([full[r][r * n:(r + 1) * n] for r in range(R)], full)          # in place
        torch.cuda.synchronize()
        for r in range(R):
            assert_bitwise(from_dev(full[r], hc.UINT8), ref[r], f"AG in place n={n} r={r}")


@pytest.mark.parametrize("wg", [0, 1, 5])
@pytest.mark.parametrize("R", [2, 5, 12])
def test_copies_of_unequal_ragged_segments(R, wg):
    """All-to-all(v) by the CU copy: segments of every length around a tile,
    empty ones among them, at odd offsets (144 of them take two launches),
    with every workgroup walking several segments or none."""
    hc.set_config(copy_path="kernel", workgroups_per_step=wg)
    lens = [0, *COPY_BYTES]
    counts = [lens[(3 * k + k // R) % len(lens)] for k in range(R * R)]
    sd = [sum(counts[s * R:s * R + d]) + d for s in range(R) for d in range(R)]       # a byte apart
    rd = [sum(counts[q * R + d] for q in range(s)) + 2 * s for s in range(R) for d in range(R)]
    sizes = [sum(counts[s * R:(s + 1) * R]) + R for s in range(R)]
    x = [W.random_bits(950 + R, r, sizes[r], 1) for r in range(R)]
    rsizes = [sum(counts[s * R + d] for s in range(R)) + 2 * R for d in range(R)]
    ref = [np.full(n, 0x5A, np.uint8) for n in rsizes]
    oracle.alltoallv(x, counts, sd, ref, rd, hc.UINT8)
    recv = [to_dev(np.full(n, 0x5A, np.uint8), hc.UINT8) for n in rsizes]
    hc.alltoallv([to_dev(a, hc.UINT8) for a in x], counts, sd, recv, rd)
    torch.cuda.synchronize()
    for r in range(R):
        assert_bitwise(from_dev(recv[r], hc.UINT8), ref[r], f"A2AV r={r}")


def test_a_broadcast_reads_its_root_once_for_eight_ranks():
    """Flows that read the same bytes share segments: a one-row
    all-to-all(v), and one whose flows only partly coincide."""
    hc.set_config(copy_path="kernel")
    R, n = 11, 70_001
    x = [W.random_bits(960, r, n, 2) for r in range(R)]
    send = [to_dev(a, hc.BF16) for a in x]
    for counts0 in ([0] + [n] * (R - 1), [0, n, n, n - 1, n, n, n, n, n, 5, 5]):
        counts = counts0 + [0] * (R * (R - 1))
        outs = outputs(R, n, hc.BF16, 2)
        ref = [np.zeros(n, np.uint16) for _ in range(R)]
        for o in outs:
            o[1].zero_()
        oracle.alltoallv(x, counts, [0] * (R * R), ref, [0] * (R * R), hc.BF16)
        hc.alltoallv(send, counts, [0] * (R * R), [o[1] for o in outs], [0] * (R * R))
        finish(outs, n, hc.BF16, ref, 2, f"broadcast {counts0[3]}")


@pytest.mark.parametrize("lead", [1, 31, 33, 63, 64, 127])
@pytest.mark.parametrize("threads, wg", [(64, 0), (64, 3), (256, 0)])
def test_heads_up_to_a_cache_line(lead, threads, wg):
    """Vectors start where a buffer reaches a 128-byte line: heads from one
    element to all but one of a line, with segments that end inside the head
    and just after it, and more left-over elements than a workgroup has
    lanes."""
    for n in (5, 64, 65, 131, 2113):
        for R, cfg in ((3, dict(reduce_algo="direct")), (9, dict(reduce_algo="direct")),
                       (4, dict(reduce_algo="ring")), (4, dict(reduce_algo="ring", fused_hops=2))):
            hc.set_config(copy_path="kernel", threads_per_workgroup=threads, workgroups_per_step=wg,
                          **{"fused_hops": 1, **cfg})
            for dt in DTS:
                x = [W.random_values(NAME[dt], 970 + R, r, R * n) for r in range(R)]
                outs = outputs(R, n, dt, 4)
                hc.reduce_scatter([shifted(a, dt, lead) for a in x], [o[1] for o in outs])
                finish(outs, n, dt, oracle.reduce_scatter_new(x, dt), 4, f"RS {cfg} n={n}")
        for R in (2, 5):
            x = [W.random_bits(980 + R, r, n, 1) for r in range(R)]
            pads = [padded(R * n, hc.UINT8, lead=lead + r) for r in range(R)]
            hc.allgather([to_dev(a, hc.UINT8) for a in x], [w for _, w in pads])
            torch.cuda.synchronize()
            for r, (full, win) in enumerate(pads):
                check_canaries(full, lead + r, R * n, hc.UINT8)
                assert_bitwise(from_dev(win, hc.UINT8), oracle.allgather_new(x, hc.UINT8)[r], f"AG n={n} r={r}")


@pytest.mark.parametrize("wg", [0, 3, 13, 24])
@pytest.mark.parametrize("R, hops, n", [(5, 1, 900_001), (9, 2, 500_003)])
def test_ring_steps_that_alternate_their_direction(R, hops, n, wg):
    """Partials of 16 MiB and more turn every other step's block order round:
    with a workgroup per tile, fewer workgroups than segments, and grids that
    do and do not divide by the XCDs."""
    hc.set_config(reduce_algo="ring", fused_hops=hops, workgroups_per_step=wg)
    for dt in (hc.INT32, hc.BF16):
        x = [W.random_values(NAME[dt], 990 + R, r, R * n) for r in range(R)]
        outs = outputs(R, n, dt, 5)
        hc.reduce_scatter([to_dev(a, dt) for a in x], [o[1] for o in outs])
        finish(outs, n, dt, oracle.reduce_scatter_new(x, dt), 5, f"RS {NAME[dt]} wg={wg}")
