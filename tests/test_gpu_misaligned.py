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
