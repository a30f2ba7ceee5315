"""The direct fold at the sizes where its blocks change their order: 4 and 8
ranks beyond 600 MiB a rank, 2 beyond 768, bf16 all-reduces of 16, 24, ... ranks
from 192 MiB of inputs, each around the limit, at odd lengths and offsets, with
canaries.  The buffers are too large for the oracle, so
that the fold of each chunk is repeated on the device, one elementwise addition
after another in the ring's order, and compared bit for bit."""
import pytest
import torch

import paper_2609_34334_amd as hc
from gpu_util import TORCH, padded

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _fresh_config():
    saved = hc.get_config()
    yield
    hc.set_config(**saved)
    torch.cuda.empty_cache()


def folded(send, j, lo, hi, partials=0):
    """Chunk j's elements lo to hi: x[j+1] + x[j+2] + ... + x[j], rounded once or
    (bf16 partials) after every addition."""
    R = len(send)
    acc = send[(j + 1) % R][lo:hi].float()
    for k in range(2, R + 1):
        acc += send[(j + k) % R][lo:hi].float()
        if partials:
            acc = acc.to(send[0].dtype).float()
    return acc.to(send[0].dtype)


@pytest.mark.parametrize("wg", [0, 300])
@pytest.mark.parametrize("R, mib, dt", [(2, 769, hc.BF16), (4, 601, hc.BF16), (8, 601, hc.BF16), (4, 601, hc.FP32)])
def test_folds_whose_blocks_go_in_turn(R, mib, dt, wg):
    hc.set_config(reduce_algo="direct", workgroups_per_step=wg)
    bits = torch.int16 if dt == hc.BF16 else torch.int32
    total = (mib << 20) // (2 if dt == hc.BF16 else 4) + 5
    g = torch.Generator(device="cuda").manual_seed(1300 + R)
    send = [torch.randn(total + 3, generator=g, device="cuda", dtype=TORCH[dt])[r % 4:r % 4 + total] for r in range(R)]

    n = total // R
    pads = [padded(n, dt, lead=1 + r) for r in range(R)]
    hc.reduce_scatter([t[:n * R] for t in send], [w for _, w in pads])
    torch.cuda.synchronize()
    for j, (full, win) in enumerate(pads):
        assert torch.equal(win.view(bits), folded(send, j, j * n, (j + 1) * n).view(bits)), f"RS R={R} j={j}"
        edge = torch.cat([full[:1 + j], full[1 + j + n:]]).view(bits)
        assert bool((edge == edge[0]).all()), f"RS R={R} j={j}: canary overwritten"
    del pads, full, win

    out = [torch.empty(total, dtype=TORCH[dt], device="cuda") for _ in range(R)]
    hc.allreduce(send, out)
    torch.cuda.synchronize()
    c = -(-total // R)
    for j in range(R):
        lo, hi = j * c, min(total, (j + 1) * c)
        want = folded(send, j, lo, hi).view(bits)
        for r in range(R):
            assert torch.equal(out[r][lo:hi].view(bits), want), f"AR R={R} chunk {j} rank {r}"


@pytest.mark.parametrize("partials", [0, 1])
@pytest.mark.parametrize("R, kib", [(16, 12287), (16, 12289), (24, 8193), (64, 3073), (20, 10241)])
def test_all_reduces_of_many_ranks_around_192_MiB(R, kib, partials):
    hc.set_config(reduce_algo="direct", bf16_partials=partials)
    total = kib * 512 + 3
    g = torch.Generator(device="cuda").manual_seed(1310 + R)
    send = [torch.randn(total + 3, generator=g, device="cuda", dtype=torch.bfloat16)[r % 4:r % 4 + total]
            for r in range(R)]
    pads = [padded(total, hc.BF16, lead=1 + r % 5) for r in range(R)]
    hc.allreduce(send, [w for _, w in pads])
    torch.cuda.synchronize()
    c = -(-total // R)
    for j in range(R):
        lo, hi = j * c, min(total, (j + 1) * c)
        want = folded(send, j, lo, hi, partials).view(torch.int16)
        for r in range(R):
            assert torch.equal(pads[r][1][lo:hi].view(torch.int16), want), f"AR R={R} chunk {j} rank {r}"
    for r, (full, _) in enumerate(pads):
        edge = torch.cat([full[:1 + r % 5], full[1 + r % 5 + total:]]).view(torch.int16)
        assert bool((edge == edge[0]).all()), f"AR R={R} rank {r}: canary overwritten"
