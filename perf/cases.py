"""What the speed of this library is measured on: collectives over R ranks
whose buffers live in one GPU's memory, called through the Python binding.

The sizes come from the training traffic the repository's own workloads are
shaped like: GPT-6.7B (hidden 4096, ffn 16384, sequence 2048, bf16) and
DeepSeek-V2-Lite (hidden 2048, 64 experts, top-6 routing), and from the
benchmark.  A case names the operation, the ranks, the elements (`n`: per
rank for all-reduce and send/recv and ring_hop, per output shard for
reduce-scatter, per shard for all-gather), the dtype, and the configuration
fields that differ from the library's defaults.  For all-to-all(v) the tokens,
the hidden size and the routing seed give the counts.
"""
import functools
import math

import torch

import paper_2609_34334_amd as hoccl

_DT = {"bf16": torch.bfloat16, "fp32": torch.float32, "int32": torch.int32, "uint8": torch.uint8}
_ES = {"bf16": 2, "fp32": 4, "int32": 4, "uint8": 1}
_DEFAULTS = {"reduce_algo": "auto", "copy_path": "auto", "bf16_partials": 0, "fused_hops": 1}
_EXPERTS, _TOPK = 64, 6


def listed():
    return [
        # A metric or a loss summed over two data-parallel ranks: the
        # smallest call, all latency.
        {"name": "allreduce_small", "op": "allreduce", "R": 2, "n": 1024, "dtype": "fp32"},
        # The benchmark's fp32 all-reduce: one medium gradient tensor.
        {"name": "allreduce_fp32_R4", "op": "allreduce", "R": 4, "n": 1048576, "dtype": "fp32"},
        # A 48 MiB DistributedDataParallel gradient bucket.
        {"name": "allreduce_bucket", "op": "allreduce", "R": 8, "n": 25165824, "dtype": "bf16"},
        # Gradients of a layer whose parameters do not divide by the ranks,
        # accumulated in fp32 over sixteen of them.
        {"name": "allreduce_R16_odd", "op": "allreduce", "R": 16, "n": 1500007, "dtype": "fp32"},
        # The data-parallel gradient reduce-scatter, as the library chooses.
        {"name": "reduce_scatter_gradients", "op": "reduce_scatter", "R": 8, "n": 3145728, "dtype": "bf16"},
        # The same by the ring, the benchmark's headline.
        {"name": "reduce_scatter_ring", "op": "reduce_scatter", "R": 8, "n": 3145728, "dtype": "bf16",
         "reduce_algo": "ring"},
        # A sharded layer of uneven size over six ranks.
        {"name": "reduce_scatter_ragged", "op": "reduce_scatter", "R": 6, "n": 1398103, "dtype": "bf16"},
        # One rank's share of one ring step of the headline.
        {"name": "ring_hop_middle", "op": "ring_hop", "R": 1, "n": 3145728, "dtype": "bf16", "hop": "middle"},
        # The FSDP parameter all-gather of one transformer block, on the copy
        # engines (the default: no compute unit).
        {"name": "allgather_block", "op": "allgather", "R": 8, "n": 25165824, "dtype": "bf16"},
        # One MLP matrix gathered by the compute units, where no compute runs
        # beside it.
        {"name": "allgather_mlp_kernel", "op": "allgather", "R": 8, "n": 8388608, "dtype": "bf16",
         "copy_path": "kernel"},
        # Expert-parallel dispatch: 4096 tokens a rank, by the compute units.
        {"name": "alltoallv_dispatch_kernel", "op": "alltoallv", "R": 8, "tokens": 4096, "hidden": 2048,
         "routing": 5, "dtype": "bf16", "copy_path": "kernel"},
        # A small pipeline message on the copy engines.
        {"name": "sendrecv_small", "op": "sendrecv", "R": 2, "n": 2048, "dtype": "bf16"},
    ]


def _log(rng, lo, hi):
    """A size between lo and hi, spread over its logarithm; half of them are
    the round ones that tensors mostly have."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5 and n >= 512:
        n = n // 256 * 256
    return max(lo, min(hi, n))


def draw(rng):
    kind = rng.choice(["allreduce"] * 3 + ["reduce_scatter"] * 4 + ["ring"] * 2 + ["ring_hop"] + ["allgather"] * 2 +
                      ["alltoallv"] * 2 + ["sendrecv"])
    if kind in ("allreduce", "reduce_scatter", "ring"):
        R = rng.choice([2, 3, 4, 5, 6, 7, 8, 8, 12, 16, 24, 32])
        dt = rng.choice(["bf16", "bf16", "fp32", "int32"])
        # Up to the headline's 48 MiB a rank, and twice its 384 MiB in all.
        total = min((48 << 20) // _ES[dt], (768 << 20) // (R * _ES[dt]))
        per_rank = _log(rng, 1024, total)
        c = {"op": "allreduce" if kind == "allreduce" else "reduce_scatter", "R": R, "dtype": dt,
             "n": per_rank if kind == "allreduce" else max(1, per_rank // R)}
        if kind == "ring":
            c["reduce_algo"] = "ring"
            c["fused_hops"] = rng.choice([1, 2, 4])
        if dt == "bf16" and rng.random() < 0.25:
            c["bf16_partials"] = 1
        return c
    if kind == "ring_hop":
        return {"op": "ring_hop", "R": 1, "n": _log(rng, 4096, 25165824), "dtype": rng.choice(["bf16", "bf16", "fp32"]),
                "hop": rng.choice(["first", "middle", "last", "only"])}
    path = rng.choice(["auto", "kernel", "kernel"])
    if kind == "allgather":
        R = rng.choice([2, 4, 6, 8, 8])
        dt = rng.choice(["bf16", "bf16", "fp32", "uint8"])
        return {"op": "allgather", "R": R, "n": _log(rng, 1024, (16 << 20) // _ES[dt]), "dtype": dt, "copy_path": path}
    if kind == "alltoallv":
        return {"op": "alltoallv", "R": rng.choice([2, 4, 8, 8]), "tokens": _log(rng, 64, 8192),
                "hidden": rng.choice([1024, 1337, 2048, 2048, 2730, 4096]), "routing": rng.randrange(1000),
                "dtype": "bf16", "copy_path": path}
    dt = rng.choice(["bf16", "bf16", "fp32", "uint8"])
    return {"op": "sendrecv", "R": rng.choice([2, 4, 8]), "n": _log(rng, 2048, (32 << 20) // _ES[dt]), "dtype": dt,
            "copy_path": path}


@functools.lru_cache(maxsize=8)
def _routing(R, tokens, hidden, seed):
    """Counts and displacements of the expert-parallel dispatch: every token
    picks 6 of 64 experts, and goes once to each rank that hosts one."""
    g = torch.Generator().manual_seed(seed)
    per = _EXPERTS // R
    counts = []
    for _ in range(R):
        rank = torch.rand(tokens, _EXPERTS, generator=g).topk(_TOPK, dim=1).indices // per
        counts += [int((rank == d).any(dim=1).sum()) * hidden for d in range(R)]
    sd = [sum(counts[s * R:s * R + d]) for s in range(R) for d in range(R)]
    rd = [sum(counts[q * R + d] for q in range(s)) for s in range(R) for d in range(R)]
    return counts, sd, rd


def _a2av(case):
    return _routing(case["R"], case["tokens"], case["hidden"], case["routing"])


def _values(dtype, n, g, std):
    if dtype == "int32":
        return torch.randint(-(2 ** 31), 2 ** 31, (n,), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    if dtype == "uint8":
        return torch.randint(0, 256, (n,), generator=g, device="cuda", dtype=torch.uint8)
    return (torch.randn(n, generator=g, device="cuda") * std).to(_DT[dtype])


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)
    op, R, dt = case["op"], case["R"], case["dtype"]
    if op == "reduce_scatter":
        return [_values(dt, R * case["n"], g, 1e-3) for _ in range(R)]      # gradients
    if op == "allreduce":
        return [_values(dt, case["n"], g, 1e-3) for _ in range(R)]
    if op == "allgather":
        return [_values(dt, case["n"], g, 0.02) for _ in range(R)]          # parameters
    if op == "sendrecv":
        return [_values(dt, case["n"], g, 1.0) for _ in range(R)]           # activations
    if op == "alltoallv":
        counts = _a2av(case)[0]
        return [_values(dt, sum(counts[s * R:(s + 1) * R]), g, 1.0) for s in range(R)]
    partial_dt = "fp32" if dt == "bf16" and case["hop"] in ("middle", "last") else dt
    return [_values(partial_dt, case["n"], g, 3e-3), _values(dt, case["n"], g, 1e-3)]


def _hop_out(case):
    return "fp32" if case["dtype"] == "bf16" and case["hop"] in ("first", "middle") else case["dtype"]


def _recv_sizes(case):
    op, R, n = case["op"], case["R"], case.get("n")
    if op == "alltoallv":
        counts = _a2av(case)[0]
        return [sum(counts[s * R + d] for s in range(R)) for d in range(R)]
    if op == "sendrecv":
        return [n] * R
    return [R * n if op == "allgather" else n] * R


# The configuration is the process's: a program sets it once, when it starts.
# It is set again here only when the case before had another.
_configured = None


def _configure(cfg):
    global _configured
    if _configured != cfg:
        hoccl.set_config(**cfg)
        _configured = cfg


def prepare(case, seed):
    cfg = {k: case.get(k, v) for k, v in _DEFAULTS.items()}
    st = {"case": case, "cfg": cfg, "send": _inputs(case, seed)}
    if case["op"] == "ring_hop":
        st["out"] = torch.empty(case["n"], dtype=_DT[_hop_out(case)], device="cuda")
    else:
        st["recv"] = [torch.empty(n, dtype=_DT[case["dtype"]], device="cuda") for n in _recv_sizes(case)]
    if case["op"] == "sendrecv":
        st["peers"] = [(r + 1) % case["R"] for r in range(case["R"])]       # a pipeline's ring
    if case["op"] == "alltoallv":
        st["counts"], st["sd"], st["rd"] = _a2av(case)
    hoccl.init()
    _configure(cfg)
    return st


def run(st):
    _configure(st["cfg"])
    case = st["case"]
    op = case["op"]
    if op == "allreduce":
        return hoccl.allreduce(st["send"], st["recv"])
    if op == "reduce_scatter":
        return hoccl.reduce_scatter(st["send"], st["recv"])
    if op == "allgather":
        return hoccl.allgather(st["send"], st["recv"])
    if op == "sendrecv":
        return hoccl.sendrecv(st["send"], st["recv"], st["peers"])
    if op == "alltoallv":
        return hoccl.alltoallv(st["send"], st["counts"], st["sd"], st["recv"], st["rd"])
    return hoccl.ring_hop(st["send"][0], st["send"][1], st["out"], hop=case["hop"])


def exact(case, seed):
    x = _inputs(case, seed)
    op, R = case["op"], case["R"]
    if op == "allgather":
        whole = torch.cat(x)
        return [whole] * R
    if op == "sendrecv":
        return [x[(r - 1) % R] for r in range(R)]
    if op == "alltoallv":
        counts, sd, _ = _a2av(case)
        return [torch.cat([x[s][sd[s * R + d]:sd[s * R + d] + counts[s * R + d]] for s in range(R)]) for d in range(R)]
    wide = torch.int64 if case["dtype"] == "int32" else torch.float64
    total = x[0].to(wide)
    for t in x[1:]:
        total += t.to(wide)
    if wide == torch.int64:                                 # sums wrap modulo 2^32
        total = (total + 2 ** 31) % 2 ** 32 - 2 ** 31
        total = total.to(torch.int32)
    if op == "ring_hop":
        return total
    return [total] * R if op == "allreduce" else list(total.split(case["n"]))


def work(case):
    """Every input read once, every output written once, and the additions."""
    op, R, es = case["op"], case["R"], _ES[case["dtype"]]
    if op == "ring_hop":
        wide = case["dtype"] == "bf16" and case["hop"] in ("middle", "last")
        return {"bytes": case["n"] * ((4 if wide else es) + es + _ES[_hop_out(case)]), "flops": case["n"]}
    out = sum(_recv_sizes(case))
    if op in ("allgather", "sendrecv", "alltoallv"):
        sent = out if op != "allgather" else R * case["n"]
        if op == "alltoallv":
            return {"bytes": 2 * out * es, "flops": 0}
        return {"bytes": (sent + out) * es, "flops": 0}
    per_rank = case["n"] if op == "allreduce" else R * case["n"]
    return {"bytes": (R * per_rank + out) * es, "flops": (R - 1) * per_rank}


def tolerance(case):
    """Copies and whole numbers are exact.  Sums: what one rounding of the
    result to its type gives (bf16 2^-9 at most, about 1.7e-3 over a tensor;
    fp32 sums of up to 32 terms below 3e-7), four times over.  With bf16
    partials each of the R - 1 additions rounds."""
    if case["op"] in ("allgather", "sendrecv", "alltoallv") or case["dtype"] == "int32":
        return "exact"
    out = _hop_out(case) if case["op"] == "ring_hop" else case["dtype"]
    if out == "fp32":
        return {"rel": 1e-6, "max": 1e-5}
    if case.get("bf16_partials"):
        return {"rel": 6e-3 * math.sqrt(case["R"]), "max": 1e-2 * case["R"]}
    return {"rel": 7e-3, "max": 1.6e-2}
