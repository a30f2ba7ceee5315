// Internal types shared by the planner, the executor and the kernels.
#pragma once

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/hoccl.h"

namespace hoccl {

enum class Op : int {
    AllReduce = 0,
    ReduceScatter = 1,
    AllGather = 2,
    SendRecv = 3,
    AllToAll = 4,
    AllToAllV = 5
};

// A symbolic buffer position: which buffer (send[rank], recv[rank] or the
// library workspace) and a byte offset into it.  Plans are built on these so
// the planner never touches device memory and can be dumped and replayed on
// the host.
enum BufKind : uint8_t { BUF_NONE = 0, BUF_SEND = 1, BUF_RECV = 2, BUF_WS = 3 };

struct BufRef {
    uint8_t kind = BUF_NONE;
    int rank = 0;
    size_t off = 0;  // bytes
};

// Element types a reduction step reads and writes.  The local contribution
// (in1) is always of the collective's dtype; in0 and out are either the
// dtype itself or the accumulator type (fp32 for bf16, the dtype otherwise).
enum Phase : int {
    PH_FIRST = 0,   // in0 = x[j+1] (dtype),  in1 = x[j+2],  out = partial (acc)
    PH_MIDDLE = 1,  // in0 = partial (acc),   in1 = x[r],    out = partial (acc)
    PH_LAST = 2,    // in0 = partial (acc),   in1 = x[j],    out = recv (dtype)
    PH_ONLY = 3     // R == 2: in0 = x[j+1],  in1 = x[j],    out = recv (dtype)
};

struct ReduceSeg {
    BufRef in0, in1, out;
    std::vector<BufRef> more;  // further contributions, added after in1 in order
    size_t n = 0;  // elements
};

// One ring step: every rank adds its contribution to the partial it
// received; one kernel launch covers all ranks' segments of the step.  A
// fused step folds `hops` consecutive ring hops in one launch: each segment
// adds in1 and then the `more` contributions to its partial, which stays in
// registers between the adds.
struct ReduceStep {
    Phase phase = PH_MIDDLE;
    int group = 0;
    int step = 0;   // the first ring hop the launch performs
    int hops = 1;
    // The launch walks its segments from their ends.  Every other step of a
    // ring does, so that a step first reads the partials that the one before
    // wrote last and the caches still hold (kBackBytes).
    bool back = false;
    std::vector<ReduceSeg> segs;
};

// Ring steps alternate their direction where a step's partials take at least
// this much and a partial is read by more than one launch.  R = 8, n =
// 3,145,728 (100 MB of fp32 partials): 241 us alternating, 252 all forward;
// fp32 308 and 319; bf16 partials 159 and 171; R = 12, n = 1,000,000 (48 MB):
// 199 and 234; R = 32, n = 300,000 (38 MB): 446 and 513; R = 16, n = 300,001
// (19 MB): 128 and 130.  Less is in the 32 MB of L2 whichever way (R = 10, n
// = 400,000, 16 MB: 65.7 and 66.1; R = 12, int32, n = 200,000, 10 MB: 81.9 and
// 80.2).  Two launches gain nothing (R = 7 in hops of 4: 53.2 and 53.4; R =
// 5, fp32, in hops of 2: 83.2 and 80.5).
constexpr size_t kBackBytes = (size_t)16 << 20;

// Ring hops one fused launch may fold (contributions per segment).
constexpr int kMaxHops = 8;

// Direct reduction: one launch folds all R inputs of every chunk in the ring
// order.  Chunk j spans elements [j*c, min(total, (j+1)*c)) of the inputs;
// its result goes to recv[j] at out_off(j) (reduce-scatter) or to every
// recv[r] at the chunk's own offset (all-reduce, write_all).
struct FoldStep {
    size_t c = 0;        // chunk length in elements
    size_t total = 0;    // input elements per rank covered by the fold
    bool write_all = false;
    bool out_at_chunk = false;  // reduce-scatter: recv[j] at 0; else j*c
};

// One copy: `bytes` from src to dst.  Copies with the same chain run in
// order (the ring hops of one chunk); different chains are independent.  A
// copy with group >= 0 may only start once the reduction of that group has
// finished (all-reduce's gather phase).  `level` is the copy's position in
// its chain, used to batch independent copies into one CU-copy launch.
struct CopyOp {
    BufRef dst, src;
    size_t bytes = 0;
    int chain = 0;
    int group = -1;
    int level = 0;
    int stage = -1;  // all-to-all stage of the collective scheduler, or -1
};

struct Plan {
    Op op = Op::AllReduce;
    hoccl_dtype_t dtype = HOCCL_FP32;
    int R = 1;
    size_t count = 0;
    int ngroups = 1;
    std::vector<ReduceStep> reduce_steps;  // in launch order, grouped
    bool has_fold = false;
    FoldStep fold;
    std::vector<CopyOp> copies;            // in issue order
    int nchains = 0;
    size_t ws_bytes = 0;                   // workspace the plan needs
    bool bf16_partials = false;            // bf16 partials, rounded at every add
    unsigned long long hbm_bytes = 0;      // algorithmic HBM bytes
    unsigned long long copy_bytes = 0;
};

struct PlanOptions {
    bool allgather_direct = false;
    int allreduce_groups = 1;  // 0: automatic (plan_allreduce)
    size_t chunk_bytes = 0;
    bool in_place = false;
    hoccl_reduce_algo_t algo = HOCCL_REDUCE_RING;
    // Ring reductions run group by group, each group's fp32 partials taking
    // at most this many bytes (0: one group), so that they stay in the
    // last-level cache from one step to the next.
    size_t group_partial_bytes = 0;
    // Ring hops per reduction launch (0 or 1: one; at most kMaxHops).
    int fused_hops = 1;
    // All-to-all(v) copy schedule (hoccl_config_t.a2a_schedule): 0 byte-
    // balanced chains; 1 and 2 the stages of the collective scheduler's
    // decomposition (copies tagged with their stage; 2 runs them serially).
    int a2a_schedule = 0;
    // bf16 reductions keep their partials in bf16, rounding every addition
    // (hoccl_config_t.bf16_partials).
    bool bf16_partials = false;
};

// HOCCL_REDUCE_AUTO folds directly up to this many ranks.  On one GPU the
// fold moves (R+1) elements per reduce-scatter output element against the
// ring's 2(R-1) (plus the fp32 partials of bf16), so it is the faster
// schedule at every size measured; beyond this rank count the ring is used.
constexpr int kDirectMaxRanks = 64;
bool use_direct(hoccl_reduce_algo_t algo, int R);

size_t dtype_size(hoccl_dtype_t dt);
// Bytes of one partial-sum element: 4 (fp32 for bf16), 2 for bf16 with
// bf16 partials.
size_t acc_size(hoccl_dtype_t dt, bool bf16_partials = false);

// Planner entry points (plan.cpp); pure host code.
Plan plan_allreduce(size_t count, hoccl_dtype_t dt, int R, const PlanOptions &o);
Plan plan_reduce_scatter(size_t recvcount, hoccl_dtype_t dt, int R, const PlanOptions &o);
Plan plan_allgather(size_t sendcount, hoccl_dtype_t dt, int R, const PlanOptions &o);
Plan plan_sendrecv(size_t count, hoccl_dtype_t dt, int R, const int *peers,
                   const PlanOptions &o);
Plan plan_alltoall(size_t count, hoccl_dtype_t dt, int R, const PlanOptions &o);
Plan plan_alltoallv(const size_t *counts, const size_t *sdispls, const size_t *rdispls,
                    hoccl_dtype_t dt, int R, const PlanOptions &o);

// Assigns each chain of a plan to one of `queues` queues so that the bytes
// per queue are balanced (largest chain first, onto the least loaded queue).
std::vector<int> assign_chains(const Plan &p, int queues);

std::string plan_to_json(const Plan &p);

// ---- kernels (kernels.hip) -------------------------------------------------

constexpr int kMaxReduceSegs = 64;
constexpr int kMaxCopySegs = 128;
constexpr int kMaxRanks = 64;

// Each kernel's argument struct has a fixed number of slots.  The executor
// fills the largest form; the launchers pass the smallest form that holds the
// launch's segments.  The HIP runtime stages the arguments of every launch
// that has not started yet, and the enqueueing thread waits once about 1 MB
// of them is pending (measured on MI355X).  With 2 KiB of slots, some 450
// launches queued behind unfinished work stall the caller; an 8-rank ring
// step passes 272 bytes (plus the runtime's own 256 bytes of hidden
// arguments), and about 1000 fit.
struct RSegArg {
    const void *in0;
    const void *in1;
    void *out;
    uint64_t n;
};
template <int CAP>
struct ReduceArgsT {
    RSegArg seg[CAP];
    int nseg;
    uint32_t threads;  // per workgroup; set at the launch
    int back;          // ReduceStep::back
};
using ReduceArgs = ReduceArgsT<kMaxReduceSegs>;

// A fused step's segment: the partial (or first operand) in0, then nloc
// contributions loc[0..nloc) added in order, into out.
struct MSegArg {
    const void *in0;
    const void *loc[kMaxHops];
    void *out;
    uint64_t n;
    int nloc;
};
constexpr int kMaxMultiSegs = 32;  // 32 segments: 3.1 KiB of arguments
template <int CAP>
struct MultiArgsT {
    MSegArg seg[CAP];
    int nseg;
    uint32_t threads;  // per workgroup; set at the launch
    int back;          // ReduceStep::back
};
using MultiArgs = MultiArgsT<kMaxMultiSegs>;

// A copy segment: one source and its nd destinations (at most ND).  `first`
// is the segments' row of tiles (copy_layout).
template <int ND>
struct CSegArgT {
    const void *src;
    void *dst[ND];
    uint64_t bytes;
    int nd;
};
template <>
struct CSegArgT<1> {
    const void *src;
    void *dst[1];
    uint64_t bytes;
    static constexpr int nd = 1;
};
template <int CAP, int ND>
struct CopyArgsT {
    CSegArgT<ND> seg[CAP];
    uint32_t first[CAP + 1];
    uint32_t unroll;   // 16-byte vectors per thread of a tile
    uint32_t row;      // the workgroups walk the row of tiles, not a segment each
    int nseg;
    uint32_t threads;  // per workgroup; set at the launch
};
using CopyArgs = CopyArgsT<kMaxCopySegs, 1>;
// Copies that read the same bytes share a segment of up to kMaxFan
// destinations: 32 segments take 3 KiB of arguments.
constexpr int kMaxFan = 8;
constexpr int kMaxFanSegs = 32;
using FanArgs = CopyArgsT<kMaxFanSegs, kMaxFan>;

template <int CAP>
struct FoldArgsT {
    const void *in[CAP];
    void *out[CAP];
    uint64_t c;
    uint64_t total;
    int R;
    int write_all;
    int out_at_chunk;
    uint32_t threads;  // per workgroup; set at the launch
};
using FoldArgs = FoldArgsT<kMaxRanks>;

// The stream side of one proxy operation's start/finish handshake.  The
// three flags are host memory mapped for the device.
struct HandshakeArgs {
    uint32_t *start;        // the kernel writes start_value; the proxy clears it
    uint32_t *finish;       // the proxy writes finish_value; the kernel clears it
    uint32_t *status;       // the kernel writes 1 here if it gave up waiting
    uint32_t start_value;
    uint32_t finish_value;
    uint64_t limit_ticks;   // give up after this many device wall-clock ticks
};

// bf16_partials: a bf16 step keeps every operand and result in bf16 (the
// middle and last phases read, and the first and middle write, bf16
// partials); a bf16 fold, or fused step, rounds after every addition.
hipError_t launch_reduce_step(hoccl_dtype_t dt, Phase ph, const ReduceArgs &a, int wg,
                              int threads, hipStream_t s, bool bf16_partials = false);
hipError_t launch_fold(hoccl_dtype_t dt, const FoldArgs &a, int wg, int threads,
                       hipStream_t s, bool bf16_partials = false, size_t lds = 0);
hipError_t launch_multihop(hoccl_dtype_t dt, Phase ph, const MultiArgs &a, int wg, int threads,
                           hipStream_t s, bool bf16_partials = false);
// Copies: copy_layout lays a launch's tiles out (call it before the launch) for
// a workgroup budget (0: none) and returns the workgroups to launch.
uint32_t copy_layout(CopyArgs &a, int threads, int budget);
uint32_t copy_layout(FanArgs &a, int threads, int budget);
hipError_t launch_copy(const CopyArgs &a, int wg, int threads, hipStream_t s, size_t lds);
hipError_t launch_fan(const FanArgs &a, int wg, int threads, hipStream_t s, size_t lds);
// LDS that a launch asks for to bound the workgroups a CU holds, on the whole
// chip and without a workgroup budget (else the caller asks for none).
size_t fold_lds(hoccl_dtype_t dt, const FoldArgs &a, int threads);
inline size_t copy_lds(const CopyArgs &, int) { return 0; }
size_t copy_lds(const FanArgs &a, int threads);

// Elements of the collective's dtype one thread covers in one pass of each
// kernel's main loop.
size_t reduce_step_elems_per_thread(hoccl_dtype_t dt, Phase ph, bool bf16_partials = false);
size_t fold_elems_per_thread(hoccl_dtype_t dt);
size_t multihop_elems_per_thread(hoccl_dtype_t dt);
hipError_t launch_handshake(const HandshakeArgs &a, hipStream_t s);

// The static device scratch of hoccl_reduce_scatter_noalloc (scratch.hip):
// its size, and this device's address of it (call with the device current).
constexpr size_t kScratchBytes = (size_t)128 << 20;
hipError_t scratch_address(void **out);

}  // namespace hoccl
