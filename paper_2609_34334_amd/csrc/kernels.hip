// gfx950 kernels of the collective hot path.
//
// * reduce_step_kernel -- one ring reduction step for every virtual rank at
//   once: out[i] = in0[i] + in1[i], where in0 is the partial received from
//   the previous rank (or, on the first step, that rank's own element) and
//   in1 is this rank's element.  bf16 partials are carried in fp32.
// * fold_kernel        -- the direct variant: folds all R inputs of a chunk
//   in the ring order in one pass (same result bit for bit, fewer bytes).
// * copy_kernel        -- a CU copy of many independent segments, each one
//   source and one or several destinations; the comparator for the SDMA
//   copy path.
//
// All three are HBM-bound streams (about one add per 8-12 bytes), so they
// use 16-byte vector loads and stores, a grid-stride loop over each segment
// with several independent vectors in flight per thread, and neither share
// data through LDS nor need MFMA: the limit is memory bandwidth, not
// arithmetic.  (Some launches ask for LDS all the same, to bound the
// workgroups in flight: fold_lds, copy_lds.)
//
// Where a comment compares two forms of the code, both sides are from one run
// of the code as it then was.  Later steps moved both, so that only the
// difference holds.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "hoccl_internal.h"

namespace hoccl {
namespace {

// ---- element types ----------------------------------------------------------
// S is the storage type in memory, A the accumulator type of the fold.
struct TBF16 {
    using S = uint16_t;
    using A = float;
    static __device__ __forceinline__ float widen(uint16_t v) {
        return __uint_as_float((uint32_t)v << 16);  // exact
    }
    static __device__ __forceinline__ uint16_t narrow(float f) {
        // v_cvt_pk_bf16_f32: round to nearest even, NaN stays NaN
        return __builtin_bit_cast(uint16_t, (__bf16)f);
    }
};
struct TF32 {
    using S = float;
    using A = float;
    static __device__ __forceinline__ float widen(float v) { return v; }
    static __device__ __forceinline__ float narrow(float f) { return f; }
};
struct TI32 {
    using S = uint32_t;
    using A = uint32_t;  // unsigned: adds wrap modulo 2^32
    static __device__ __forceinline__ uint32_t widen(uint32_t v) { return v; }
    static __device__ __forceinline__ uint32_t narrow(uint32_t v) { return v; }
};

// VE elements in one vector register group.  It is aligned like its element
// only: ldp and stp below move it in 8- or 16-byte accesses at any element
// address.
template <typename S, int VE>
struct Pack {
    S v[VE];
};

// Tuning knobs (compile time).  Vectors in flight per thread in the ring
// step, and whether streamed operands use non-temporal loads / stores.
#ifndef HOCCL_RS_UNROLL_BF16
#define HOCCL_RS_UNROLL_BF16 2
#endif
#ifndef HOCCL_RS_UNROLL_32
#define HOCCL_RS_UNROLL_32 4
#endif
// Non-temporal access for operands touched once per collective: the ranks'
// inputs (HOCCL_NT_X) and the final output (HOCCL_NT_FINAL).  Partials are
// always accessed normally so that the next step can hit the cache.
#ifndef HOCCL_NT_X
#define HOCCL_NT_X 1
#endif
#ifndef HOCCL_NT_FINAL
#define HOCCL_NT_FINAL 0
#endif
#ifndef HOCCL_FOLD_NT
#define HOCCL_FOLD_NT 1
#endif
#ifndef HOCCL_FOLD_NT_OUT
#define HOCCL_FOLD_NT_OUT 1
#endif
// Whether the CU copy's stores are non-temporal.  Normal ones made the EP
// all-to-all(v) 6% slower and a 128 MiB send/recv 3%.
#ifndef HOCCL_COPY_NT_OUT
#define HOCCL_COPY_NT_OUT 1
#endif
// bit 0: in0 non-temporal, bit 1: in1, bit 2: out
constexpr int kNtFirst = (HOCCL_NT_X ? 3 : 0);
constexpr int kNtMiddle = (HOCCL_NT_X ? 2 : 0);
constexpr int kNtLast = (HOCCL_NT_X ? 2 : 0) | (HOCCL_NT_FINAL ? 4 : 0);
constexpr int kNtOnly = (HOCCL_NT_X ? 3 : 0) | (HOCCL_NT_FINAL ? 4 : 0);

// Lane layout of the ring step.  A lane holds VE consecutive elements of
// every operand.  Where bf16 meets fp32 partials, VE = 4: a lane moves 8 B
// of bf16 and 16 B of fp32, so each load or store instruction of a wave
// covers one contiguous span (512 B or 1 KiB).  With VE = 8 the fp32 side
// would take two 16-byte accesses 32 B apart per lane, each instruction
// touching every line of a 2 KiB span half; that layout ran the headline
// reduce-scatter about 5% slower.  bf16-only steps keep 16-byte vectors.
constexpr int kVeBf16Partial = 4;
constexpr int kVeBf16Only = 8;
constexpr int kVe32 = 4;
constexpr int kDeepCopy = 4;  // vectors per thread of a deep copy tile (copy_layout)
constexpr int kWideFan = 5;   // destinations from which a copy is write-bound (copy_layout)

// Byte-aligned vectors.  The compute units take a 16-byte global access at any
// byte address (the HSA target runs with unaligned access enabled), so the
// same instruction serves aligned and misaligned operands.  A misaligned
// stream costs almost nothing where HBM is the limit, as a wave's 1 KiB span
// only touches one line more: the bf16 fold into shards of odd length takes
// 2% longer at R = 6, n = 1,398,103 than at n + 1 and 1% at R = 8,
// n = 3,145,727, where an element-by-element fallback took 2.3 and 1.3 times
// as long, and 1.6 times for four fused ring hops of the latter.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2), aligned(1)));

// Vector load / store of a Pack in 16-byte pieces (8 bytes for an 8-byte
// Pack), optionally non-temporal.
template <bool NT, typename P>
__device__ __forceinline__ P ldp(const P *p) {
    static_assert(sizeof(P) == 8 || sizeof(P) % 16 == 0, "Pack must be 8 bytes or a multiple of 16");
    P r;
    if constexpr (sizeof(P) == 8) {
        u32x2 v = NT ? __builtin_nontemporal_load((const u32x2 *)p) : *(const u32x2 *)p;
        __builtin_memcpy(&r, &v, 8);
    } else {
#pragma unroll
        for (int i = 0; i < (int)(sizeof(P) / 16); ++i) {
            u32x4 v = NT ? __builtin_nontemporal_load((const u32x4 *)p + i) : ((const u32x4 *)p)[i];
            __builtin_memcpy((char *)&r + 16 * i, &v, 16);
        }
    }
    return r;
}
template <bool NT, typename P>
__device__ __forceinline__ void stp(P *p, const P &x) {
    if constexpr (sizeof(P) == 8) {
        u32x2 v;
        __builtin_memcpy(&v, &x, 8);
        if (NT)
            __builtin_nontemporal_store(v, (u32x2 *)p);
        else
            *(u32x2 *)p = v;
    } else {
#pragma unroll
        for (int i = 0; i < (int)(sizeof(P) / 16); ++i) {
            u32x4 v;
            __builtin_memcpy(&v, (const char *)&x + 16 * i, 16);
            if (NT)
                __builtin_nontemporal_store(v, (u32x4 *)p + i);
            else
                ((u32x4 *)p)[i] = v;
        }
    }
}

// Where a segment's vectors start: the first element at which `p` reaches a
// cache line (128 bytes).  A wave's span of a line-aligned stream is whole
// lines; from any other 16-byte boundary, every span shares its first and
// last line with its neighbours', and the writes of both are parts of lines:
// aligned to 16 bytes only, the gather of six shards of 3,333,333 bytes took
// 32% longer, an fp32 all-reduce of 1,500,007 elements at R = 16 9%, one of
// 2,100,001 bf16 at R = 12 8%.
constexpr uint32_t kLineBytes = 128;
template <typename S>
__device__ __forceinline__ uint64_t head_of(const S *p, uint64_t n) {
    const uint64_t h = ((kLineBytes - ((uintptr_t)p & (kLineBytes - 1))) & (kLineBytes - 1)) / sizeof(S);
    return h < n ? h : n;
}

// The elements before the vectors (h of them) and after (from `tail` to n),
// one per lane: f(k).  They go to the last block of the segment, from its last
// lane down: that block's vectors mostly end before its lanes do, so that its
// idle waves take them (the all-reduce at R = 16 above: 13% less than with the
// first block's lanes).  Every wave runs the loop's test, on purpose: the
// eight-rank fold, whose waves all start with it, took 8% longer at
// n = 3,145,728 (bf16) with a uniform branch around the loop.
template <typename F>
__device__ __forceinline__ void for_each_edge(uint64_t h, uint64_t tail, uint64_t n, int lb, int nb, uint32_t bd,
                                              F &&f) {
    const uint64_t back = (uint64_t)(nb - 1 - lb) * bd + (bd - 1 - threadIdx.x);
    for (uint64_t k = back; k < h + (n - tail); k += (uint64_t)nb * bd) f(k < h ? k : tail + (k - h));
}

// Workgroups are dealt to the GPU's eight XCDs, each with an L2, in turn.
constexpr int kXcds = 8;

// Splits the blocks of a launch over `nseg` segments; f(seg, lb, nb) is block
// lb of the nb blocks of segment seg.  With fewer blocks than segments each
// block walks several segments.  Otherwise
// * IN_TURN: block b serves segment b % nseg.  The ring's steps take this
//   one: at 8 ranks chunk j then stays on XCD j from step to step (headline:
//   1 to 2% less than with runs of blocks).
// * else a run of consecutive blocks serves each segment, so that the launch
//   sweeps the segments one after another and the blocks in flight read and
//   write a few narrow windows of memory instead of nseg times as many.  The
//   fold at R = 8, n = 3,145,728 (bf16) takes 74.3 us so and 78.6 in turn,
//   at R = 7 71.9 and 84.1.  (Runs of blocks per XCD are no better than in
//   turn: 78.9 and 77.7.)
// `back` turns the blocks' order round, in groups of kXcds so that every part
// of a segment stays on its XCD (ReduceStep::back says where and why).
template <bool IN_TURN, typename F>
__device__ __forceinline__ void for_each_segment(int nseg, bool back, F &&f) {
    const int g = (int)gridDim.x;
    int b = (int)blockIdx.x;
    if (back) {
        const int whole = g & ~(kXcds - 1);  // a rest of the grid keeps its place
        if (b < whole) b = whole - kXcds - (b & ~(kXcds - 1)) + (b & (kXcds - 1));
    }
    if (g >= nseg && IN_TURN) {
        int seg = b % nseg;
        f(seg, b / nseg, (g - seg + nseg - 1) / nseg);
    } else if (g >= nseg) {
        // The first `more` segments get q + 1 blocks, the others q.
        const int q = g / nseg, more = g % nseg, c = b - more * (q + 1);
        if (c < 0)
            f(b / (q + 1), b % (q + 1), q + 1);
        else
            f(more + c / q, c % q, q);
    } else {
        for (int seg = b; seg < nseg; seg += g) f(seg, 0, 1);
    }
}

// ---- one ring step --------------------------------------------------------------
template <class T0, class T1, class TO, int VE, int U, int NT>
__device__ __forceinline__ void reduce_segment(const RSegArg &s, int lb, int nb, uint32_t threads) {
    constexpr bool NT0 = NT & 1, NT1 = NT & 2, NTO = NT & 4;
    using S0 = typename T0::S;
    using S1 = typename T1::S;
    using SO = typename TO::S;
    using P0 = Pack<S0, VE>;
    using P1 = Pack<S1, VE>;
    using PO = Pack<SO, VE>;
    const S0 *in0 = (const S0 *)s.in0;
    const S1 *in1 = (const S1 *)s.in1;
    SO *out = (SO *)s.out;
    const uint64_t n = s.n;

    // in0 and out mostly reach a line with in1; where they do not (the ring's
    // last step into an output shard whose length is odd), their vectors are
    // misaligned.
    const uint64_t h = head_of(in1, n);
    const uint64_t nv = (n - h) / VE;
    const uint64_t tail = h + nv * VE;

    const uint64_t bd = threads;
    const uint64_t stride = (uint64_t)nb * bd;
    for_each_edge(h, tail, n, lb, nb, threads,
                  [&](uint64_t k) { out[k] = TO::narrow(T0::widen(in0[k]) + T1::widen(in1[k])); });

    const P0 *v0 = (const P0 *)(in0 + h);
    const P1 *v1 = (const P1 *)(in1 + h);
    PO *vo = (PO *)(out + h);
    auto one = [&](const P0 &a, const P1 &b) {
        PO y;
#pragma unroll
        for (int e = 0; e < VE; ++e) y.v[e] = TO::narrow(T0::widen(a.v[e]) + T1::widen(b.v[e]));
        return y;
    };
    // Main loop: U vectors per thread, all in range, loads issued before use.
    uint64_t base = (uint64_t)lb * bd * U + threadIdx.x;
    for (; base + (uint64_t)(U - 1) * bd < nv; base += stride * U) {
        P0 a[U];
        P1 b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            a[u] = ldp<NT0>(v0 + base + (uint64_t)u * bd);
            b[u] = ldp<NT1>(v1 + base + (uint64_t)u * bd);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) stp<NTO>(vo + base + (uint64_t)u * bd, one(a[u], b[u]));
    }
    // At most one partial iteration is left for this thread.
#pragma unroll
    for (int u = 0; u < U; ++u) {
        uint64_t i = base + (uint64_t)u * bd;
        if (i < nv) stp<NTO>(vo + i, one(ldp<NT0>(v0 + i), ldp<NT1>(v1 + i)));
    }
}

template <typename A>
__device__ __forceinline__ const A &kernargs();

template <class T0, class T1, class TO, int VE, int U, int NT, int CAP>
__global__ void __launch_bounds__(1024) reduce_step_kernel(ReduceArgsT<CAP>) {
    const ReduceArgsT<CAP> &a = kernargs<ReduceArgsT<CAP>>();
    for_each_segment<true>(a.nseg, a.back, [&](int seg, int lb, int nb) {
        reduce_segment<T0, T1, TO, VE, U, NT>(a.seg[seg], lb, nb, a.threads);
    });
}

// ---- fused ring hops ---------------------------------------------------------------
// One launch folds several consecutive ring hops of every segment: the
// partial (or, on the ring's first hop, the previous rank's own element) is
// loaded once, the nloc contributions are added to it in the ring's order
// while it stays in registers, and the result is stored once.  The adds are
// the ring's adds in the ring's order, so the bits are the ring's; only the
// partial's round trips through memory between the fused hops are gone.
// nloc is the same for every lane, so the guards on the unrolled
// contribution loop are uniform branches.
template <class T0, class T1, class TO, int VE, int U, int NT, int MAXL, bool RH>
__device__ __forceinline__ void multihop_segment(const MSegArg &s, int lb, int nb, uint32_t threads) {
    constexpr bool NT0 = NT & 1, NT1 = NT & 2, NTO = NT & 4;
    using S0 = typename T0::S;
    using S1 = typename T1::S;
    using SO = typename TO::S;
    using A = typename T1::A;
    // RH: every addition's result is rounded to the contribution's type
    // before the next (bf16 partials), as separate hops would round it.
    auto add = [](A acc, S1 x) -> A {
        A y = acc + T1::widen(x);
        if constexpr (RH) y = T1::widen(T1::narrow(y));
        return y;
    };
    using P0 = Pack<S0, VE>;
    using P1 = Pack<S1, VE>;
    using PO = Pack<SO, VE>;
    const S0 *in0 = (const S0 *)s.in0;
    SO *out = (SO *)s.out;
    const int nl = s.nloc;
    const uint64_t n = s.n;
    const S1 *loc[MAXL];
#pragma unroll
    for (int m = 0; m < MAXL; ++m) loc[m] = m < nl ? (const S1 *)s.loc[m] : (const S1 *)s.loc[0];

    // The operands that do not reach a line with the first contribution are
    // read or written misaligned.
    const uint64_t h = head_of(loc[0], n);
    const uint64_t nv = (n - h) / VE;
    const uint64_t tail = h + nv * VE;

    const uint64_t bd = threads;
    const uint64_t stride = (uint64_t)nb * bd;
    for_each_edge(h, tail, n, lb, nb, threads, [&](uint64_t k) {
        const S0 a = in0[k];
        S1 b[MAXL];
#pragma unroll
        for (int m = 0; m < MAXL; ++m)
            if (m < nl) b[m] = loc[m][k];
        A acc = T0::widen(a);
#pragma unroll
        for (int m = 0; m < MAXL; ++m)
            if (m < nl) acc = add(acc, b[m]);
        out[k] = TO::narrow(acc);
    });

    const P0 *v0 = (const P0 *)(in0 + h);
    const P1 *vl[MAXL];
#pragma unroll
    for (int m = 0; m < MAXL; ++m) vl[m] = (const P1 *)(loc[m] + h);
    PO *vo = (PO *)(out + h);
    auto one = [&](uint64_t i) {
        P0 a = ldp<NT0>(v0 + i);
        P1 b[MAXL];
#pragma unroll
        for (int m = 0; m < MAXL; ++m)
            if (m < nl) b[m] = ldp<NT1>(vl[m] + i);
        A acc[VE];
#pragma unroll
        for (int e = 0; e < VE; ++e) acc[e] = T0::widen(a.v[e]);
#pragma unroll
        for (int m = 0; m < MAXL; ++m)
            if (m < nl)
#pragma unroll
                for (int e = 0; e < VE; ++e) acc[e] = add(acc[e], b[m].v[e]);
        PO y;
#pragma unroll
        for (int e = 0; e < VE; ++e) y.v[e] = TO::narrow(acc[e]);
        stp<NTO>(vo + i, y);
    };
    // Main loop: U vectors of every operand per thread, all in range, every
    // load issued before the adds consume them.
    uint64_t base = (uint64_t)lb * bd * U + threadIdx.x;
    for (; base + (uint64_t)(U - 1) * bd < nv; base += stride * U) {
        P0 a[U];
        P1 b[U][MAXL];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = ldp<NT0>(v0 + base + (uint64_t)u * bd);
#pragma unroll
        for (int m = 0; m < MAXL; ++m)
            if (m < nl)
#pragma unroll
                for (int u = 0; u < U; ++u) b[u][m] = ldp<NT1>(vl[m] + base + (uint64_t)u * bd);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            A acc[VE];
#pragma unroll
            for (int e = 0; e < VE; ++e) acc[e] = T0::widen(a[u].v[e]);
#pragma unroll
            for (int m = 0; m < MAXL; ++m)
                if (m < nl)
#pragma unroll
                    for (int e = 0; e < VE; ++e) acc[e] = add(acc[e], b[u][m].v[e]);
            PO y;
#pragma unroll
            for (int e = 0; e < VE; ++e) y.v[e] = TO::narrow(acc[e]);
            stp<NTO>(vo + base + (uint64_t)u * bd, y);
        }
    }
    // At most one partial iteration is left for this thread.
#pragma unroll
    for (int u = 0; u < U; ++u) {
        uint64_t i = base + (uint64_t)u * bd;
        if (i < nv) one(i);
    }
}

template <class T0, class T1, class TO, int VE, int U, int NT, int MAXL, int CAP, bool RH>
__global__ void __launch_bounds__(1024) multihop_kernel(MultiArgsT<CAP>) {
    const MultiArgsT<CAP> &a = kernargs<MultiArgsT<CAP>>();
    for_each_segment<true>(a.nseg, a.back, [&](int seg, int lb, int nb) __attribute__((always_inline)) {
        multihop_segment<T0, T1, TO, VE, U, NT, MAXL, RH>(a.seg[seg], lb, nb, a.threads);
    });
}

// ---- direct fold ------------------------------------------------------------------
// Chunk j reads x[(j+1)%R], x[(j+2)%R], ..., x[j] at the chunk's elements and
// adds them left to right; loads are issued in batches of KB ranks so several
// are in flight before the adds consume them in order.  RH rounds every
// addition's result to the element type before the next addition (the
// partials a ring of bf16 forwarding ranks would hold).
template <class T, int VE, int NR, bool RH, class FA>
__device__ __forceinline__ void fold_chunk(const FA &a, int j, int lb, int nb) {
    using S = typename T::S;
    using A = typename T::A;
    using P = Pack<S, VE>;
    auto add = [](A acc, S x) -> A {
        A y = acc + T::widen(x);
        if constexpr (RH) y = T::widen(T::narrow(y));
        return y;
    };
    const int R = NR > 0 ? NR : a.R;
    const uint64_t e0 = (uint64_t)j * a.c;
    if (e0 >= a.total) return;
    const uint64_t n = (a.total - e0 < a.c) ? a.total - e0 : a.c;
    // k-th operand of chunk j's fold (k = 0 .. R-1) is rank (j + 1 + k) mod R.
    auto src = [&](int k) -> const S * {
        int r = j + 1 + k;
        if (r >= R) r -= R;
        if (r >= R) r -= R;
        return (const S *)a.in[r] + e0;
    };
    const uint64_t oe = a.out_at_chunk ? 0 : e0;
    const int nout = a.write_all ? R : 1;
    auto dst = [&](int q) -> S * { return (S *)a.out[a.write_all ? q : j] + oe; };

    // A chunk of odd length leaves the inputs' phase and the output shard's
    // apart: the reads are kept aligned (R streams) and the one write is
    // misaligned (R = 6, n = 1,398,103 bf16: 7% less than the other way).
    const uint64_t h = head_of(src(0), n);
    const uint64_t nv = (n - h) / VE;
    const uint64_t tail = h + nv * VE;

    const uint64_t bd = a.threads;
    const uint64_t t = (uint64_t)lb * bd + threadIdx.x;
    const uint64_t stride = (uint64_t)nb * bd;
    // The ranks' loads go out in batches here, too, not each after the last.
    for_each_edge(h, tail, n, lb, nb, a.threads, [&](uint64_t k) __attribute__((always_inline)) {
        constexpr int B = NR > 0 ? NR : 8;
        A acc = T::widen(src(0)[k]);
        for (int q0 = 1; q0 < R; q0 += B) {
            S x[B];
#pragma unroll
            for (int q = 0; q < B; ++q) x[q] = src(q0 + q < R ? q0 + q : 0)[k];
#pragma unroll
            for (int q = 0; q < B; ++q)
                if (q0 + q < R) acc = add(acc, x[q]);
        }
        const S y = T::narrow(acc);
        for (int q = 0; q < nout; ++q) dst(q)[k] = y;
    });

    constexpr bool NT = HOCCL_FOLD_NT;
    constexpr bool NTO = HOCCL_FOLD_NT_OUT;
    if constexpr (NR > 0) {
        // The operand and output pointers are computed once, outside the
        // loop; every operand's vector is loaded before the in-order adds
        // consume them.  Reading an output pointer from the argument buffer
        // inside the loop put a scalar load and its wait in front of every
        // store (about 7% of the headline fold's time).
        const P *sp[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) sp[k] = (const P *)(src(k) + h);
        auto run = [&](auto outs) {
            constexpr int NO = decltype(outs)::value;
            P *dp[NO];
#pragma unroll
            for (int q = 0; q < NO; ++q) dp[q] = (P *)(dst(q) + h);
            for (uint64_t i = t; i < nv; i += stride) {
                P v[NR];
#pragma unroll
                for (int k = 0; k < NR; ++k) v[k] = ldp<NT>(sp[k] + i);
                A acc[VE];
#pragma unroll
                for (int e = 0; e < VE; ++e) acc[e] = T::widen(v[0].v[e]);
#pragma unroll
                for (int k = 1; k < NR; ++k)
#pragma unroll
                    for (int e = 0; e < VE; ++e) acc[e] = add(acc[e], v[k].v[e]);
                P y;
#pragma unroll
                for (int e = 0; e < VE; ++e) y.v[e] = T::narrow(acc[e]);
#pragma unroll
                for (int q = 0; q < NO; ++q) stp<NTO>(dp[q] + i, y);
            }
        };
        if (a.write_all)
            run(std::integral_constant<int, NR>{});
        else
            run(std::integral_constant<int, 1>{});
        return;
    }
    // Any other R, in batches of KB ranks: the batch's pointers are read from
    // the argument buffer together, then its vectors are loaded together,
    // so that one scalar wait and one memory latency serve KB ranks, and the
    // output pointers likewise.  With a scalar wait before every rank's load
    // and store, and cached accesses, an fp32 all-reduce of 1,500,007
    // elements at R = 16 took 30% longer, one of 6,291,456 bf16 at R = 32 13%,
    // and a reduce-scatter of 26 MB a rank (bf16, R = 16) 17%.  Where one call
    // after another folds the same inputs, cached loads would be the faster
    // ones (R = 9, 72 MB in all: 23.4 us instead of 28.9); over inputs that
    // change they are not (31.4 instead of 30.0; R = 9, 432 MB 173 instead of
    // 160).
    constexpr int KB = 8;
    for (uint64_t i = t; i < nv; i += stride) {
        A acc[VE];
        {
            P v0 = ldp<NT>((const P *)(src(0) + h) + i);
#pragma unroll
            for (int e = 0; e < VE; ++e) acc[e] = T::widen(v0.v[e]);
        }
        int k = 1;
        for (; k + KB <= R; k += KB) {
            const P *sp[KB];
            P v[KB];
#pragma unroll
            for (int q = 0; q < KB; ++q) sp[q] = (const P *)(src(k + q) + h);
#pragma unroll
            for (int q = 0; q < KB; ++q) v[q] = ldp<NT>(sp[q] + i);
#pragma unroll
            for (int q = 0; q < KB; ++q)
#pragma unroll
                for (int e = 0; e < VE; ++e) acc[e] = add(acc[e], v[q].v[e]);
        }
        if (k < R) {
            const P *sp[KB - 1];
            P v[KB - 1];
#pragma unroll
            for (int q = 0; q < KB - 1; ++q) sp[q] = (const P *)(src(k + q < R ? k + q : 0) + h);
#pragma unroll
            for (int q = 0; q < KB - 1; ++q)
                if (k + q < R) v[q] = ldp<NT>(sp[q] + i);
#pragma unroll
            for (int q = 0; q < KB - 1; ++q)
                if (k + q < R)
#pragma unroll
                    for (int e = 0; e < VE; ++e) acc[e] = add(acc[e], v[q].v[e]);
        }
        P y;
#pragma unroll
        for (int e = 0; e < VE; ++e) y.v[e] = T::narrow(acc[e]);
        if (!a.write_all) {
            stp<NTO>((P *)(dst(0) + h) + i, y);
            continue;
        }
        for (int q0 = 0; q0 < R; q0 += KB) {
            P *dp[KB];
#pragma unroll
            for (int q = 0; q < KB; ++q) dp[q] = (P *)(dst(q0 + q < R ? q0 + q : 0) + h);
#pragma unroll
            for (int q = 0; q < KB; ++q)
                if (q0 + q < R) stp<NTO>(dp[q] + i, y);
        }
    }
}

// The argument structs are indexed with run-time rank numbers.  Reading them
// through the kernarg segment pointer keeps those reads scalar loads from the
// (read-only) argument buffer; indexing the by-value parameter instead makes
// the compiler copy the whole struct into per-thread scratch memory.
template <typename A>
__device__ __forceinline__ const A &kernargs() {
    return *(const A *)__builtin_amdgcn_kernarg_segment_ptr();
}

template <class T, int VE, int NR, int CAP, bool RH, bool IN_TURN = false>
__global__ void __launch_bounds__(1024) fold_kernel(FoldArgsT<CAP>) {
    const FoldArgsT<CAP> &a = kernargs<FoldArgsT<CAP>>();
    // Forced inline: for_each_segment calls the body from two places, and
    // the eight-rank rounding fold was otherwise left an out-of-line call
    // with a scratch frame.
    for_each_segment<IN_TURN>(a.R, false, [&](int j, int lb, int nb) __attribute__((always_inline)) {
        fold_chunk<T, VE, NR, RH>(a, j, lb, nb);
    });
}

// ---- CU copy ----------------------------------------------------------------------
// Tiles `at`, at + G, at + 2G, ... of one segment, up to its last one or not
// (`last`); a tile is U 16-byte vectors per thread.  The vectors start where the first destination
// reaches a line; a source or a further destination at another phase is read
// or written misaligned.  The bytes before and after the vectors, fewer than
// 144, go to the block of the last tile.
template <int U, int ND, bool NT_IN>
__device__ __forceinline__ void copy_tiles(const CSegArgT<ND> &s, uint32_t at, bool last, uint32_t G,
                                           uint32_t bd) {
    using V = Pack<uint32_t, 4>;  // HIP's uint4 is a union and defeats SROA
    const char *src = (const char *)s.src;
    const uint64_t n = s.bytes;
    char *dst[ND];
#pragma unroll
    for (int q = 0; q < ND; ++q) dst[q] = (char *)s.dst[q < s.nd ? q : 0];
    const uint64_t h = head_of(dst[0], n);
    const uint64_t nv = (n - h) / 16;
    const uint32_t t = threadIdx.x;
    if (last)
        for_each_edge(h, h + nv * 16, n, 0, 1, bd, [&](uint64_t k) {
            const char x = src[k];
#pragma unroll
            for (int q = 0; q < ND; ++q)
                if (q < s.nd) dst[q][k] = x;
        });
    const V *vs = (const V *)(src + h);
    const uint64_t tile = (uint64_t)bd * U, step = tile * G;
    uint64_t base = tile * at;
    for (; base + tile <= nv; base += step) {
        V v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = ldp<NT_IN>(vs + base + t + (uint64_t)u * bd);
#pragma unroll
        for (int q = 0; q < ND; ++q)
            if (q < s.nd)
#pragma unroll
                for (int u = 0; u < U; ++u)
                    stp<HOCCL_COPY_NT_OUT>((V *)(dst[q] + h) + base + t + (uint64_t)u * bd, v[u]);
    }
    // At most one tile of this block reaches past the segment's end.
    if (base >= nv) return;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint64_t i = base + t + (uint64_t)u * bd;
        if (i < nv) {
            V v = ldp<NT_IN>(vs + i);
#pragma unroll
            for (int q = 0; q < ND; ++q)
                if (q < s.nd) stp<HOCCL_COPY_NT_OUT>((V *)(dst[q] + h) + i, v);
        }
    }
}

// ROW: the tiles of all segments form one row (segment s has tiles first[s] up
// to first[s + 1]); block b takes tiles b, b + G, b + 2G, ... of it.  Otherwise
// every segment has blocks of its own that walk its tiles: one read of the
// arguments serves a block, where a step along the row takes a search and a
// read per segment.  copy_layout says which launch takes which.
template <int CAP, int ND, int U, bool NT_IN, bool ROW>
__global__ void __launch_bounds__(1024) copy_kernel(CopyArgsT<CAP, ND>) {
    const CopyArgsT<CAP, ND> &a = kernargs<CopyArgsT<CAP, ND>>();
    if constexpr (!ROW) {
        for_each_segment<true>(a.nseg, false, [&](int seg, int lb, int nb) __attribute__((always_inline)) {
            copy_tiles<U, ND, NT_IN>(a.seg[seg], (uint32_t)lb, lb == nb - 1, (uint32_t)nb, a.threads);
        });
        return;
    }
    const uint32_t G = gridDim.x;
    for (uint32_t at = blockIdx.x; at < a.first[a.nseg];) {
        int lo = 0, hi = a.nseg;
        while (hi - lo > 1) {
            const int mid = (lo + hi) / 2;
            if (a.first[mid] <= at)
                lo = mid;
            else
                hi = mid;
        }
        const uint32_t b = a.first[lo], left = a.first[lo + 1] - 1 - at, jump = left / G * G;
        copy_tiles<U, ND, NT_IN>(a.seg[lo], at - b, jump == left, G, a.threads);
        at += jump + G;
    }
}

}  // namespace

// ---- launchers --------------------------------------------------------------------

// hipLaunchKernel reports this launch's own status (hipGetLastError would
// also return errors left behind by unrelated earlier calls).
// Sets a.threads: a kernel that read its workgroup size from the hidden
// arguments would start every wave with a vector load of it and the wait (the
// headline ring, whose waves make one pass each, took 3% longer so than with
// the size among the arguments' scalar loads).
template <typename Args>
static hipError_t launch(const void *kernel, Args a, int wg, int threads, hipStream_t s, size_t lds = 0) {
    a.threads = (uint32_t)threads;
    void *args[] = {&a};
    return hipLaunchKernel(kernel, dim3((unsigned)wg), dim3((unsigned)threads), args, lds, s);
}

// The first a.nseg slots of `a` in an argument struct of CAP slots.
template <int CAP>
static ReduceArgsT<CAP> fit(const ReduceArgs &a) {
    ReduceArgsT<CAP> b{};
    for (int k = 0; k < a.nseg; ++k) b.seg[k] = a.seg[k];
    b.nseg = a.nseg;
    b.back = a.back;
    return b;
}
template <int CAP>
static MultiArgsT<CAP> fit(const MultiArgs &a) {
    MultiArgsT<CAP> b{};
    for (int k = 0; k < a.nseg; ++k) b.seg[k] = a.seg[k];
    b.nseg = a.nseg;
    b.back = a.back;
    return b;
}
template <int CAP, int C0, int ND>
static CopyArgsT<CAP, ND> fit_copy(const CopyArgsT<C0, ND> &a) {
    CopyArgsT<CAP, ND> b{};
    for (int k = 0; k < a.nseg; ++k) {
        b.seg[k] = a.seg[k];
        b.first[k] = a.first[k];
    }
    b.first[a.nseg] = a.first[a.nseg];
    b.nseg = a.nseg;
    return b;
}
template <int CAP>
static FoldArgsT<CAP> fit(const FoldArgs &a) {
    FoldArgsT<CAP> b{};
    for (int r = 0; r < a.R; ++r) {
        b.in[r] = a.in[r];
        b.out[r] = a.out[r];
    }
    b.c = a.c;
    b.total = a.total;
    b.R = a.R;
    b.write_all = a.write_all;
    b.out_at_chunk = a.out_at_chunk;
    return b;
}

// Ring steps of up to 8 ranks (272 bytes of arguments) or up to 64 (2 KiB).
constexpr int kSmallSegs = 8;

template <class T0, class T1, class TO, int VE, int U, int NT>
static hipError_t launch_rs(const ReduceArgs &a, int wg, int threads, hipStream_t s) {
    if (a.nseg <= kSmallSegs)
        return launch((const void *)reduce_step_kernel<T0, T1, TO, VE, U, NT, kSmallSegs>,
                      fit<kSmallSegs>(a), wg, threads, s);
    return launch((const void *)reduce_step_kernel<T0, T1, TO, VE, U, NT, kMaxReduceSegs>, a, wg,
                  threads, s);
}

hipError_t launch_reduce_step(hoccl_dtype_t dt, Phase ph, const ReduceArgs &a, int wg, int threads,
                              hipStream_t s, bool bf16_partials) {
    constexpr int UB = HOCCL_RS_UNROLL_BF16, U4 = HOCCL_RS_UNROLL_32;
    constexpr int VP = kVeBf16Partial, VB = kVeBf16Only, V4 = kVe32;
    if (dt == HOCCL_BF16 && bf16_partials) {
        // Every operand and result in bf16: each step rounds its sum, as a
        // ring that forwards bf16 partials does.  The same in-flight rule
        // as below, on 8-element vectors.
        uint64_t n = 0;
        for (int k = 0; k < a.nseg; ++k) n += a.seg[k].n;
        const bool deep = n > (uint64_t)wg * (uint64_t)threads * (uint64_t)(VB * UB);
        if (deep) {
            switch (ph) {
            case PH_FIRST: return launch_rs<TBF16, TBF16, TBF16, VB, 2 * UB, kNtFirst>(a, wg, threads, s);
            case PH_MIDDLE: return launch_rs<TBF16, TBF16, TBF16, VB, 2 * UB, kNtMiddle>(a, wg, threads, s);
            case PH_LAST: return launch_rs<TBF16, TBF16, TBF16, VB, 2 * UB, kNtLast>(a, wg, threads, s);
            case PH_ONLY: break;
            }
        }
        switch (ph) {
        case PH_FIRST: return launch_rs<TBF16, TBF16, TBF16, VB, UB, kNtFirst>(a, wg, threads, s);
        case PH_MIDDLE: return launch_rs<TBF16, TBF16, TBF16, VB, UB, kNtMiddle>(a, wg, threads, s);
        case PH_LAST: return launch_rs<TBF16, TBF16, TBF16, VB, UB, kNtLast>(a, wg, threads, s);
        case PH_ONLY: return launch_rs<TBF16, TBF16, TBF16, VB, UB, kNtOnly>(a, wg, threads, s);
        }
    } else if (dt == HOCCL_BF16) {
        // A launch that leaves each thread several passes (a small
        // workgroup budget) keeps twice the vectors in flight per thread:
        // there the bytes in flight per wave, not the number of waves, set
        // the rate (8 workgroups: 777 us per headline step with 2 vectors,
        // 497 us with 4).
        uint64_t n = 0;
        for (int k = 0; k < a.nseg; ++k) n += a.seg[k].n;
        const bool deep = n > (uint64_t)wg * (uint64_t)threads * (uint64_t)(VP * UB);
        if (deep) {
            switch (ph) {
            case PH_FIRST: return launch_rs<TBF16, TBF16, TF32, VP, 2 * UB, kNtFirst>(a, wg, threads, s);
            case PH_MIDDLE: return launch_rs<TF32, TBF16, TF32, VP, 2 * UB, kNtMiddle>(a, wg, threads, s);
            case PH_LAST: return launch_rs<TF32, TBF16, TBF16, VP, 2 * UB, kNtLast>(a, wg, threads, s);
            case PH_ONLY: return launch_rs<TBF16, TBF16, TBF16, VB, UB, kNtOnly>(a, wg, threads, s);
            }
        }
        switch (ph) {
        case PH_FIRST: return launch_rs<TBF16, TBF16, TF32, VP, UB, kNtFirst>(a, wg, threads, s);
        case PH_MIDDLE: return launch_rs<TF32, TBF16, TF32, VP, UB, kNtMiddle>(a, wg, threads, s);
        case PH_LAST: return launch_rs<TF32, TBF16, TBF16, VP, UB, kNtLast>(a, wg, threads, s);
        case PH_ONLY: return launch_rs<TBF16, TBF16, TBF16, VB, UB, kNtOnly>(a, wg, threads, s);
        }
    } else if (dt == HOCCL_FP32) {
        switch (ph) {
        case PH_FIRST: return launch_rs<TF32, TF32, TF32, V4, U4, kNtFirst>(a, wg, threads, s);
        case PH_MIDDLE: return launch_rs<TF32, TF32, TF32, V4, U4, kNtMiddle>(a, wg, threads, s);
        case PH_LAST: return launch_rs<TF32, TF32, TF32, V4, U4, kNtLast>(a, wg, threads, s);
        case PH_ONLY: return launch_rs<TF32, TF32, TF32, V4, U4, kNtOnly>(a, wg, threads, s);
        }
    } else if (dt == HOCCL_INT32) {
        switch (ph) {
        case PH_FIRST: return launch_rs<TI32, TI32, TI32, V4, U4, kNtFirst>(a, wg, threads, s);
        case PH_MIDDLE: return launch_rs<TI32, TI32, TI32, V4, U4, kNtMiddle>(a, wg, threads, s);
        case PH_LAST: return launch_rs<TI32, TI32, TI32, V4, U4, kNtLast>(a, wg, threads, s);
        case PH_ONLY: return launch_rs<TI32, TI32, TI32, V4, U4, kNtOnly>(a, wg, threads, s);
        }
    }
    return hipErrorInvalidValue;
}

// Fused ring hops.  Every lane moves 4 elements of every operand (8 bytes of
// bf16, 16 of fp32 / int32), and keeps U such vectors of each operand in
// flight, U chosen per bound on the contributions so that the registers
// they need stay within the 128 VGPRs a 1024-thread launch bound allows
// without spilling: bf16 2 whatever the bound; 32-bit types 4, 2 and 1 for
// at most 2, 4 and 8 contributions.
template <class T0, class T1, class TO, int NT, int MAXL, bool RH>
static hipError_t launch_mh_l(const MultiArgs &a, int wg, int threads, hipStream_t s) {
    constexpr int U = sizeof(typename T1::S) == 2 ? 2 : (MAXL <= 2 ? 4 : (MAXL <= 4 ? 2 : 1));
    if (a.nseg <= kSmallSegs)
        return launch((const void *)multihop_kernel<T0, T1, TO, 4, U, NT, MAXL, kSmallSegs, RH>,
                      fit<kSmallSegs>(a), wg, threads, s);
    return launch((const void *)multihop_kernel<T0, T1, TO, 4, U, NT, MAXL, kMaxMultiSegs, RH>, a, wg,
                  threads, s);
}

template <class T0, class T1, class TO, int NT, bool RH = false>
static hipError_t launch_mh(const MultiArgs &a, int wg, int threads, hipStream_t s) {
    int nl = 0;
    for (int k = 0; k < a.nseg; ++k) nl = a.seg[k].nloc > nl ? a.seg[k].nloc : nl;
    if (nl <= 2) return launch_mh_l<T0, T1, TO, NT, 2, RH>(a, wg, threads, s);
    if (nl <= 4) return launch_mh_l<T0, T1, TO, NT, 4, RH>(a, wg, threads, s);
    return launch_mh_l<T0, T1, TO, NT, kMaxHops, RH>(a, wg, threads, s);
}

hipError_t launch_multihop(hoccl_dtype_t dt, Phase ph, const MultiArgs &a, int wg, int threads,
                           hipStream_t s, bool bf16_partials) {
    if (dt == HOCCL_BF16 && bf16_partials) {
        switch (ph) {
        case PH_FIRST: return launch_mh<TBF16, TBF16, TBF16, kNtFirst, true>(a, wg, threads, s);
        case PH_MIDDLE: return launch_mh<TBF16, TBF16, TBF16, kNtMiddle, true>(a, wg, threads, s);
        case PH_LAST: return launch_mh<TBF16, TBF16, TBF16, kNtLast, true>(a, wg, threads, s);
        case PH_ONLY: return launch_mh<TBF16, TBF16, TBF16, kNtOnly, true>(a, wg, threads, s);
        }
    } else if (dt == HOCCL_BF16) {
        switch (ph) {
        case PH_FIRST: return launch_mh<TBF16, TBF16, TF32, kNtFirst>(a, wg, threads, s);
        case PH_MIDDLE: return launch_mh<TF32, TBF16, TF32, kNtMiddle>(a, wg, threads, s);
        case PH_LAST: return launch_mh<TF32, TBF16, TBF16, kNtLast>(a, wg, threads, s);
        case PH_ONLY: return launch_mh<TBF16, TBF16, TBF16, kNtOnly>(a, wg, threads, s);
        }
    } else if (dt == HOCCL_FP32) {
        switch (ph) {
        case PH_FIRST: return launch_mh<TF32, TF32, TF32, kNtFirst>(a, wg, threads, s);
        case PH_MIDDLE: return launch_mh<TF32, TF32, TF32, kNtMiddle>(a, wg, threads, s);
        case PH_LAST: return launch_mh<TF32, TF32, TF32, kNtLast>(a, wg, threads, s);
        case PH_ONLY: return launch_mh<TF32, TF32, TF32, kNtOnly>(a, wg, threads, s);
        }
    } else if (dt == HOCCL_INT32) {
        switch (ph) {
        case PH_FIRST: return launch_mh<TI32, TI32, TI32, kNtFirst>(a, wg, threads, s);
        case PH_MIDDLE: return launch_mh<TI32, TI32, TI32, kNtMiddle>(a, wg, threads, s);
        case PH_LAST: return launch_mh<TI32, TI32, TI32, kNtLast>(a, wg, threads, s);
        case PH_ONLY: return launch_mh<TI32, TI32, TI32, kNtOnly>(a, wg, threads, s);
        }
    }
    return hipErrorInvalidValue;
}

// Grid sizing for fused launches assumes 2 vectors of 4 elements per pass.
size_t multihop_elems_per_thread(hoccl_dtype_t) { return 8; }

// Elements one thread covers in one pass of each kernel's main loop; the
// executor sizes automatic launches to about one pass per thread.
size_t reduce_step_elems_per_thread(hoccl_dtype_t dt, Phase ph, bool bf16_partials) {
    if (dt == HOCCL_BF16)
        return (size_t)(ph == PH_ONLY || bf16_partials ? kVeBf16Only : kVeBf16Partial) *
               HOCCL_RS_UNROLL_BF16;
    return (size_t)kVe32 * HOCCL_RS_UNROLL_32;
}
size_t fold_elems_per_thread(hoccl_dtype_t dt) { return 16 / dtype_size(dt); }

// R up to 8 has a kernel of its own, whose arguments hold R ranks and whose
// pointers all stay in scalar registers (R = 6, n = 1,398,103 bf16: 13% less
// than by the kernel for any R; R = 5, n = 5,242,880 bf16: 11%).  More ranks would need more than the 100 or so scalar registers a
// wave has.
template <class T, int VE, int NR, bool RH>
static hipError_t launch_fold_r(const FoldArgs &a, int wg, int threads, hipStream_t s, size_t lds) {
    // Beyond 600 MiB a rank, folds of 4 and 8 ranks take their blocks in turn,
    // and of two ranks beyond 768 MiB: runs of blocks, which are the faster ones
    // below, lose to it there (bf16, us, runs and in turn over the same buffers):
    //   reduce-scatter  R = 8  384 MiB 652 and 688, 1 GiB 2010 and 1840, 2 GiB 4370
    //     and 3720;  R = 4  384 MiB 397 and 408, 1280 MiB 1555 and 1297, 2 GiB
    //     2796 and 2178;  R = 2  640 MiB 402 and 425, 1 GiB 675 and 625
    //   all-reduce  R = 8  384 MiB 1208 and 1270, 1 GiB 3530 and 3340;  R = 4  448
    //     MiB 723 and 809, 1536 MiB 2990 and 2565;  R = 2  640 MiB 532 and 568, 1
    //     GiB 855 and 793
    // Between 512 and 600 MiB it goes by the size; three, six and 16 ranks take
    // as long either way.
    if constexpr (NR == 2 || NR == 4 || NR == 8) {
        const uint64_t bytes = a.total * sizeof(typename T::S);
        if (bytes > ((uint64_t)(NR == 2 ? 768 : 600) << 20))
            return launch((const void *)fold_kernel<T, VE, NR, NR, RH, true>, fit<NR>(a), wg, threads, s, lds);
    }
    return launch((const void *)fold_kernel<T, VE, NR, NR, RH>, fit<NR>(a), wg, threads, s, lds);
}

// An all-reduce writes as much as it reads, and HBM takes that better when
// fewer workgroups are in flight and the windows they write stay narrow:
// asking for LDS that the kernel does not use bounds them to 1024 threads per
// CU (40 KiB of 160 for 256).  It is asked for where it gained and nothing
// else: all-reduces of three to five ranks of 16 MiB a rank or more (us,
// bounded and not):
//   R = 3, 48 MiB:  bf16 48.7 and 53.3, fp32 52.3 and 53.6
//   R = 4, n = 16,777,216:  bf16 43.8 and 45.5, fp32 85.0 and 88.1
//   R = 5, 48 MiB:  bf16 82.7 and 84.3, fp32 87.9 and 89.6
//   R = 6, 48 MiB:  bf16 108 and 104;  R = 7, fp32 127 and 123;  R = 8 equal
//   R = 3, 8 MiB:   bf16 10.2 and 9.9;  R = 4, 12 MB: 18.6 and 18.3
//   reduce-scatter, R = 4, n = 6,000,000:  bf16 43.1 and 38.2
// Beside a bf16 GEMM of 8192^3 it costs neither side anything (R = 4, 48 MiB:
// 668 us a call and 665, the GEMM 9.1% slower and 8.6%; R = 3: 650 and 656).
// On a stream with 32 of the CUs it does (R = 3, bf16: 228 us and 183; R = 4:
// 278 and 264), so that the caller drops it there and under a workgroup
// budget, where too few bytes are in flight already.  Above 256 threads the
// same bound takes more than the 64 KiB a launch may ask for.
size_t fold_lds(hoccl_dtype_t dt, const FoldArgs &a, int threads) {
    const bool wide = a.R >= 3 && a.R <= 5 && a.total * dtype_size(dt) >= ((uint64_t)16 << 20);
    return a.write_all && wide && threads <= 256 ? (size_t)threads * 160 : 0;
}

template <class T, int VE, bool RH = false>
static hipError_t launch_fold_t(const FoldArgs &a, int wg, int threads, hipStream_t s, size_t lds) {
    switch (a.R) {
    case 2: return launch_fold_r<T, VE, 2, RH>(a, wg, threads, s, lds);
    case 3: return launch_fold_r<T, VE, 3, RH>(a, wg, threads, s, lds);
    case 4: return launch_fold_r<T, VE, 4, RH>(a, wg, threads, s, lds);
    case 5: return launch_fold_r<T, VE, 5, RH>(a, wg, threads, s, lds);
    case 6: return launch_fold_r<T, VE, 6, RH>(a, wg, threads, s, lds);
    case 7: return launch_fold_r<T, VE, 7, RH>(a, wg, threads, s, lds);
    case 8: return launch_fold_r<T, VE, 8, RH>(a, wg, threads, s, lds);
    }
    // A bf16 all-reduce of 16, 24, 32, ... ranks takes its blocks in turn, from
    // 192 MiB of inputs on: each chunk then stays on one XCD, and R streams to
    // write beside R to read lose less to each other.  Over the same buffers, in
    // turn against runs of blocks: R = 16  32 MiB a rank 0.90, 48 MiB 0.92 (313 us
    // and 340), 64 MiB 0.85, other sizes 0.96 to 1.04;  R = 24  16, 24 and 48 MiB
    // 0.89 to 0.92, others to 1.03;  R = 32  16 MiB 0.88, others to 1.00.  Less
    // gains nothing (R = 16, 8 MiB 1.08, 4 MiB 0.97), other rank counts lose (R =
    // 12, 14, 20: 1.00 to 1.12, one point at 0.92), and so does fp32 at R = 16
    // (0.86 to 1.16, 1.02 in the mean).
    if constexpr (sizeof(typename T::S) == 2) {
        if (a.write_all && a.R % kXcds == 0 && (uint64_t)a.R * a.total * 2 >= ((uint64_t)192 << 20))
            return launch((const void *)fold_kernel<T, VE, 0, kMaxRanks, RH, true>, a, wg, threads, s, lds);
    }
    return launch((const void *)fold_kernel<T, VE, 0, kMaxRanks, RH>, a, wg, threads, s, lds);
}

hipError_t launch_fold(hoccl_dtype_t dt, const FoldArgs &a, int wg, int threads, hipStream_t s,
                       bool bf16_partials, size_t lds) {
    if (dt == HOCCL_BF16 && bf16_partials) return launch_fold_t<TBF16, 8, true>(a, wg, threads, s, lds);
    if (dt == HOCCL_BF16) return launch_fold_t<TBF16, 8>(a, wg, threads, s, lds);
    if (dt == HOCCL_FP32) return launch_fold_t<TF32, 4>(a, wg, threads, s, lds);
    if (dt == HOCCL_INT32) return launch_fold_t<TI32, 4>(a, wg, threads, s, lds);
    return hipErrorInvalidValue;
}

// Lays a launch out in tiles of `unroll` vectors per thread, in a row or
// segment by segment, and returns the workgroups that take one tile each: all
// tiles of the row, or as many for every segment as the longest one has.
template <int CAP, int ND>
static uint32_t lay_tiles(CopyArgsT<CAP, ND> &a, int threads, int unroll, bool row) {
    const uint64_t tile = (uint64_t)threads * 16 * (uint64_t)unroll;
    uint32_t at = 0, longest = 0;
    for (int k = 0; k < a.nseg; ++k) {
        const uint32_t tiles = (uint32_t)((a.seg[k].bytes + tile - 1) / tile);
        a.first[k] = at;
        at += tiles;
        longest = tiles > longest ? tiles : longest;
    }
    a.first[a.nseg] = at;
    a.unroll = (uint32_t)unroll;
    a.row = row;
    return row ? at : longest * (uint32_t)a.nseg;
}

template <int CAP, int ND>
static uint64_t bytes_written(const CopyArgsT<CAP, ND> &a) {
    uint64_t n = 0;
    for (int k = 0; k < a.nseg; ++k) n += a.seg[k].bytes * (uint64_t)a.seg[k].nd;
    return n;
}

// Segments of one destination.  Times in us over buffers the caches hold and
// over rotating ones, as "row, one vector / row, four / segment by segment".
// * Equal segments, up to 16 MiB in all, or of up to 1 MiB each and 64 MiB in
//   all: segment by segment, four vectors (all-to-all at R = 8, 256 KiB a
//   pair 6.6, 9.0 / 5.5, 8.7 / 4.7, 7.6; 1 MiB 22.3, 26.5 / 18.9, 26.6 / 17.4,
//   26.3; a 2 MiB pair at R = 2 3.7, 4.7 / 3.3, 4.3 / 3.2, 4.1).  Few long
//   segments walked side by side spread HBM's windows (64 MiB in four 18.0,
//   23.4 / 17.6, 24.7 / 17.3, 26.4), unequal ones leave workgroups idle.
// * From 16 to 48 MiB: the row, four vectors (an all-to-all(v) of 36 MB
//   12.0, 12.2 / 10.6, 11.4 / -).  Beyond, one vector, as deeper tiles read
//   and write a wider window at once (256 MiB in 64 segments 75.2, 86.0 /
//   64.3, 98.1 / -; the EP all-to-all(v) of 608 MB 10% less with one), and
//   below 16 MiB where segments are unequal (64 of 23 KB on average, skewed:
//   3.0, 3.5 / 3.3, 4.3 / 3.1, 3.5).
// * A workgroup budget of fewer than those: deep tiles, as the bytes in flight
//   per wave then set the rate (8 workgroups: 2.5 ms for 512 MiB with 4
//   vectors, 4.2 with 2), segment by segment for equal segments (all-to-all at
//   R = 8 on 64 workgroups, 512 KiB a pair: - / 33.5, 43.1 / 14.9, 29.0; on 8,
//   64 KiB: - / 25.7, 36.2 / 10.9, 16.1), else the row (skewed, 0.6 MB a pair
//   on 64: - / 28.9, 29.8 / 96, 96).
uint32_t copy_layout(CopyArgs &a, int threads, int budget) {
    constexpr uint64_t MiB = 1u << 20;
    const uint64_t bytes = bytes_written(a);
    uint64_t longest = 0;
    for (int k = 0; k < a.nseg; ++k) longest = a.seg[k].bytes > longest ? a.seg[k].bytes : longest;
    const bool even = longest * (uint64_t)a.nseg * 4 <= bytes * 5;
    uint32_t wg;
    if (even && (bytes <= 16 * MiB || (longest <= MiB && bytes <= 64 * MiB)))
        wg = lay_tiles(a, threads, kDeepCopy, false);
    else
        wg = lay_tiles(a, threads, bytes > 16 * MiB && bytes <= 48 * MiB ? kDeepCopy : 1, true);
    if (budget > 0 && (uint32_t)budget < wg) lay_tiles(a, threads, kDeepCopy, !even);
    return budget > 0 ? (uint32_t)budget : wg;
}

// Segments of several destinations, whose tiles each write several times
// themselves; times as above, row / segment by segment.
// * Up to 16 MiB written: segment by segment, one vector (gathers of 64 KiB
//   shards at R = 8 3.3, 2.9 / 3.0, 2.8, of 256 KiB at R = 3 3.3, 3.1 / 2.6,
//   2.6).
// * Beyond, the row: one vector under the bound of copy_lds from kWideFan
//   destinations on, where writes dominate (eight 16 MiB shards 187 us; 211
//   without the bound, 201 with four vectors), four vectors and no bound for
//   fewer, which leave too few bytes in flight so (two 16 MiB shards 13.7 and
//   21.0 with one vector, four 1 MiB shards 4.7 and 5.2).
// * A budget of fewer workgroups: the row with four vectors (eight 16 MiB
//   shards on 8 workgroups 1290, with one vector 1700; on 64 202 and 231).
uint32_t copy_layout(FanArgs &a, int threads, int budget) {
    int nd = 0;
    for (int k = 0; k < a.nseg; ++k) nd = a.seg[k].nd > nd ? a.seg[k].nd : nd;
    const bool row = bytes_written(a) > ((uint64_t)16 << 20);
    const uint32_t wg = lay_tiles(a, threads, row && nd < kWideFan ? kDeepCopy : 1, row);
    if (budget > 0 && (uint32_t)budget < wg) lay_tiles(a, threads, kDeepCopy, true);
    return budget > 0 ? (uint32_t)budget : wg;
}

// Copy launches of up to 8, 32 or 128 segments (250 bytes to 4 KiB of arguments).
template <int U, bool NT, bool ROW>
static hipError_t launch_copy_as(const CopyArgs &a, int wg, int threads, hipStream_t s) {
    if (a.nseg <= 8) return launch((const void *)copy_kernel<8, 1, U, NT, ROW>, fit_copy<8>(a), wg, threads, s);
    if (a.nseg <= 32) return launch((const void *)copy_kernel<32, 1, U, NT, ROW>, fit_copy<32>(a), wg, threads, s);
    return launch((const void *)copy_kernel<kMaxCopySegs, 1, U, NT, ROW>, a, wg, threads, s);
}
hipError_t launch_copy(const CopyArgs &a, int wg, int threads, hipStream_t s, size_t) {
    if (!a.row) return launch_copy_as<kDeepCopy, false, false>(a, wg, threads, s);
    if (a.unroll != 1) return launch_copy_as<kDeepCopy, false, true>(a, wg, threads, s);
    // Reading more than the 256 MB last-level cache holds, little of it can be
    // there from an earlier write, and non-temporal loads are the faster ones:
    // 6% for the EP all-to-all(v) (608 MB), 3% for a 2 GiB copy (at 4 vectors
    // per thread).  Where the data is in the cache they are slower: a pipeline
    // schedule of 16 MiB messages, each read soon after it was written, took
    // 10% longer, a 64 MiB copy 16%.
    return bytes_written(a) > ((uint64_t)256 << 20) ? launch_copy_as<1, true, true>(a, wg, threads, s)
                                                    : launch_copy_as<1, false, true>(a, wg, threads, s);
}

template <int U, bool ROW>
static hipError_t launch_fan_as(const FanArgs &a, int wg, int threads, hipStream_t s, size_t lds) {
    if (a.nseg <= 8)
        return launch((const void *)copy_kernel<8, kMaxFan, U, false, ROW>, fit_copy<8>(a), wg, threads, s, lds);
    return launch((const void *)copy_kernel<kMaxFanSegs, kMaxFan, U, false, ROW>, a, wg, threads, s, lds);
}
hipError_t launch_fan(const FanArgs &a, int wg, int threads, hipStream_t s, size_t lds) {
    if (!a.row) return launch_fan_as<1, false>(a, wg, threads, s, lds);
    if (a.unroll != 1) return launch_fan_as<kDeepCopy, true>(a, wg, threads, s, lds);
    return launch_fan_as<1, true>(a, wg, threads, s, lds);
}

// The kernel uses no LDS; asking for it bounds how many workgroups a CU holds
// (64 KiB of 160 KiB: two of 256 threads).  Eight 16 MiB shards take 187 us
// so and 211 without, eight of 48 MiB 565 and 698.  Beside a bf16 GEMM of
// 8192^3 the 16 MiB gather takes 460 us and 821, the GEMM being 66% and 26%
// slower meanwhile, which is 0.18 and 0.17 ms of its time per gather.  On a
// stream with 32 of the CUs the bound costs (638 us and 366): the caller drops
// it there and under a workgroup budget.  Above 256 threads it would take more
// than the 64 KiB a launch may ask for.
size_t copy_lds(const FanArgs &a, int threads) {
    return a.row && a.unroll == 1 && threads <= 256 ? (size_t)threads << 8 : 0;
}

}  // namespace hoccl
