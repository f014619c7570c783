// The refit and row-absmax bodies for heads of any row-width mix ("slot"
// bodies, completed in stepq_refit_body.h): any d_k, d_v = 64 or 128, FP16
// pivot rows, the row splits of a row-unit calibration.  Frozen steps of these
// heads run the generic or the row-mix body (stepq_kernels.hip).
//
// Every thread holds 4 columns (word cg of a row group) of its slice's rows,
// in NP pairs of row slots.  The classes take whole pairs: the 8-bit words of
// the slice fill slots r = 0 .. M8 - 1, two to a pair; each 4-bit word takes
// one pair, each 2-bit word two, from an even pair on.  So which width a pair
// holds is the same for the whole workgroup: the width tests are scalar
// branches, and every value keeps a register fixed at compile time.  Slots
// without a row (the last word-step of a class, an empty field, pairs past the
// head's last) have zero constants; their codes are not stored (words past the
// class's last group are out of the buffer's range) or stay 0 (empty fields).
//
// NP is the pairs of the launch's largest head (slot_pairs in
// stepq_layout.h), rounded up to the next size that is compiled; live_pairs
// says which of them a wave needs.
#pragma once

#include "stepq_device.h"

namespace stepq {
namespace {

template <int DV, int NP>
struct SlotShared {
    static constexpr int CG = DV / 4;
    static constexpr int NSL = 256 / CG;
    static constexpr int NR = 4 * ((NP + 1) / 2);   // row slots per slice, whole float4s
    float4 red[2][NSL][CG];
    alignas(16) float av[NSL][NR];               // beta k_i q_b / r_i
    alignas(16) float al[NSL][NR];               // d_i 2^(b-8)
    alignas(16) float2 kq[NSL][NR];              // k and q weights
    float sk[kMaxDk], sq[kMaxDk], sd[kMaxDk];    // k, q, gate in logical row order
    float bcol[DV];                              // v_j, then delta_j / c_j
    float cpiv[DV];                              // c_j
    float4 pvc[kMaxPivots];                      // pivot rows: (k_i d_i, q_i d_i, d_i, beta k_i)
    float kap[4];
};

// A head's classes in pairs: pairs below p4 hold 8-bit rows, those below e4
// 4-bit words, those from p2 (even) to pt 2-bit words.  All uniform.
struct SlotGeom {
    int g8, g4, g2, p4, e4, p2, pt;
    __device__ __forceinline__ SlotGeom(const HeadInfo &hi, int nsl_shift)
    {
        const int r = (1 << nsl_shift) - 1;
        g8 = __builtin_amdgcn_readfirstlane(static_cast<int>(hi.g8));
        g4 = __builtin_amdgcn_readfirstlane(static_cast<int>(hi.g4));
        g2 = __builtin_amdgcn_readfirstlane(static_cast<int>(hi.g2));
        p4 = (((g8 + r) >> nsl_shift) + 1) >> 1;
        e4 = p4 + ((g4 + r) >> nsl_shift);
        p2 = (e4 + 1) & ~1;
        pt = p2 + 2 * ((g2 + r) >> nsl_shift);
    }
};

// The pairs in which this wave's slices have a row at all, one bit each: a
// class's last word-step fills only some of the slices, and NP is that of the
// launch's largest head.  Uniform per wave; the other pairs' slots have zero
// constants, so leaving them out changes no sum and no maximum.
template <int NSL>
__device__ __forceinline__ uint32_t live_pairs(const SlotGeom &g, int slice)
{
    constexpr int SH = NSL == 8 ? 3 : 4, R = NSL - 1, S = NSL / 4;     // S slices per wave
    const int s0 = __builtin_amdgcn_readfirstlane(slice);
    const int e4 = g.g8 + g.g4, e2 = e4 + g.g2;
    int n4 = 0, n2 = 0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        // word-steps of slice s0 + s up to the end of each class
        const int r = R - s0 - s;
        const int a8 = (g.g8 + r) >> SH, a4 = (e4 + r) >> SH, a2 = (e2 + r) >> SH;
        n4 = max(n4, a4 - a8);
        n2 = max(n2, a2 - a4);
    }
    const int n8 = ((g.g8 + R - s0) >> SH) + 1;
    return ((1u << (n8 >> 1)) - 1u) | (((1u << n4) - 1u) << g.p4) | (((1u << (2 * n2)) - 1u) << g.p2);
}

// The code words of a slot-body tile.  The slices take the row groups of the
// whole codes region in turn (group g belongs to slice g mod NSL), so where a
// class begins inside a round its first word-step m4 (m2) differs by one
// between slices.  Byte offsets are formed in the vector offset alone (the
// part the range check surely covers): words past the class's last group read
// 0, and their stores are dropped.
template <int DV>
struct SlotWords {
    __amdgpu_buffer_rsrc_t r8, r4, r2;
    int v8, v4, v2;      // byte offset of the thread's first word of each class
    __device__ __forceinline__ SlotWords(void *codes, const SlotGeom &g, int slice)
    {
        constexpr int SH = DV == 128 ? 3 : 4, R = (1 << SH) - 1;
        const int b4 = DV * g.g8, b2 = b4 + DV * g.g4;
        r8 = __builtin_amdgcn_make_buffer_rsrc(codes, 0, b4, 0x00020000);
        r4 = __builtin_amdgcn_make_buffer_rsrc(codes, 0, b2, 0x00020000);
        r2 = __builtin_amdgcn_make_buffer_rsrc(codes, 0, b2 + DV * g.g2, 0x00020000);
        v8 = 4 * static_cast<int>(threadIdx.x);
        v4 = v8 + 1024 * ((g.g8 - slice + R) >> SH);
        v2 = v8 + 1024 * ((g.g8 + g.g4 - slice + R) >> SH);
    }
    // v + 1024 m for a uniform run-time m >= 0; the scalar part is kept apart,
    // so that no negative constant is folded into the instruction's offset
    static __device__ __forceinline__ int at(int v, int m)
    {
        int s = 1024 * m;
        asm("" : "+s"(s));
        return v + s;
    }
    __device__ __forceinline__ uint32_t ld8(int m) const
    {
        return __builtin_amdgcn_raw_buffer_load_b32(r8, v8 + 1024 * m, 0, CodeWords::kLoad);
    }
    __device__ __forceinline__ void st8(int m, uint32_t v) const
    {
        __builtin_amdgcn_raw_buffer_store_b32(v, r8, v8 + 1024 * m, 0, CodeWords::kStore);
    }
    __device__ __forceinline__ uint32_t ld4(int m) const
    {
        return __builtin_amdgcn_raw_buffer_load_b32(r4, at(v4, m), 0, CodeWords::kLoad);
    }
    __device__ __forceinline__ void st4(int m, uint32_t v) const
    {
        __builtin_amdgcn_raw_buffer_store_b32(v, r4, at(v4, m), 0, CodeWords::kStore);
    }
    __device__ __forceinline__ uint32_t ld2(int m) const
    {
        return __builtin_amdgcn_raw_buffer_load_b32(r2, at(v2, m), 0, CodeWords::kLoad);
    }
    __device__ __forceinline__ void st2(int m, uint32_t v) const
    {
        __builtin_amdgcn_raw_buffer_store_b32(v, r2, at(v2, m), 0, CodeWords::kStore);
    }
};

// All code words of the thread, issued together: wa[p], wb[p] the 8-bit words
// of pair p's two slots, or wa[p] a 4-bit word, or (p even) the 2-bit word of
// pairs p and p + 1.
template <int DV, int NP, bool HAS2>
__device__ __forceinline__ void slot_load(const SlotWords<DV> &cw, const SlotGeom &g, uint32_t (&wa)[NP],
                                          uint32_t (&wb)[NP])
{
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        wa[p] = 0u;
        wb[p] = 0u;
        if (p < g.p4) {
            wa[p] = cw.ld8(2 * p);
            wb[p] = cw.ld8(2 * p + 1);
        } else if (p < g.e4) {
            wa[p] = cw.ld4(p - g.p4);
        } else if (HAS2 && (p & 1) == 0 && p >= g.p2 && p < g.pt) {
            wa[p] = cw.ld2((p - g.p2) >> 1);
        }
    }
}

// The two rows of pair p as bytes, each field at the top of its byte.
template <int NP, bool HAS2>
__device__ __forceinline__ void slot_views(const SlotGeom &g, const uint32_t (&wa)[NP], const uint32_t (&wb)[NP],
                                           int p, uint32_t &lo, uint32_t &hi)
{
    if (p < g.p4) {
        lo = wa[p];
        hi = wb[p];
    } else if (!HAS2 || p < g.p2) {
        lo = slot_top<4>(wa[p], 0);
        hi = slot_top<4>(wa[p], 1);
    } else {
        lo = slot_top<2>(wa[p & ~1], (p & 1) * 2);
        hi = slot_top<2>(wa[p & ~1], (p & 1) * 2 + 1);
    }
}

// The row a thread owns in the row constants: physical row p = tid < d_k, with
// its place in the slot tables (slice -1: a pivot row, or no row).
struct SlotRow {
    int slice, r;
    int bw;
};

template <int NSL>
__device__ __forceinline__ SlotRow slot_of_row(const HeadInfo &hi, const SlotGeom &g, int p, int dk)
{
    constexpr int SH = NSL == 8 ? 3 : 4;
    int i = p - static_cast<int>(hi.n16);
    if (i < 0 || p >= dk) return {-1, 0, 8};
    int w, r, bw;
    if (i < hi.n8) {
        bw = 8;
        w = i;
        r = w >> SH;
    } else if ((i -= hi.n8) < hi.n4) {
        bw = 4;
        w = i >> 1;
        r = 2 * (g.p4 + (w >> SH)) + (i & 1);
    } else {
        i -= hi.n4;
        bw = 2;
        w = i >> 2;
        r = 2 * g.p2 + 4 * (w >> SH) + (i & 3);
    }
    // group index of the word in the whole region, modulo the slices
    const int first = bw == 8 ? 0 : (bw == 4 ? g.g8 : g.g8 + g.g4);
    return {(first + w) & (NSL - 1), r, bw};
}

// Row constants by slot (slots without a row: 0).  Two barriers; returns q.k.
template <bool DIAG, int DV, int NP, class Ops>
__device__ __forceinline__ float slot_constants(const HeadInfo &hi, int dk, float alpha, float beta,
                                                const Ops &op, SlotShared<DV, NP> &sh, const LevelTable &lv,
                                                const SlotRow &row)
{
    using SH = SlotShared<DV, NP>;
    constexpr int NE = SH::NSL * SH::NR;
    const int tid = threadIdx.x;
    if (tid < dk) {
        sh.sk[tid] = op.k();
        sh.sq[tid] = op.q();
        if constexpr (DIAG) sh.sd[tid] = op.d();
    }
    if (own_column<DV>() >= 0) {
        sh.bcol[tid - 128] = op.v();       // v_j and c_j wait in LDS for the column phase
        sh.cpiv[tid - 128] = op.c;
    }
    // slots without a row keep zero constants
    if (tid < NE) {
        (&sh.av[0][0])[tid] = 0.f;
        (&sh.al[0][0])[tid] = 0.f;
        (&sh.kq[0][0])[tid] = make_float2(0.f, 0.f);
    }
    __syncthreads();
    float kq = 0.f;
    if (tid < 128) {
        if (tid < dk) {
            const float ki = sh.sk[op.perm], qi = sh.sq[op.perm];
            const float di = DIAG ? sh.sd[op.perm] : 1.0f;
            kq = qi * ki;
            if (row.slice >= 0) {
                const float rs = op.r * by_width(lv.fq, row.bw) * di;
                sh.kq[row.slice][row.r] = make_float2(ki * rs, qi * rs);
                sh.av[row.slice][row.r] = beta * ki * by_width(lv.iq, row.bw) * __builtin_amdgcn_rcpf(op.r);
                sh.al[row.slice][row.r] = (DIAG ? di : alpha) *
                                          (row.bw == 8 ? 1.0f : (row.bw == 4 ? 1.0f / 16.0f : 1.0f / 64.0f));
            } else {
                // a pivot row (physical rows 0 .. n16 - 1); the scalar gate is applied with the columns
                sh.pvc[tid] = make_float4(ki * di, qi * di, DIAG ? di : alpha, beta * ki);
            }
        }
        kq = wave_sum(kq);
        if ((tid & 63) == 0) sh.kap[tid >> 6] = kq;
    }
    __syncthreads();
    return uniform_f(sh.kap[0] + sh.kap[1]);
}

}  // namespace
}  // namespace stepq
