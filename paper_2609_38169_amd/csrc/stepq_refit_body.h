// Decode step with a scale refit fused in: the online Key-Row-Aware Dual-Axis refit
// (paper: Section 4.3 row and column factors, the fixed-code column update
// of Appendix C.1, Table C2 steps 4-6).  One 256-thread workgroup per
// (request, value head) tile, as in the frozen-scale kernel, and the same
// first half: unpack, S^T k and S^T q, residual, readout.
//
// Working unit.  Per element the frozen-scale body forms the unrounded new
// code on the old scales,
//     y_ij = X_ij q_b / (r_i c_j).
// Every quantity of the refit is a row or column rescaling of y, so the tile
// is still never formed in real units:
//     m_i   = (r_i / (q_b d_v)) sum_j c_j |y_ij|       r'_i = (m_i / w_i)^(1/2)
//     yh_ij = y_ij r_i / r'_i                         (= X_ij q_b / (r'_i c_j))
//     c0_j  = c_j max_i |yh_ij| / q_b                 (absmax start)
//     z_ij  = round(yh_ij c_j / c0_j)                 (fixed codes; |.| <= q_b)
//     c'_j  = c_j sum_i W_i z_ij yh_ij / sum_i W_i z_ij^2,   W_i = (w_i r'_i / q_b)^2
//     q'_ij = clip(round(yh_ij c_j / c'_j), -q_b, q_b)
// Four passes over the thread's values with three LDS reductions between
// them: row sums (over the lanes that share a row), column maxima (kept per
// width in the thread, so that the scaling by 1/q_b happens once per column
// and thread), and the column sums of the least-squares numerator and
// denominator.  The new r' and c' overwrite the tile's scales; a zero
// denominator keeps c_j.
//
// The slot bodies also run the single-axis baseline the paper compares
// against (Section 5.1: symmetric row-wise absmax INT-b): every step
//     r'_i = max_j |X_ij| = (r_i / q_b) max_j c_j |y_ij|,   c'_j = 1,
//     q'_ij = clip(round(y_ij c_j r_i / r'_i), -q_b, q_b),
// i.e. pass 1 with a row maximum instead of a row sum, then pass 4; the
// uniform layouts have a lean body of their own for it (stepq_rowmax.hip).
#pragma once

#include "stepq_slots.h"

#include <type_traits>

namespace stepq {
namespace {

constexpr float kScaleFloor = 0x1p-60f;
constexpr float kRoundMagic = 0x1.8p+23f;     // 1.5 2^23: x + this rounds x to an integer (|x| < 2^22)

enum class Refit : int {
    DualAxis = 0,    // Key-Row-Aware Dual-Axis fit (Section 4.3, Appendix C.1)
    RowAbsmax = 1,   // row-wise absmax, column factors 1 (the INT-b baseline)
};

template <int DV>
struct RefitShared {
    DecodeShared<DV> d;
    union {
        float rowp[kSlotTable][DV / 8];            // partials of sum_j c_j |y_ij| by row slot, per column-lane pair
        float4 cmax[256 / (DV / 4)][DV / 4];       // per slice column maxima of |yh| / q_b
    } u;
    float hrow[kSlotTable];                        // r_i / r'_i by row slot (0 for empty slots)
    float wrow[kSlotTable];                        // W_i by row slot
    float wphys[kMaxDk];                           // w by physical row
    float ccol[DV];                                // previous c_j
    float ecol[DV];                                // c_j / c0_j
    float gcol[DV];                                // c_j / c'_j
};

// One row partial of a thread (4 columns of one row slot), combined with
// that of the neighbouring lane (the next 4 columns of the same row) before
// it goes to LDS.  Both lanes of a pair write the same value.
__device__ __forceinline__ void put_row_partial(RefitShared<128> &sh, int x, int cg, float acc)
{
    sh.u.rowp[x][cg >> 1] = acc + dpp_term<0xB1, 0xF>(acc);    // quad_perm [1,0,3,2]
}

// Row partial over the thread's 4 columns: sum_e c_e |y_e| (dual axis) or
// max_e c_e |y_e| (row absmax).
template <Refit MODE>
__device__ __forceinline__ float row_partial(const float *y, const float (&cc)[4])
{
    if constexpr (MODE == Refit::DualAxis) {
        float acc = fabsf(y[0]) * cc[0];
        acc = fmaf(fabsf(y[1]), cc[1], acc);
        acc = fmaf(fabsf(y[2]), cc[2], acc);
        return fmaf(fabsf(y[3]), cc[3], acc);
    } else {
        return fmaxf(fmaxf(fabsf(y[0]) * cc[0], fabsf(y[1]) * cc[1]), fmaxf(fabsf(y[2]) * cc[2], fabsf(y[3]) * cc[3]));
    }
}

// A row of width bw and old scale r_p: r' from its PR lane partials, and h
// and W.  The partials are sums (or
// maxima) of c_j |y_ij| with y = X / (r c nu), nu the width's level step:
// the mean |X_ij| is r nu sum / d_v, W = (w r' nu)^2, and the row-absmax
// factor r' = r max / q_b puts the row's largest entry on the top level in
// either normalisation.  The row and column
// factors are formed with the hardware reciprocal and square root (about one
// ulp each): every later step uses the stored fp32 values, so the codes stay
// consistent with them.
template <Refit MODE, int PR>
__device__ __forceinline__ float refit_row(const float4 *part, int bw, float r_p, float w, const LevelTable &lv,
                                           float &h, float &W)
{
    const float iq = bw == 8 ? (1.0f / 127.0f) : (bw == 4 ? (1.0f / 7.0f) : 1.0f);     // 1 / q_b
    const float nu = by_width(lv.nu, bw);
    if constexpr (MODE == Refit::RowAbsmax) {
        float mx = 0.f;
#pragma unroll
        for (int l = 0; l < PR / 4; ++l) {
            const float4 v4 = part[l];
            mx = fmaxf(mx, fmaxf(fmaxf(v4.x, v4.y), fmaxf(v4.z, v4.w)));
        }
        const float rn = fmaxf((r_p * iq) * mx, kScaleFloor);
        h = r_p * __builtin_amdgcn_rcpf(rn);
        W = 0.f;
        return rn;
    }
    float sum = 0.f;
#pragma unroll
    for (int l = 0; l < PR / 4; ++l) {
        const float4 v4 = part[l];
        sum += (v4.x + v4.y) + (v4.z + v4.w);
    }
    const float m = (r_p * nu) * (sum * (1.0f / static_cast<float>(8 * PR)));
    const float rn = fmaxf(__builtin_amdgcn_sqrtf(m * __builtin_amdgcn_rcpf(w)), kScaleFloor);
    h = r_p * __builtin_amdgcn_rcpf(rn);
    const float t = (w * rn) * nu;
    W = t * t;
    return rn;
}

// Per-thread column maxima of |yh| kept per width, divided by q_b once.
__device__ __forceinline__ float4 width_max(const float (&m8)[4], const float (&m4)[4], const float (&m2)[4])
{
    float r[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = fmaxf(fmaxf(m8[e] * (1.0f / 127.0f), m4[e] * (1.0f / 7.0f)), m2[e]);
    return make_float4(r[0], r[1], r[2], r[3]);
}

// Column j: absmax start c0_j from the slice maxima; e_j = c_j / c0_j.
template <int DV, class SH>
__device__ __forceinline__ void refit_colmax(SH &sh, int j)
{
    constexpr int NSL = 256 / (DV / 4);
    const float *mx = reinterpret_cast<const float *>(&sh.u.cmax[0][0]);
    float M = 0.f;
#pragma unroll
    for (int s = 0; s < NSL; ++s) M = fmaxf(M, mx[s * DV + j]);
    const float cj = sh.ccol[j];
    const float c0 = fmaxf(cj * M, kScaleFloor);
    sh.ecol[j] = M > 0.f ? cj * __builtin_amdgcn_rcpf(c0) : 0.f;
}

// Column j: the least-squares column factor from the slice sums in d.red.
template <int DV, class SH>
__device__ __forceinline__ void refit_colfit(SH &sh, int j, float *cc_out)
{
    constexpr int NSL = 256 / (DV / 4);
    const float *rn = reinterpret_cast<const float *>(&sh.d.red[0][0][0]);
    const float *rd = reinterpret_cast<const float *>(&sh.d.red[1][0][0]);
    float num = rn[j], den = rd[j];
#pragma unroll
    for (int s = 1; s < NSL; ++s) {
        num += rn[s * DV + j];
        den += rd[s * DV + j];
    }
    const float cj = sh.ccol[j];
    // num / den as a full division: den may be tiny for very small states
    const float cn = den > 0.f ? fmaxf(cj * (num / den), kScaleFloor) : cj;
    sh.gcol[j] = cj * __builtin_amdgcn_rcpf(cn);
    cc_out[j] = cn;
}

// ---- per-word passes on values held in registers (4 columns x 8/B rows)

// y of a word from the row-pair registers of the matrix-core path; the row
// partial sum_e c_e |y| (or max) of each slot goes to LDS.  Slot s of the
// word is thread row r0 + s (a constant once the caller's loops unroll).
template <int B, bool DIAG>
__device__ __forceinline__ void word_y_p(const uint32_t (&Ub)[4][4][2], int r0, RefitShared<128> &sh, int x0, int cg,
                                         float al_w, const float (&bc)[4], const float (&cc)[4], float *Y)
{
#pragma unroll
    for (int s = 0; s < 8 / B; ++s) {
        const int r = r0 + s, g = r >> 2, h = (r >> 1) & 1;
        const float a_s = sh.d.av[x0 + s];
        const float al = DIAG ? sh.d.al[x0 + s] : al_w;
        float *y = Y + 4 * s;
        if (r & 1) {
            y[0] = fma_mix<1>(al, Ub[0][g][h], a_s * bc[0]);
            y[1] = fma_mix<1>(al, Ub[1][g][h], a_s * bc[1]);
            y[2] = fma_mix<1>(al, Ub[2][g][h], a_s * bc[2]);
            y[3] = fma_mix<1>(al, Ub[3][g][h], a_s * bc[3]);
        } else {
            y[0] = fma_mix<0>(al, Ub[0][g][h], a_s * bc[0]);
            y[1] = fma_mix<0>(al, Ub[1][g][h], a_s * bc[1]);
            y[2] = fma_mix<0>(al, Ub[2][g][h], a_s * bc[2]);
            y[3] = fma_mix<0>(al, Ub[3][g][h], a_s * bc[3]);
        }
        put_row_partial(sh, x0 + s, cg, row_partial<Refit::DualAxis>(y, cc));
    }
}

// Pass 1 of a uniform body with the gate term of y on the matrix cores
// (gate_on_matrix_cores must hold): per row group g and column e, one
// diagonal 4x4x4 block gives y = al U + (av_i bc_j) for the group's 4 rows
// (within one ulp of word_y_p's FMA); Y[4 r + e] for thread row r, and the
// row partials to LDS.
template <int M8, int M4, int M2>
__device__ __forceinline__ void refit_y_mfma(const uint32_t (&Ub)[4][4][2], RefitShared<128> &sh, int tid, int slice,
                                             int cg, float alpha, const float (&bc)[4], const float (&cc)[4],
                                             float (&Y)[64])
{
    constexpr int G4 = M8 / 4, G2 = (M8 + 2 * M4) / 4;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const float al = g < G4 ? alpha : (g < G2 ? alpha * (1.0f / 16.0f) : alpha * (1.0f / 64.0f));
        const u32x2 A = diag_operand(al, tid & 3);
        float as[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) as[k] = sh.d.av[thread_row_slot<M8, M4>(4 * g + k, slice)];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const f32x4 d = mfma4x4x4(A, Ub[e][g][0], Ub[e][g][1],
                                      f32x4{as[0] * bc[e], as[1] * bc[e], as[2] * bc[e], as[3] * bc[e]});
#pragma unroll
            for (int k = 0; k < 4; ++k) Y[4 * (4 * g + k) + e] = d[k];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            put_row_partial(sh, thread_row_slot<M8, M4>(4 * g + k, slice), cg,
                            row_partial<Refit::DualAxis>(&Y[4 * (4 * g + k)], cc));
    }
}

template <int B>
__device__ __forceinline__ void word_scale_max(float *Y, const float *hrow, int x0, float (&mx)[4])
{
#pragma unroll
    for (int s = 0; s < 8 / B; ++s) {
        const float h = hrow[x0 + s];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            Y[4 * s + e] *= h;
            mx[e] = fmaxf(mx[e], fabsf(Y[4 * s + e]));
        }
    }
}

// One row's share of the least-squares sums (4 columns).
__device__ __forceinline__ void row_fit(const float *Y, float W, const float (&ec)[4], float (&num)[4], float (&den)[4])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float yh = Y[e];
        // round to nearest even by the fp32 grid at 1.5 2^23 (|z| <= q_b):
        // one rounding of the exact product, in two full-rate operations
        const float z = fmaf(yh, ec[e], kRoundMagic) - kRoundMagic;
        const float u = W * z;
        num[e] = fmaf(u, yh, num[e]);
        den[e] = fmaf(u, z, den[e]);
    }
}

template <int B>
__device__ __forceinline__ void word_fit(const float *Y, const float *wrow, int x0, const float (&ec)[4],
                                         float (&num)[4], float (&den)[4])
{
#pragma unroll
    for (int s = 0; s < 8 / B; ++s) row_fit(Y + 4 * s, wrow[x0 + s], ec, num, den);
}

// New word: per field round(yh g_j) clamped to +-q_b, packed with a bias of
// 2^(B-1) that the final XOR removes (as in the frozen-scale requantizer).
template <int B>
__device__ __forceinline__ uint32_t word_requant(const float *Y, const float (&g)[4])
{
    constexpr float bias = static_cast<float>(1 << (B - 1));
    constexpr float top = static_cast<float>((1 << B) - 1);
    constexpr uint32_t flip = B == 8 ? 0x80808080u : (B == 4 ? 0x88888888u : 0xAAAAAAAAu);
    uint32_t out = 0;
#pragma unroll
    for (int s = 0; s < 8 / B; ++s) {
        uint32_t P = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float y = fmaf(Y[4 * s + e], g[e], bias);
            y = __builtin_amdgcn_fmed3f(y, 1.0f, top);
            P = __builtin_amdgcn_cvt_pk_u8_f32(y, e, P);
        }
        out |= P << (s * B);
    }
    return out ^ flip;
}

__device__ __forceinline__ void ld4(const float *p, float (&v)[4])
{
    const float4 t = *reinterpret_cast<const float4 *>(p);
    v[0] = t.x;
    v[1] = t.y;
    v[2] = t.z;
    v[3] = t.w;
}

// Uniform layouts at d_v = 128: widths known at compile time, all 64 values
// of the thread kept in registers across the four passes.  PIV: a padded
// pivot head (up to kCompactPivots FP16 pivot rows beside the padded mix,
// t.hi from the head list): its pivot rows join the sums over rows and are
// updated in binary16, and take no part in the fits; the padded mix's empty
// slots (zero codes, no row) get h = W = 0, so they add nothing to the fits
// and keep zero codes.
template <bool BF16, bool DIAG, int M8, int M4, int M2, bool PIV = false>
__device__ __forceinline__ void refit_uniform(const DecodeArgs &a, const TileCtx &t, RefitShared<128> &sh)
{
    // uniform layouts take the lean row-absmax body of stepq_rowmax.hip
    constexpr int M = M8 + M4 + M2;
    constexpr int NE = 4 * (M8 + 2 * M4 + 4 * M2);
    constexpr int X4 = 8 * M8, X2 = 8 * M8 + 16 * M4;
    constexpr int Y4 = 4 * M8, Y2 = 4 * M8 + 8 * M4;     // value offsets of the 4- and 2-bit words
    const int tid = threadIdx.x;
    const int cg = tid & 31, slice = tid >> 5;
    float *rr_out = const_cast<float *>(t.rr);
    float *cc_out = const_cast<float *>(t.cc);
    const LevelTable lv = hold_levels(a.pool.lv);
    const CodeWords cw(t.codes, 1024u * M);
    uint32_t w[M];
#pragma unroll
    for (int m = 0; m < M; ++m) w[m] = cw.load_m(tid, m);
    PivotRegs<128, kCompactPivots> pr;
    if constexpr (PIV) pivot_load<128, kCompactPivots>(t, slice, cg, pr);

    const RowColOps<BF16> op = load_ops<BF16, DIAG, 128>(a, 128, t.tile, t.b, t.hq, t.h, t.rr, t.cc);
    if (tid < 128) sh.wphys[tid] = (a.pool.roww + static_cast<size_t>(t.h) * 128)[static_cast<unsigned>(tid)];
    else sh.ccol[tid - 128] = op.c;
    // S^T k and S^T q on the matrix cores, as in the frozen-scale body
    int ek, eq;
    float kappa;
    if constexpr (PIV)
        kappa = row_constants_mfma_piv<DIAG, M8, M4, M2, 128>(t.hi, t.alpha, t.beta, op, sh.d, lv, ek, eq);
    else
        kappa = row_constants_mfma<DIAG, M8, M4, M2, 128>(t.beta, op, sh.d, lv, ek, eq);
    uint32_t Ub[4][4][2];
    unpack_row_pairs<M8, M4, M2>(w, Ub);
    __syncthreads();    // operand table written
    matvec_partials(sh.d, slice, cg, Ub, ek, eq);
    if constexpr (PIV) pivot_partials_slice(t, slice, cg, pr, sh.d);

    column_sums<128>(a, t.tile, DIAG ? 1.0f : t.alpha, t.beta, sh.d, kappa, op.c, op.v());

    // pass 1: y on the old scales and the row partials
    float bc[4], cc[4];
    ld4(&sh.d.bcol[4 * cg], bc);
    ld4(&sh.ccol[4 * cg], cc);
    if constexpr (PIV) pivot_update<128, kCompactPivots>(t, slice, cg, pr, sh.d, bc);
    float Y[NE];
    bool y_done = false;
    if constexpr (!DIAG) {
        if (gate_on_matrix_cores<M8, M4, M2>(t.alpha)) {
            refit_y_mfma<M8, M4, M2>(Ub, sh, tid, slice, cg, t.alpha, bc, cc, Y);
            y_done = true;
        }
    }
    if (!y_done) {
#pragma unroll
        for (int m = 0; m < M8; ++m)
            word_y_p<8, DIAG>(Ub, m, sh, slice + 8 * m, cg, t.alpha, bc, cc, &Y[4 * m]);
#pragma unroll
        for (int m = 0; m < M4; ++m)
            word_y_p<4, DIAG>(Ub, M8 + 2 * m, sh, X4 + 2 * (slice + 8 * m), cg, t.alpha * (1.0f / 16.0f), bc,
                                    cc, &Y[Y4 + 8 * m]);
#pragma unroll
        for (int m = 0; m < M2; ++m)
            word_y_p<2, DIAG>(Ub, M8 + 2 * M4 + 4 * m, sh, X2 + 4 * (slice + 8 * m), cg,
                                    t.alpha * (1.0f / 64.0f), bc, cc, &Y[Y2 + 16 * m]);
    }
    __syncthreads();
    if (tid < 128) {
        if constexpr (PIV) {
            // row-table slot tid holds physical row p, or no row
            int bw;
            const int p = slot_row(t.hi, tid, bw);
            if (p >= 0) {
                rr_out[p] = refit_row<Refit::DualAxis, 16>(reinterpret_cast<const float4 *>(&sh.u.rowp[tid][0]), bw, sh.d.sr[p],
                                                sh.wphys[p], lv, sh.hrow[tid], sh.wrow[tid]);
            } else {
                sh.hrow[tid] = 0.f;
                sh.wrow[tid] = 0.f;
            }
        } else {
            rr_out[tid] = refit_row<Refit::DualAxis, 16>(reinterpret_cast<const float4 *>(&sh.u.rowp[tid][0]),
                                              tid < X4 ? 8 : (tid < X2 ? 4 : 2), op.r, sh.wphys[tid], lv,
                                              sh.hrow[tid], sh.wrow[tid]);
        }
    }
    __syncthreads();

    // pass 2: yh = y r / r' and the column maxima per width
    {
        float mx8[4] = {0.f, 0.f, 0.f, 0.f}, mx4[4] = {0.f, 0.f, 0.f, 0.f}, mx2[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int m = 0; m < M8; ++m) word_scale_max<8>(&Y[4 * m], sh.hrow, slice + 8 * m, mx8);
#pragma unroll
        for (int m = 0; m < M4; ++m) word_scale_max<4>(&Y[Y4 + 8 * m], sh.hrow, X4 + 2 * (slice + 8 * m), mx4);
#pragma unroll
        for (int m = 0; m < M2; ++m) word_scale_max<2>(&Y[Y2 + 16 * m], sh.hrow, X2 + 4 * (slice + 8 * m), mx2);
        sh.u.cmax[slice][cg] = width_max(mx8, mx4, mx2);
    }
    __syncthreads();
    if (tid >= 128) refit_colmax<128>(sh, tid - 128);
    __syncthreads();

    // pass 3: fixed codes and the least-squares sums
    {
        float ec[4];
        ld4(&sh.ecol[4 * cg], ec);
        float num[4] = {0.f, 0.f, 0.f, 0.f}, den[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int m = 0; m < M8; ++m) word_fit<8>(&Y[4 * m], sh.wrow, slice + 8 * m, ec, num, den);
#pragma unroll
        for (int m = 0; m < M4; ++m) word_fit<4>(&Y[Y4 + 8 * m], sh.wrow, X4 + 2 * (slice + 8 * m), ec, num, den);
#pragma unroll
        for (int m = 0; m < M2; ++m) word_fit<2>(&Y[Y2 + 16 * m], sh.wrow, X2 + 4 * (slice + 8 * m), ec, num, den);
        sh.d.red[0][slice][cg] = make_float4(num[0], num[1], num[2], num[3]);
        sh.d.red[1][slice][cg] = make_float4(den[0], den[1], den[2], den[3]);
    }
    __syncthreads();
    if (tid >= 128) refit_colfit<128>(sh, tid - 128, cc_out);
    __syncthreads();

    // pass 4: requantize on the new scales, store in place
    float g[4];
    ld4(&sh.gcol[4 * cg], g);
#pragma unroll
    for (int m = 0; m < M8; ++m) cw.store_m(tid, m, word_requant<8>(&Y[4 * m], g));
#pragma unroll
    for (int m = 0; m < M4; ++m)
        cw.store_m(tid, M8 + m, word_requant<4>(&Y[Y4 + 8 * m], g));
#pragma unroll
    for (int m = 0; m < M2; ++m)
        cw.store_m(tid, M8 + M4 + m, word_requant<2>(&Y[Y2 + 16 * m], g));
}

// ---- heads of any mix (the slot bodies of stepq_slots.h): the thread's rows
// in NP pairs of slots, all values in registers through the passes as in the
// uniform body.  Slots without a row have al = av = 0, so y = 0 there, and
// h = W = 0: they add nothing to the sums and maxima.
//
// Bound by VALU issue (about 4.6 cycles per wave64 instruction and SIMD, in
// every instruction class of these bodies), so what counts is the number of
// instructions.  Keeping the values and taking the width tests as scalar
// branches, against bodies that unpacked the words again in each pass
// (generic) or tested each lane's width in each word-step (row-mix): a
// 512-request x 16-head row-unit map with channel-wise gates 120.7 -> 98.4 us
// (1,942 -> 1,645 instructions per wave), 201 requests x 6 heads of random
// 2/4/8-bit rows at d_k = 96, d_v = 64 16.0 -> 10.9 us.

// ROWMIX: the first half is the frozen row-mix body's (rowmix_sums, with its
// own row tables in d); the slot constants are then copies of those.
template <int DV, int NP, bool ROWMIX>
struct SlotRefitShared {
    using D = SlotShared<DV, NP>;
    static constexpr int PR = DV / 8;              // partials per row: one per column-lane pair
    typename std::conditional<ROWMIX, DecodeShared<128>, D>::type d;
    union {
        // partials of sum_j c_j |y_ij| by slice and slot; the slices' tables
        // are PR floats apart from a multiple of the banks
        float rowp[D::NSL][(D::NR + 1) * PR];
        float4 cmax[D::NSL][D::CG];
    } u;
    alignas(16) float av[ROWMIX ? D::NSL : 1][D::NR], al[ROWMIX ? D::NSL : 1][D::NR];
    alignas(16) float hrow[D::NSL][D::NR];         // r_i / r'_i (0 for slots without a row)
    alignas(16) float wrow[D::NSL][D::NR];         // W_i
    float ccol[DV], ecol[DV], gcol[DV];            // c_j, c_j / c0_j, c_j / c'_j
};

// The row partial of slot r, combined with the neighbouring lane's (the next
// 4 columns of the row); both lanes of a pair write the same value.
template <Refit MODE>
__device__ __forceinline__ void put_slot_partial(float *rowp, int r, int pr, float acc)
{
    if constexpr (MODE == Refit::DualAxis) acc += dpp_term<0xB1, 0xF>(acc);    // quad_perm [1,0,3,2]
    else acc = __uint_as_float(max(__float_as_uint(acc), dpp_bits<0xB1, 0xF>(__float_as_uint(acc))));
    rowp[r * pr] = acc;
}

// Slots of B-bit rows from Y (4 columns each), packed without the bias flip.
template <int B, int NS>
__device__ __forceinline__ uint32_t requant_rows(const float *Y, const float (&g)[4])
{
    constexpr float bias = static_cast<float>(1 << (B - 1));
    constexpr float top = static_cast<float>((1 << B) - 1);
    uint32_t out = 0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        uint32_t P = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            P = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_amdgcn_fmed3f(fmaf(Y[4 * s + e], g[e], bias), 1.0f, top), e, P);
        out |= P << (s * B);
    }
    return out;
}

// The unpacked fields of the thread's rows as fp32, in the registers that
// hold the values afterwards.
template <int NP, bool HAS2>
__device__ __forceinline__ void slot_fields(const SlotGeom &g, uint32_t live, const uint32_t (&wa)[NP], const uint32_t (&wb)[NP],
                                            float (&Y)[NP][8])
{
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        if (!(live >> p & 1u)) continue;
        uint32_t lo, hi;
        slot_views<NP, HAS2>(g, wa, wb, p, lo, hi);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            Y[p][e] = sbyte(lo, e);
            Y[p][4 + e] = sbyte(hi, e);
        }
    }
}

template <bool BF16, bool DIAG, int DV, int NP, bool HAS2, int PMAX, Refit MODE, bool ROWMIX>
__device__ __forceinline__ void refit_slots(const DecodeArgs &a, const TileCtx &t, SlotRefitShared<DV, NP, ROWMIX> &sh)
{
    using SH = SlotRefitShared<DV, NP, ROWMIX>;
    using D = typename SH::D;
    const int tid = threadIdx.x;
    const int cg = tid % D::CG, slice = tid / D::CG;
    const int dk = a.pool.dk;
    float *rr_out = const_cast<float *>(t.rr);
    float *cc_out = const_cast<float *>(t.cc);
    const SlotGeom g(t.hi, D::NSL == 8 ? 3 : 4);
    const LevelTable lv = hold_levels(a.pool.lv);
    const SlotWords<DV> cw(t.codes, g, slice);
    // Pairs without a row in this wave are left out of the passes: d_k = 96, d_v
    // = 64 with rows of 2/4/8 bits at random, 201 requests x 6 heads, 14.5 -> 10.9
    // us; 256 x 16 heads of d_k = 72, d_v = 128 37.8 -> 30.3 us; d_k = 128 59.3 ->
    // 59.2 us.  The row-mix launches have few such pairs (9 for 8 pairs' rows;
    // the tests cost more: 98.4 -> 101.7 us), and so have the row absmax's three
    // passes (from 4% slower to 6% faster): those run all pairs.
    constexpr bool kSkip = !ROWMIX && MODE == Refit::DualAxis;
    // Without those branches the weights of later pairs are read ahead into
    // registers.  Kept in order where that crosses a step of occupancy: at 10
    // pairs (spills at 4 waves per SIMD; d_k = 120 rows @8 / @4, 256 x 16 heads
    // 40.9 -> 34.5 us), at 4 with the scalar gate (7 waves; d_k = d_v = 64, 400 x
    // 12 heads 19.5 -> 17.5 us); elsewhere it is 1 to 5% slower.
    constexpr bool kInOrder = MODE == Refit::RowAbsmax && (NP == 10 || (NP == 4 && !DIAG));
    const uint32_t live = kSkip ? live_pairs<D::NSL>(g, slice) : ~0u;
    uint32_t wa[NP], wb[NP];
    u32x16 w16;
    const int ng = g.g8 + g.g4;
    if constexpr (ROWMIX) {
        // the codes region only (128 ng bytes): words past the head's last group read 0
        const CodeWords all(t.codes, t.hi.piv_off);
#pragma unroll
        for (int m = 0; m < 16; ++m) w16[m] = 8 * m < ng ? all.load(tid + 256 * m) : 0u;
    } else {
        slot_load<DV, NP, HAS2>(cw, g, wa, wb);
    }
    PivotRegs<DV, PMAX> pr;
    pivot_load(t, slice, cg, pr);
    const RowColOps<BF16> op = load_ops<BF16, DIAG, DV>(a, dk, t.tile, t.b, t.hq, t.h, t.rr, t.cc);
    const SlotRow row = slot_of_row<D::NSL>(t.hi, g, tid, dk);
    float w_row = 1.0f;
    if (MODE == Refit::DualAxis && row.slice >= 0) w_row = a.pool.roww[t.h * dk + tid];
    const int col = own_column<DV>();
    if (col >= 0) sh.ccol[col] = op.c;
    if (tid < D::NSL * D::NR) {
        (&sh.hrow[0][0])[tid] = 0.f;
        (&sh.wrow[0][0])[tid] = 0.f;
        if constexpr (ROWMIX) {
            (&sh.av[0][0])[tid] = 0.f;
            (&sh.al[0][0])[tid] = 0.f;
        }
    }
    // The row sums keep the order of the rows (8-, 4-, then 2-bit words of the
    // slice, then the slices): a fixed code of the fit that lies near a
    // rounding boundary depends on their last bits.
    float Y[NP][8];
    if constexpr (ROWMIX) {
        rowmix_sums<DIAG, false>(a, t, sh.d, w16, pr, op, lv, g.g8, ng, [&] {
            if (row.slice >= 0) {
                // row-table slot of physical row tid: the integer rows in order
                const int x = tid - static_cast<int>(t.hi.n16);
                sh.av[row.slice][row.r] = sh.d.av[x];
                sh.al[row.slice][row.r] = DIAG ? sh.d.al[x] : (row.bw == 8 ? t.alpha : t.alpha * (1.0f / 16.0f));
            }
        });
        // the words by class: 8-bit word-step m is m, a slice's 4-bit words
        // follow its 8-bit ones (one earlier in slices past the class's end)
        const bool early = g.g8 % 8 != 0 && slice >= g.g8 % 8;
        const int m4 = (g.g8 + 7) >> 3;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            wa[p] = wb[p] = 0u;
            if (p < g.p4) {
                wa[p] = 2 * p < 16 ? w16[2 * p < 16 ? 2 * p : 0] : 0u;
                wb[p] = 2 * p + 1 < 16 ? w16[2 * p + 1 < 16 ? 2 * p + 1 : 0] : 0u;
            } else if (p < g.pt) {
                const int i = m4 + p - g.p4;
                const uint32_t late = i < 16 ? w16[i & 15] : 0u, soon = w16[(i - 1) & 15];
                wa[p] = early ? soon : late;
            }
        }
        slot_fields<NP, HAS2>(g, live, wa, wb, Y);
    } else {
        // in scalar registers once they have come: held as loaded, two vector
        // registers more make the launch bounds spill
        const float alpha = uniform_f(t.alpha), beta = uniform_f(t.beta);
        const float kappa = slot_constants<DIAG>(t.hi, dk, alpha, beta, op, sh.d, lv, row);
        slot_fields<NP, HAS2>(g, live, wa, wb, Y);
        // row-mix heads: two chains a column and the slices in pairs: o's error
        // against 64 bits (64 requests x 16 heads, channel-wise gates, fp32) is
        // 9.0e-8, as with the matrix cores' fewer roundings; 9.7e-8 in one chain
        constexpr bool kTwoChains = !HAS2;
        float acK[4] = {0.f, 0.f, 0.f, 0.f}, acQ[4] = {0.f, 0.f, 0.f, 0.f};
        float acK1[4] = {0.f, 0.f, 0.f, 0.f}, acQ1[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            if (!(live >> p & 1u)) continue;
            const float4 c = *reinterpret_cast<const float4 *>(&sh.d.kq[slice][2 * p]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (kTwoChains) {
                    acK[e] = fmaf(c.x, Y[p][e], acK[e]);
                    acQ[e] = fmaf(c.y, Y[p][e], acQ[e]);
                    acK1[e] = fmaf(c.z, Y[p][4 + e], acK1[e]);
                    acQ1[e] = fmaf(c.w, Y[p][4 + e], acQ1[e]);
                } else {
                    acK[e] = fmaf(c.z, Y[p][4 + e], fmaf(c.x, Y[p][e], acK[e]));
                    acQ[e] = fmaf(c.w, Y[p][4 + e], fmaf(c.y, Y[p][e], acQ[e]));
                }
            }
            if constexpr (kInOrder) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (kTwoChains) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acK[e] += acK1[e];
                acQ[e] += acQ1[e];
            }
        }
        pivot_acc(t, slice, cg, pr, sh.d, acK, acQ);
        sh.d.red[0][slice][cg] = make_float4(acK[0], acK[1], acK[2], acK[3]);
        sh.d.red[1][slice][cg] = make_float4(acQ[0], acQ[1], acQ[2], acQ[3]);
        column_sums<DV, false, kTwoChains>(a, t.tile, DIAG ? 1.0f : alpha, beta, sh.d, kappa,
                                           sh.d.cpiv[tid & (DV - 1)], sh.d.bcol[tid & (DV - 1)]);
    }

    // pass 1: y on the old scales and the row partials
    float bc[4], cc[4];
    ld4(&sh.d.bcol[4 * cg], bc);
    ld4(&sh.ccol[4 * cg], cc);
    pivot_update(t, slice, cg, pr, sh.d, bc);      // pivot rows take no part in the fits
    const float *avs, *als;
    if constexpr (ROWMIX) {
        avs = sh.av[slice];
        als = sh.al[slice];
    } else {
        avs = sh.d.av[slice];
        als = sh.d.al[slice];
    }
    float *rowp = &sh.u.rowp[slice][cg >> 1];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        if (!(live >> p & 1u)) continue;
        const float2 as = *reinterpret_cast<const float2 *>(avs + 2 * p);
        const float2 ag = *reinterpret_cast<const float2 *>(als + 2 * p);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            Y[p][e] = fmaf(ag.x, Y[p][e], as.x * bc[e]);
            Y[p][4 + e] = fmaf(ag.y, Y[p][4 + e], as.y * bc[e]);
        }
        put_slot_partial<MODE>(rowp, 2 * p, SH::PR, row_partial<MODE>(&Y[p][0], cc));
        put_slot_partial<MODE>(rowp, 2 * p + 1, SH::PR, row_partial<MODE>(&Y[p][4], cc));
    }
    __syncthreads();
    if (row.slice >= 0) {
        const float4 *part = reinterpret_cast<const float4 *>(&sh.u.rowp[row.slice][row.r * SH::PR]);
        float h, W;
        rr_out[tid] = refit_row<MODE, SH::PR>(part, row.bw, op.r, w_row, lv, h, W);
        sh.hrow[row.slice][row.r] = h;
        if constexpr (MODE == Refit::DualAxis) sh.wrow[row.slice][row.r] = W;
    }
    if constexpr (MODE == Refit::RowAbsmax) {
        if (col >= 0) cc_out[col] = 1.0f;
    }
    __syncthreads();

    float gc[4];
    if constexpr (MODE == Refit::RowAbsmax) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            if (!(live >> p & 1u)) continue;
            const float2 h = *reinterpret_cast<const float2 *>(&sh.hrow[slice][2 * p]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                Y[p][e] = Y[p][e] * h.x;
                Y[p][4 + e] = Y[p][4 + e] * h.y;
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) gc[e] = cc[e];
    } else {
        // pass 2: yh = y r / r' and the column maxima per width
        {
            // the running maxima of one class fold into top[], divided by its
            // q_b, where the next class begins
            float mx[4] = {0.f, 0.f, 0.f, 0.f}, top[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                if (p == g.p4 || (HAS2 && p == g.p2 && g.p2 != g.p4)) {
                    const float f = p == g.p4 ? 1.0f / 127.0f : 1.0f / 7.0f;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        top[e] = fmaxf(top[e], mx[e] * f);
                        mx[e] = 0.f;
                    }
                }
                if (!(live >> p & 1u)) continue;
                const float2 h = *reinterpret_cast<const float2 *>(&sh.hrow[slice][2 * p]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    Y[p][e] = Y[p][e] * h.x;
                    Y[p][4 + e] = Y[p][4 + e] * h.y;
                    mx[e] = max3_abs(mx[e], Y[p][e], Y[p][4 + e]);
                }
            }
            const float f = HAS2 && g.p2 < g.pt ? 1.0f : (g.p4 < g.e4 ? 1.0f / 7.0f : 1.0f / 127.0f);
            sh.u.cmax[slice][cg] = make_float4(fmaxf(top[0], mx[0] * f), fmaxf(top[1], mx[1] * f),
                                               fmaxf(top[2], mx[2] * f), fmaxf(top[3], mx[3] * f));
        }
        __syncthreads();
        if (col >= 0) refit_colmax<DV>(sh, col);
        __syncthreads();

        // pass 3: fixed codes and the least-squares sums
        {
            float ec[4];
            ld4(&sh.ecol[4 * cg], ec);
            float num[4] = {0.f, 0.f, 0.f, 0.f}, den[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                if (!(live >> p & 1u)) continue;
                const float2 W = *reinterpret_cast<const float2 *>(&sh.wrow[slice][2 * p]);
                row_fit(&Y[p][0], W.x, ec, num, den);
                row_fit(&Y[p][4], W.y, ec, num, den);
            }
            sh.d.red[0][slice][cg] = make_float4(num[0], num[1], num[2], num[3]);
            sh.d.red[1][slice][cg] = make_float4(den[0], den[1], den[2], den[3]);
        }
        __syncthreads();
        if (col >= 0) refit_colfit<DV>(sh, col, cc_out);
        __syncthreads();
        ld4(&sh.gcol[4 * cg], gc);
    }

    // pass 4: requantize on the new scales, store in place
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        if (!(live >> p & 1u)) continue;
        if (p < g.p4) {
            cw.st8(2 * p, requant_rows<8, 1>(&Y[p][0], gc) ^ 0x80808080u);
            cw.st8(2 * p + 1, requant_rows<8, 1>(&Y[p][4], gc) ^ 0x80808080u);
        } else if (p < g.e4) {
            cw.st4(p - g.p4, requant_rows<4, 2>(&Y[p][0], gc) ^ 0x88888888u);
        } else if (HAS2 && (p & 1) == 0 && p >= g.p2 && p < g.pt) {
            const uint32_t P = requant_rows<2, 2>(&Y[p][0], gc) |
                               (requant_rows<2, 2>(&Y[p + 1 < NP ? p + 1 : p][0], gc) << 4);
            cw.st2((p - g.p2) >> 1, P ^ 0xAAAAAAAAu);
        }
    }
}

// A tile of uniform layout L: codes (1024 bytes per word-step), then r, c.
template <bool BF16, bool DIAG, int L>
__device__ __forceinline__ void run_refit_uniform(const DecodeArgs &a, TileCtx &t, int slot, RefitShared<128> &sh)
{
    constexpr UniformLayout u = kUniformLayouts[L - 1];
    constexpr uint32_t r_off = 1024u * (u.m8 + u.m4 + u.m2);
    uint8_t *rec = a.pool.base + static_cast<uint64_t>(slot) * a.pool.slot_bytes + t.off;
    t.codes = reinterpret_cast<uint32_t *>(rec);
    t.rr = reinterpret_cast<const float *>(rec + r_off);
    t.cc = t.rr + 128;
    refit_uniform<BF16, DIAG, u.m8, u.m4, u.m2>(a, t, sh);
}

// A padded pivot head of uniform layout L (its row counts from the head
// list), or a layout-L head taken as one with no pivot rows.
template <bool BF16, bool DIAG, int L>
__device__ __forceinline__ void run_refit_uniform_piv(const DecodeArgs &a, TileCtx &t, int slot, RefitShared<128> &sh)
{
    constexpr UniformLayout u = kUniformLayouts[L - 1];
    padded_pivot_tile<L>(a, t, slot);
    refit_uniform<BF16, DIAG, u.m8, u.m4, u.m2, true>(a, t, sh);
}

// NP: the row pairs of the slot bodies (layouts 0 and kRowMix; 0 for the
// compiled layouts).
// The slot bodies' second bound is the waves per SIMD that their 8 NP values
// leave room for; without it the compiler takes a few registers more than the
// next step of occupancy.  No body spills under it.
constexpr int refit_waves(int np) { return np == 0 ? 1 : (np <= 6 ? 5 : (np <= 10 ? 4 : 3)); }

template <int DV, bool BF16, int LAYOUT, bool DIAG, Refit MODE, int NP = 0>
__global__ __launch_bounds__(256, refit_waves(NP)) void refit_kernel(DecodeArgs a)
{
    // row-mix heads: the fit takes the frozen row-mix body's first half, the row
    // absmax the fp32 sums of every other mix in that step (512 requests x 16
    // heads with channel-wise gates: 60.0 us, with the binary16 split 75.5)
    constexpr bool ROWMIX = LAYOUT == kRowMix && MODE == Refit::DualAxis;
    using Shared = typename std::conditional<NP == 0, RefitShared<128>, SlotRefitShared<DV, NP == 0 ? 1 : NP, ROWMIX>>::type;
    __shared__ Shared sh;
    const PoolView &P = a.pool;
    TileCtx t;
    uint32_t tile_bytes = 0;
    constexpr bool UNIFORM = DV == 128 && LAYOUT > 0 && LAYOUT <= kNumUniformLayouts;
    if constexpr (UNIFORM) {
        constexpr UniformLayout u = kUniformLayouts[LAYOUT - 1];
        tile_bytes = 1024u * (u.m8 + u.m4 + u.m2 + 1);
    }
    tile_of(a, tile_bytes, t);
    const int slot = a.slot_ids[t.b];
    t.alpha = DIAG ? 1.0f : act_ld<BF16>(a.alpha, t.tile);
    t.beta = act_ld<BF16>(a.beta, t.tile);
    if constexpr (UNIFORM) {
        run_refit_uniform<BF16, DIAG, LAYOUT>(a, t, slot, sh);
    } else if constexpr (DV == 128 && LAYOUT > kPivotUniformBase && LAYOUT <= kPivotUniformBase + kNumUniformLayouts) {
        run_refit_uniform_piv<BF16, DIAG, LAYOUT - kPivotUniformBase>(a, t, slot, sh);
    } else if constexpr (DV == 128 && LAYOUT > kMixedPivotBase && LAYOUT <= kMixedPivotBase + 2) {
        // layout-L heads and layout-L padded pivot heads in one launch of one
        // body: a layout-L head is a padded pivot head with no pivot rows
        run_refit_uniform_piv<BF16, DIAG, LAYOUT - kMixedPivotBase>(a, t, slot, sh);
    } else if constexpr (DV == 128 && LAYOUT == kMultiUniform) {
        // heads of several uniform layouts and whole FP16 heads in one launch
        // (the head list), each tile on its own body; a whole FP16 head has
        // no integer rows to fit and takes the frozen-step body
        switch (t.layout) {
        case 1: run_refit_uniform<BF16, DIAG, 1>(a, t, slot, sh); break;
        case 2: run_refit_uniform<BF16, DIAG, 2>(a, t, slot, sh); break;
        case 3: run_refit_uniform<BF16, DIAG, 3>(a, t, slot, sh); break;
        case 4: run_refit_uniform<BF16, DIAG, 4>(a, t, slot, sh); break;
        case 5: run_refit_uniform<BF16, DIAG, 5>(a, t, slot, sh); break;
        default: run_f16head<BF16, DIAG>(a, t, slot, sh.d); break;
        }
    } else {
        t.hi = head_info(P, t.h);
        uint8_t *rec = P.base + static_cast<uint64_t>(slot) * P.slot_bytes + t.hi.tile_off;
        t.codes = reinterpret_cast<uint32_t *>(rec);
        t.rr = reinterpret_cast<const float *>(rec + t.hi.r_off);
        t.cc = t.rr + P.dk;
        refit_slots<BF16, DIAG, DV, NP, LAYOUT != kRowMix, LAYOUT == kRowMix ? kCompactPivots : kMaxPivots, MODE, ROWMIX>(
            a, t, sh);
    }
}

// Heads of any mix at the compiled pair count that holds the launch's
// largest head.
template <bool BF16, bool DIAG, Refit MODE>
hipError_t launch_refit_slots(const DecodeArgs &a, int pairs, unsigned grid, hipStream_t s)
{
    const int np = slot_pairs_compiled(pairs, a.pool.dv);
    if (a.pool.dv == 64) {
        switch (np) {
        case 4: hipLaunchKernelGGL((refit_kernel<64, BF16, 0, DIAG, MODE, 4>), dim3(grid), dim3(256), 0, s, a); break;
        case 6: hipLaunchKernelGGL((refit_kernel<64, BF16, 0, DIAG, MODE, 6>), dim3(grid), dim3(256), 0, s, a); break;
        default:
            hipLaunchKernelGGL((refit_kernel<64, BF16, 0, DIAG, MODE, kSlotPairs64>), dim3(grid), dim3(256), 0, s, a);
            break;
        }
    } else {
        switch (np) {
        case 6: hipLaunchKernelGGL((refit_kernel<128, BF16, 0, DIAG, MODE, 6>), dim3(grid), dim3(256), 0, s, a); break;
        case 8: hipLaunchKernelGGL((refit_kernel<128, BF16, 0, DIAG, MODE, 8>), dim3(grid), dim3(256), 0, s, a); break;
        case 10: hipLaunchKernelGGL((refit_kernel<128, BF16, 0, DIAG, MODE, 10>), dim3(grid), dim3(256), 0, s, a); break;
        default:
            hipLaunchKernelGGL((refit_kernel<128, BF16, 0, DIAG, MODE, kSlotPairsAny>), dim3(grid), dim3(256), 0, s, a);
            break;
        }
    }
    return hipGetLastError();
}

template <bool BF16, bool DIAG, Refit MODE>
hipError_t launch_refit_any(const DecodeArgs &a, int layout, int pairs, unsigned grid, hipStream_t s)
{
    if (a.pool.dv == 128 && layout == kRowMix) {
        hipLaunchKernelGGL((refit_kernel<128, BF16, kRowMix, DIAG, MODE, kSlotPairs84>), dim3(grid), dim3(256), 0, s, a);
        return hipGetLastError();
    }
    if constexpr (MODE == Refit::DualAxis) {
        // (in the row-absmax step uniform layouts are launched on the lean body, launch_decode_rowmax)
        switch (a.pool.dv == 128 ? layout : 0) {
        case 1: hipLaunchKernelGGL((refit_kernel<128, BF16, 1, DIAG, MODE>), dim3(grid), dim3(256), 0, s, a); break;
        case 2: hipLaunchKernelGGL((refit_kernel<128, BF16, 2, DIAG, MODE>), dim3(grid), dim3(256), 0, s, a); break;
        case 3: hipLaunchKernelGGL((refit_kernel<128, BF16, 3, DIAG, MODE>), dim3(grid), dim3(256), 0, s, a); break;
        case 4: hipLaunchKernelGGL((refit_kernel<128, BF16, 4, DIAG, MODE>), dim3(grid), dim3(256), 0, s, a); break;
        case 5: hipLaunchKernelGGL((refit_kernel<128, BF16, 5, DIAG, MODE>), dim3(grid), dim3(256), 0, s, a); break;
        case kMultiUniform:
            hipLaunchKernelGGL((refit_kernel<128, BF16, kMultiUniform, DIAG, MODE>), dim3(grid), dim3(256), 0, s, a);
            break;
        case kPivotUniformBase + 1:
            hipLaunchKernelGGL((refit_kernel<128, BF16, kPivotUniformBase + 1, DIAG, MODE>), dim3(grid), dim3(256), 0, s, a);
            break;
        case kPivotUniformBase + 2:
            hipLaunchKernelGGL((refit_kernel<128, BF16, kPivotUniformBase + 2, DIAG, MODE>), dim3(grid), dim3(256), 0, s, a);
            break;
        case kPivotUniformBase + 3:
            hipLaunchKernelGGL((refit_kernel<128, BF16, kPivotUniformBase + 3, DIAG, MODE>), dim3(grid), dim3(256), 0, s, a);
            break;
        case kPivotUniformBase + 4:
            hipLaunchKernelGGL((refit_kernel<128, BF16, kPivotUniformBase + 4, DIAG, MODE>), dim3(grid), dim3(256), 0, s, a);
            break;
        case kPivotUniformBase + 5:
            hipLaunchKernelGGL((refit_kernel<128, BF16, kPivotUniformBase + 5, DIAG, MODE>), dim3(grid), dim3(256), 0, s, a);
            break;
        case kMixedPivotBase + 1:
            hipLaunchKernelGGL((refit_kernel<128, BF16, kMixedPivotBase + 1, DIAG, MODE>), dim3(grid), dim3(256), 0, s, a);
            break;
        case kMixedPivotBase + 2:
            hipLaunchKernelGGL((refit_kernel<128, BF16, kMixedPivotBase + 2, DIAG, MODE>), dim3(grid), dim3(256), 0, s, a);
            break;
        default: return launch_refit_slots<BF16, DIAG, MODE>(a, pairs, grid, s);
        }
        return hipGetLastError();
    }
    return launch_refit_slots<BF16, DIAG, MODE>(a, pairs, grid, s);
}

template <Refit MODE>
hipError_t launch_refit_mode(const DecodeArgs &a, bool bf16, bool diag, int pool_layout, int pairs, hipStream_t stream)
{
    const unsigned grid = static_cast<unsigned>(a.batch) * static_cast<unsigned>(a.n_heads);
    if (grid == 0) return hipSuccess;
    if (bf16) return diag ? launch_refit_any<true, true, MODE>(a, pool_layout, pairs, grid, stream)
                          : launch_refit_any<true, false, MODE>(a, pool_layout, pairs, grid, stream);
    return diag ? launch_refit_any<false, true, MODE>(a, pool_layout, pairs, grid, stream)
                : launch_refit_any<false, false, MODE>(a, pool_layout, pairs, grid, stream);
}

}  // namespace
}  // namespace stepq
