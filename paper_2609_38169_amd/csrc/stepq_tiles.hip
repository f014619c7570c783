// Whole-tile operations off the decode path: pack (from fp32 states or raw
// codes), unpack and dequantize, one 256-thread workgroup per tile.
//
// Memory bound: each moves a tile's rows between the caller's row-major
// arrays and the record once, so what counts is bytes per instruction and
// loads in flight.  A thread owns V neighbouring columns of every NS-th row
// group: V = 16 where the caller's rows are bytes, 8 for binary16, 4 for fp32,
// one 16-byte access a row.  The classes are walked one after the other with
// several words' rows loaded before the first is used; the permutation and the
// row scales wait in LDS.  Rows are whole multiples of 16 bytes, but the
// caller's base pointers need only their element's alignment: accesses to
// them are typed so.  Against the earlier one-word, one-dword-per-access form:
// pack of 64 requests x 32 heads 41.4 -> 32.5 us, export + import with FP16
// rows of 32 requests x 32 heads 72.1 -> 35.2 us (four calls; the host's share is
// in stepq_args.cpp).
#include "stepq_device.h"

namespace stepq {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4_any1 __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u32x4_any2 __attribute__((ext_vector_type(4), aligned(2)));

// A tile of the call: its record and where its rows sit in the caller's arrays.
struct TileRef {
    HeadInfo hi;
    uint8_t *rec;
    const uint8_t *perm;
    size_t tdk, tdv;      // first row and first column entry of the tile in r, c (and rows of the states)
};

__device__ __forceinline__ TileRef tile_ref(const TileArgs &a)
{
    const PoolView &P = a.pool;
    const int tile = blockIdx.x;
    const int n_i = fdiv(tile, P.div_hv);
    const int h = tile - n_i * P.Hv;
    TileRef t;
    t.hi = P.heads[h];
    t.rec = P.base + static_cast<uint64_t>(a.slot_ids[n_i]) * P.slot_bytes + t.hi.tile_off;
    t.perm = P.perm + h * P.dk;
    t.tdk = static_cast<size_t>(tile) * P.dk;
    t.tdv = static_cast<size_t>(tile) * P.dv;
    return t;
}

// Scales in, and zeros in the record's padding (end of the codes region, end
// of the record).  Leaves the permutation and r in LDS.
template <int DV>
__device__ __forceinline__ void take_scales(const TileArgs &a, const TileRef &t, int *sperm, float *sr)
{
    const int tid = threadIdx.x, dk = a.pool.dk;
    float *rr = reinterpret_cast<float *>(t.rec + t.hi.r_off);
    if (tid < dk) {
        const int i = t.perm[tid];
        const float r = a.r_in[t.tdk + i];
        sperm[tid] = i;
        sr[tid] = r;
        rr[tid] = r;
    }
    if (tid < DV) rr[dk + tid] = a.c_in[t.tdv + tid];
    uint32_t *rec32 = reinterpret_cast<uint32_t *>(t.rec);
    for (uint32_t d = t.hi.groups * (DV / 4) + tid; d < t.hi.piv_off / 4; d += 256) rec32[d] = 0u;
    for (uint32_t d = (t.hi.r_off + 4u * (dk + DV)) / 4 + tid; d < t.hi.tile_bytes / 4; d += 256) rec32[d] = 0u;
}

// The groups of one width class that a thread owns, N at a time: f(k0) gets
// the first of up to N groups k0, k0 + NS, ...; k counts within the class.
template <int NS, int N, class F>
__device__ __forceinline__ void each_batch(int first, int count, F &&f)
{
    for (int k = first; k < count; k += N * NS) f(k);
}

// Bytes with the B-bit fields of slot s of four packed words, sign-extended.
template <int B>
__device__ __forceinline__ u32x4 slot_bytes(u32x4 w, int s)
{
    constexpr uint32_t ones = 0x01010101u;
    constexpr uint32_t field = ones * ((1u << B) - 1u), sign = ones << (B - 1);
    if constexpr (B == 8) return w;
    const u32x4 x = (w >> (s * B)) & field;
    const u32x4 m = (x & sign) << 1;            // 2^B in the bytes of negative fields
    return x | ((m << (8 - B)) - m);            // 256 - 2^B there
}

// ---- raw codes out and in: 16 columns a thread

template <int DV, int B>
__device__ __forceinline__ void export_class(const TileArgs &a, const TileRef &t, const int *sperm, int g0, int p0,
                                             int rows, int slice, int col)
{
    constexpr int NS = 4096 / DV, S = 8 / B, N = 4 / S > 1 ? 4 / S : 1;
    each_batch<NS, N>(slice, (rows + S - 1) / S, [&](int k0) {
        u32x4 w[N];
#pragma unroll
        for (int n = 0; n < N; ++n)
            if (S * (k0 + NS * n) < rows)
                w[n] = *reinterpret_cast<const u32x4 *>(t.rec + static_cast<uint32_t>(g0 + k0 + NS * n) * DV + col);
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int x = S * (k0 + NS * n) + s;
                if (x < rows)
                    *reinterpret_cast<u32x4_any1 *>(a.codes_out + (t.tdk + sperm[p0 + x]) * DV + col) =
                        slot_bytes<B>(w[n], s);
            }
    });
}

template <int DV>
__global__ __launch_bounds__(256) void export_kernel(TileArgs a)
{
    __shared__ int sperm[kMaxDk];
    const TileRef t = tile_ref(a);
    const int tid = threadIdx.x, dk = a.pool.dk;
    const float *rr = reinterpret_cast<const float *>(t.rec + t.hi.r_off);
    if (tid < dk) {
        const int i = t.perm[tid];
        sperm[tid] = i;
        a.r_out[t.tdk + i] = rr[tid];
    }
    if (tid < DV) a.c_out[t.tdv + tid] = rr[dk + tid];
    __syncthreads();
    constexpr int LPR = DV / 16, NS = 256 / LPR;
    const int col = 16 * (tid % LPR), slice = tid / LPR;
    const HeadInfo &hi = t.hi;
    for (int p = slice; p < hi.n16; p += NS)     // FP16 rows hold no codes
        *reinterpret_cast<u32x4_any1 *>(a.codes_out + (t.tdk + sperm[p]) * DV + col) = u32x4{0u, 0u, 0u, 0u};
    export_class<DV, 8>(a, t, sperm, 0, hi.n16, hi.n8, slice, col);
    export_class<DV, 4>(a, t, sperm, hi.g8, hi.n16 + hi.n8, hi.n4, slice, col);
    export_class<DV, 2>(a, t, sperm, hi.g8 + hi.g4, hi.n16 + hi.n8 + hi.n4, hi.n2, slice, col);
}

// Groups g0 .. g0 + groups of one class; the fields of rows past the class's
// last (empty slots, padding groups) are 0.
template <int DV, int B>
__device__ __forceinline__ void import_class(const TileArgs &a, const TileRef &t, const int *sperm, int g0, int groups,
                                             int p0, int rows, int slice, int col)
{
    constexpr int NS = 4096 / DV, S = 8 / B, N = 4 / S > 1 ? 4 / S : 1;
    constexpr uint32_t field = 0x01010101u * ((1u << B) - 1u);
    each_batch<NS, N>(slice, groups, [&](int k0) {
        u32x4 c[N][S];
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int x = S * (k0 + NS * n) + s;
                c[n][s] = u32x4{0u, 0u, 0u, 0u};
                if (x < rows)
                    c[n][s] = *reinterpret_cast<const u32x4_any1 *>(a.codes_in + (t.tdk + sperm[p0 + x]) * DV + col);
            }
#pragma unroll
        for (int n = 0; n < N; ++n) {
            u32x4 w = c[n][0] & field;
#pragma unroll
            for (int s = 1; s < S; ++s) w |= (c[n][s] & field) << (s * B);
            if (k0 + NS * n < groups)
                *reinterpret_cast<u32x4 *>(t.rec + static_cast<uint32_t>(g0 + k0 + NS * n) * DV + col) = w;
        }
    });
}

template <int DV>
__global__ __launch_bounds__(256) void import_kernel(TileArgs a)
{
    __shared__ int sperm[kMaxDk];
    __shared__ float sr[kMaxDk];
    const TileRef t = tile_ref(a);
    take_scales<DV>(a, t, sperm, sr);
    __syncthreads();
    constexpr int LPR = DV / 16;
    const int col = 16 * (static_cast<int>(threadIdx.x) % LPR), slice = static_cast<int>(threadIdx.x) / LPR;
    const HeadInfo &hi = t.hi;
    import_class<DV, 8>(a, t, sperm, 0, hi.g8, hi.n16, hi.n8, slice, col);
    import_class<DV, 4>(a, t, sperm, hi.g8, hi.g4, hi.n16 + hi.n8, hi.n4, slice, col);
    import_class<DV, 2>(a, t, sperm, hi.g8 + hi.g4, hi.g2, hi.n16 + hi.n8 + hi.n4, hi.n2, slice, col);
}

// ---- FP16 rows out (zeros elsewhere) and in: 8 columns a thread

template <int DV>
__global__ __launch_bounds__(256) void export_pivots_kernel(TileArgs a)
{
    const TileRef t = tile_ref(a);
    constexpr int LPR = DV / 8, NS = 256 / LPR;
    const int col = 8 * (static_cast<int>(threadIdx.x) % LPR), slice = static_cast<int>(threadIdx.x) / LPR;
    const uint16_t *piv = reinterpret_cast<const uint16_t *>(t.rec + t.hi.piv_off);
    for (int p = slice; p < a.pool.dk; p += NS) {
        u32x4 v{0u, 0u, 0u, 0u};
        if (p < t.hi.n16) v = *reinterpret_cast<const u32x4 *>(piv + p * DV + col);
        *reinterpret_cast<u32x4_any2 *>(a.piv_out + (t.tdk + t.perm[p]) * DV + col) = v;
    }
}

template <int DV>
__global__ __launch_bounds__(256) void import_pivots_kernel(TileArgs a)
{
    const TileRef t = tile_ref(a);
    constexpr int LPR = DV / 8, NS = 256 / LPR;
    const int col = 8 * (static_cast<int>(threadIdx.x) % LPR), slice = static_cast<int>(threadIdx.x) / LPR;
    uint16_t *piv = reinterpret_cast<uint16_t *>(t.rec + t.hi.piv_off);
    for (int p = slice; p < t.hi.n16; p += NS)
        *reinterpret_cast<u32x4 *>(piv + p * DV + col) =
            *reinterpret_cast<const u32x4_any2 *>(a.piv_in + (t.tdk + t.perm[p]) * DV + col);
}

// ---- fp32 states in (quantize) and out (dequantize): 4 columns a thread

constexpr float kMagic = 0x1.8p+23f;     // 1.5 2^23: x + this has x rounded to an integer in its low bits
// Scales in here have reciprocals and products that stay normal: r c and
// 1 / (r c) lie within 2^-124 .. 2^124.
constexpr float kScaleLo = 0x1p-62f, kScaleHi = 0x1p+62f;

// A quotient this close to a half (0.5 - 2^-14 from its code) is divided again.
constexpr float kNearHalf = 0.49993896484375f;

// Codes of 4 columns of a row: round(x iq / (r c)) to +-q_b, as bytes, from the
// division's correctly rounded quotient.  Away from the halves any quotient
// close to it gives the same code: the reciprocals' product, within
// 3.5 2^-23 of 1 / (r c), and one residual step are within 2^-23 |y| <= 2^-16
// of the division's value where |y| <= q_b (the residual's own rounding
// below the normal range adds at most 2^-26).  Quotients near a half and
// scales outside the plain range take the division; infinite and NaN states
// come out as with it.
__device__ __forceinline__ uint32_t quantize4(f32x4_any x, float iq, float qb, float r, float ir, bool plain,
                                              const float (&c)[4], const float (&ic)[4])
{
    float y[4];
    bool divide = !plain;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float num = x[e] * iq, rc = r * c[e];
        const float inv = ir * ic[e];
        const float q0 = __builtin_amdgcn_fmed3f(num * inv, -256.0f, 256.0f);
        y[e] = fminf(fmaxf(fmaf(fmaf(-q0, rc, num), inv, q0), -qb), qb);
        divide = divide || fabsf(y[e] - ((y[e] + kMagic) - kMagic)) > kNearHalf;
    }
    if (divide) {
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = fminf(fmaxf((x[e] * iq) / (r * c[e]), -qb), qb);
    }
    uint32_t t[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] = __float_as_uint(y[e] + kMagic);
    // the low bytes
    return __builtin_amdgcn_perm(__builtin_amdgcn_perm(t[3], t[2], 0x0c0c0400u), __builtin_amdgcn_perm(t[1], t[0], 0x0c0c0400u),
                                 0x05040100u);
}

template <int DV, int B>
__device__ __forceinline__ void load_class(const TileArgs &a, const TileRef &t, const int *sperm, const float *sr,
                                           int g0, int groups, int p0, int rows, int slice, int cg, bool c_plain,
                                           const float (&c)[4], const float (&ic)[4])
{
    constexpr int NS = 1024 / DV, S = 8 / B, N = 4 / S > 1 ? 4 / S : 1;
    constexpr uint32_t field = 0x01010101u * ((1u << B) - 1u);
    constexpr float qb = static_cast<float>((1 << (B - 1)) - 1);
    const float iq = a.pool.lv.iq[B == 8 ? 0 : (B == 4 ? 1 : 2)];
    uint32_t *codes = reinterpret_cast<uint32_t *>(t.rec);
    each_batch<NS, N>(slice, groups, [&](int k0) {
        f32x4_any x[N][S];
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int xr = S * (k0 + NS * n) + s;
                x[n][s] = f32x4_any{0.f, 0.f, 0.f, 0.f};
                if (xr < rows)
                    x[n][s] = __builtin_nontemporal_load(
                        reinterpret_cast<const f32x4_any *>(a.state + (t.tdk + sperm[p0 + xr]) * DV + 4 * cg));
            }
#pragma unroll
        for (int n = 0; n < N; ++n) {
            if (k0 + NS * n >= groups) break;
            uint32_t w = 0u;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int xr = S * (k0 + NS * n) + s;
                if (xr < rows) {
                    const float r = sr[p0 + xr];
                    const bool plain = c_plain && r >= kScaleLo && r <= kScaleHi;
                    const uint32_t b = quantize4(x[n][s], iq, qb, r, __builtin_amdgcn_rcpf(r), plain, c, ic);
                    w |= (b & field) << (s * B);
                }
            }
            codes[(g0 + k0 + NS * n) * (DV / 4) + cg] = w;
        }
    });
}

template <int DV>
__global__ __launch_bounds__(256) void load_kernel(TileArgs a)
{
    __shared__ int sperm[kMaxDk];
    __shared__ float sr[kMaxDk];
    const TileRef t = tile_ref(a);
    constexpr int CG = DV / 4, NS = 256 / CG;
    const int cg = static_cast<int>(threadIdx.x) % CG, slice = static_cast<int>(threadIdx.x) / CG;
    const f32x4_any c4 = *reinterpret_cast<const f32x4_any *>(a.c_in + t.tdv + 4 * cg);
    take_scales<DV>(a, t, sperm, sr);
    const float c[4] = {c4[0], c4[1], c4[2], c4[3]};
    float ic[4];
    bool c_plain = true;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        ic[e] = __builtin_amdgcn_rcpf(c[e]);
        c_plain = c_plain && c[e] >= kScaleLo && c[e] <= kScaleHi;
    }
    __syncthreads();
    const HeadInfo &hi = t.hi;
    uint8_t *piv = t.rec + hi.piv_off;
    for (int p = slice; p < hi.n16; p += NS) {     // FP16 rows: binary16 values, nearest even
        const f32x4_any x = *reinterpret_cast<const f32x4_any *>(a.state + (t.tdk + sperm[p]) * DV + 4 * cg);
        *reinterpret_cast<u32x2 *>(piv + p * 2 * DV + 8 * cg) = u32x2{pack_halves(x[0], x[1]), pack_halves(x[2], x[3])};
    }
    load_class<DV, 8>(a, t, sperm, sr, 0, hi.g8, hi.n16, hi.n8, slice, cg, c_plain, c, ic);
    load_class<DV, 4>(a, t, sperm, sr, hi.g8, hi.g4, hi.n16 + hi.n8, hi.n4, slice, cg, c_plain, c, ic);
    load_class<DV, 2>(a, t, sperm, sr, hi.g8 + hi.g4, hi.g2, hi.n16 + hi.n8 + hi.n4, hi.n2, slice, cg, c_plain, c, ic);
}

// f / iq for an integer field, |f| <= 128, by the reciprocal and one residual
// step: the quotient's correctly rounded value for every field of every width
// and level normalisation (checked over all of them on the CPU).
__device__ __forceinline__ float level(float f, float iq, float nu)
{
    const float q = f * nu;
    return fmaf(fmaf(-q, iq, f), nu, q);
}

template <int DV, int B>
__device__ __forceinline__ void dequant_class(const TileArgs &a, const TileRef &t, const int *sperm, const float *sr,
                                              int g0, int p0, int rows, int slice, int cg, const float (&c)[4])
{
    constexpr int NS = 1024 / DV, S = 8 / B, N = 8 / S;
    const int wi = B == 8 ? 0 : (B == 4 ? 1 : 2);
    const float iq = a.pool.lv.iq[wi], nu = a.pool.lv.nu[wi];
    const uint32_t *codes = reinterpret_cast<const uint32_t *>(t.rec);
    each_batch<NS, N>(slice, (rows + S - 1) / S, [&](int k0) {
        uint32_t w[N];
#pragma unroll
        for (int n = 0; n < N; ++n)
            if (S * (k0 + NS * n) < rows) w[n] = codes[(g0 + k0 + NS * n) * (DV / 4) + cg];
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int xr = S * (k0 + NS * n) + s;
                if (xr < rows) {
                    const float r = sr[p0 + xr];
                    const uint32_t b = slot_top<B>(w[n], s);
                    f32x4_any v;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        v[e] = (r * c[e]) * level(sbyte(b, e) * (1.0f / static_cast<float>(1 << (8 - B))), iq, nu);
                    __builtin_nontemporal_store(
                        v, reinterpret_cast<f32x4_any *>(a.deq_out + (t.tdk + sperm[p0 + xr]) * DV + 4 * cg));
                }
            }
    });
}

template <int DV>
__global__ __launch_bounds__(256) void dequant_kernel(TileArgs a)
{
    __shared__ int sperm[kMaxDk];
    __shared__ float sr[kMaxDk];
    const TileRef t = tile_ref(a);
    constexpr int CG = DV / 4, NS = 256 / CG;
    const int tid = threadIdx.x, dk = a.pool.dk;
    const int cg = tid % CG, slice = tid / CG;
    const float *rr = reinterpret_cast<const float *>(t.rec + t.hi.r_off);
    if (tid < dk) {
        sperm[tid] = t.perm[tid];
        sr[tid] = rr[tid];
    }
    float c[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) c[e] = rr[dk + 4 * cg + e];
    __syncthreads();
    const HeadInfo &hi = t.hi;
    const uint8_t *piv = t.rec + hi.piv_off;
    for (int p = slice; p < hi.n16; p += NS) {
        const u32x2 h = *reinterpret_cast<const u32x2 *>(piv + p * 2 * DV + 8 * cg);
        *reinterpret_cast<f32x4_any *>(a.deq_out + (t.tdk + sperm[p]) * DV + 4 * cg) =
            f32x4_any{half_lo(h.x), half_hi(h.x), half_lo(h.y), half_hi(h.y)};
    }
    dequant_class<DV, 8>(a, t, sperm, sr, 0, hi.n16, hi.n8, slice, cg, c);
    dequant_class<DV, 4>(a, t, sperm, sr, hi.g8, hi.n16 + hi.n8, hi.n4, slice, cg, c);
    dequant_class<DV, 2>(a, t, sperm, sr, hi.g8 + hi.g4, hi.n16 + hi.n8 + hi.n4, hi.n2, slice, cg, c);
}

template <int DV>
void launch_op(const TileArgs &a, TileOp op, unsigned grid, hipStream_t s)
{
    switch (op) {
    case TileOp::Load: hipLaunchKernelGGL(load_kernel<DV>, dim3(grid), dim3(256), 0, s, a); break;
    case TileOp::Import: hipLaunchKernelGGL(import_kernel<DV>, dim3(grid), dim3(256), 0, s, a); break;
    case TileOp::Export: hipLaunchKernelGGL(export_kernel<DV>, dim3(grid), dim3(256), 0, s, a); break;
    case TileOp::Dequant: hipLaunchKernelGGL(dequant_kernel<DV>, dim3(grid), dim3(256), 0, s, a); break;
    case TileOp::ExportPivots: hipLaunchKernelGGL(export_pivots_kernel<DV>, dim3(grid), dim3(256), 0, s, a); break;
    case TileOp::ImportPivots: hipLaunchKernelGGL(import_pivots_kernel<DV>, dim3(grid), dim3(256), 0, s, a); break;
    }
}

}  // namespace

hipError_t launch_tile_op(const TileArgs &a, TileOp op, hipStream_t stream)
{
    const unsigned grid = static_cast<unsigned>(a.n) * static_cast<unsigned>(a.pool.Hv);
    if (grid == 0) return hipSuccess;
    if (a.pool.dv == 128) launch_op<128>(a, op, grid, stream);
    else launch_op<64>(a, op, grid, stream);
    return hipGetLastError();
}

}  // namespace stepq
