// MX family (App. A.3 "MX Formats"): main product in MXFP4 (E2M1 elements, blocks of 32 along K,
// E8M0 power-of-two scale) on v_mfma_scale_f32_32x32x64_f8f6f4 -- the hardware applies both block
// scales, so there is no vector-ALU dequantisation at all -- and the low-rank branch in FP8 E4M3
// with one fp32 scale per token / per row of L, R (Fig. 1, Eq. 5).
//
//   pack      : Q2(R), Q2(L) -> E4M3;  P = W - deq(Q2 L) deq(Q2 R) (fp64 chain, one rounding);
//               Q1(P) -> E2M1 + E8M0 per 32 values
//   act       : Q1(X) -> E2M1 + E8M0;  Q2(X) -> E4M3 (registers only);  T = (X8 . R8^T * sxb) * sr;
//               Q2(T) -> E4M3 + st
//   forward   : t = sum_blocks 2^(ex+ew) (x . p)  [scaled MFMA, fp32 accumulate];
//               y = t + (tq8 . l8^T * st) * sl;  Y = bf16_rne(y)
//
// Block scale exponent = (exponent field of the block amax) - 2, i.e. floor(log2 amax) - 2; elements
// are converted by v_cvt_scalef32_pk_fp4_f32 (nearest even, saturating at +-6) and
// v_cvt_pk_fp8_f32 or its scaled form (nearest even; they return NaN, not 448, above 464: inputs are
// clamped to +-448 first where they can lie there, but for X of the FP8 branch, see mx_act_kernel).
#include <type_traits>

#include "lq_pack.h"

namespace lq {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned short us2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------------------------
// shared device helpers
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ size_t mx_code_offset(int row, int k, int C64)  // dword holding code (row,k)
{
    const int blk = row >> 5, c = k >> 6, half = (k & 63) >> 5, d = (k & 31) >> 3;
    return ((size_t)((size_t)blk * C64 + c) * 64 + (row & 31) + 32 * half) * 16 + d * 4;
}
__device__ __forceinline__ size_t mx_scale_offset(int row, int c, int half, int CQ)  // byte of block (row, c, half)
{
    return ((size_t)((size_t)(row >> 5) * CQ + (c >> 2)) * 64 + (row & 31) + 32 * half) * 4 + (c & 3);
}
__device__ __forceinline__ size_t mx_rq_offset(int j, int k, int r)
{
    const int c = k >> 6, kq = (k & 63) >> 4;
    return ((size_t)((size_t)c * (r >> 4) + (j >> 4)) * 64 + (j & 15) + 16 * kq) * 16 + (k & 15);
}
__device__ __forceinline__ uint32_t e8m0_of(float amax)  // floor(log2 amax) - 2 + 127, clamped at 0
{
    const int e = (int)((__float_as_uint(amax) >> 23) & 0xFFu) - 2;
    return (amax == 0.0f || e < 0) ? 0u : (uint32_t)e;
}
__device__ __forceinline__ float e8m0_value(uint32_t E)  // 2^(E-127) as a float (E >= 1), 2^-127 for E = 0
{
    return E ? __uint_as_float(E << 23) : __uint_as_float(0x00400000u);
}
__device__ __forceinline__ uint32_t fp8_byte(float u)  // E4M3, nearest even, saturating
{
    u = fminf(fmaxf(u, -448.0f), 448.0f);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(u, u, 0, false) & 0xFFu;
}
__device__ __forceinline__ uint32_t fp8_pair(float u0, float u1)  // two E4M3 bytes in the low half
{
    u0 = fminf(fmaxf(u0, -448.0f), 448.0f);
    u1 = fminf(fmaxf(u1, -448.0f), 448.0f);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(u0, u1, 0, false) & 0xFFFFu;
}
// four E4M3 bytes from four in-range-or-not values: one median (saturation) and half a convert each
__device__ __forceinline__ uint32_t fp8_quad(float u0, float u1, float u2, float u3)
{
    u0 = __builtin_amdgcn_fmed3f(u0, -448.0f, 448.0f);
    u1 = __builtin_amdgcn_fmed3f(u1, -448.0f, 448.0f);
    u2 = __builtin_amdgcn_fmed3f(u2, -448.0f, 448.0f);
    u3 = __builtin_amdgcn_fmed3f(u3, -448.0f, 448.0f);
    const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(u0, u1, 0, false);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(u2, u3, lo, true);
}
__device__ __forceinline__ float fp8_value(uint32_t byte) { return __builtin_amdgcn_cvt_f32_fp8((int)byte, 0); }
__device__ __forceinline__ float fp8_value_of(uint32_t quad, int t)  // byte t (a constant)
{
    return t == 0   ? __builtin_amdgcn_cvt_f32_fp8((int)quad, 0)
           : t == 1 ? __builtin_amdgcn_cvt_f32_fp8((int)quad, 1)
           : t == 2 ? __builtin_amdgcn_cvt_f32_fp8((int)quad, 2)
                    : __builtin_amdgcn_cvt_f32_fp8((int)quad, 3);
}
__device__ __forceinline__ void fp8_scales(float amax, float* s, float* inv)
{
    if (amax == 0.0f) {
        *s = 1.0f;
        *inv = 1.0f;
    } else {
        *s = amax / 448.0f;
        *inv = 448.0f / amax;
    }
}
// ---- MXFP8e4 branch (block-scaled E4M3): operand layouts of the 8-bit scaled MFMA forms ----
__device__ __forceinline__ size_t mxb_frag8_offset(int row, int j, int rp)  // byte (row, rank index j) of lq / tq
{
    const int blk = row >> 5, cc = j >> 6, jj = j & 63;
    const int h = (jj & 31) >> 4, byte = (jj & 15) + ((jj >> 5) << 4);
    return ((size_t)((size_t)blk * (rp >> 6) + cc) * 64 + (row & 31) + 32 * h) * 32 + byte;
}
__device__ __forceinline__ size_t mxb_scale_offset(int row, int rb)  // scale byte (row, rank block rb) of le / te
{
    return ((size_t)(row >> 5) * 64 + (row & 31) + 32 * (rb & 1)) * 4 + (rb >> 1);
}
__device__ __forceinline__ size_t mxb_rq_offset(int j, int k, int r)  // byte (rank row j, k) of rq
{
    const int c = k >> 7, kk = k & 127;
    const int q = (kk & 63) >> 4, byte = (kk & 15) + ((kk >> 6) << 4);
    return ((size_t)((size_t)c * (r >> 4) + (j >> 4)) * 64 + (j & 15) + 16 * q) * 32 + byte;
}
__device__ __forceinline__ size_t mxb_re_offset(int j, int kb, int r)  // scale dword (rank row j, K block kb) of re
{
    return ((size_t)((size_t)(kb >> 2) * (r >> 4) + (j >> 4)) * 64 + (j & 15) + 16 * (kb & 3)) * 4;
}
__device__ __forceinline__ uint32_t e8m0_of_fp8(float amax)  // floor(log2 amax) - 8 + 127, clamped at 0
{
    const int e = (int)((__float_as_uint(amax) >> 23) & 0xFFu) - 8;
    return (amax == 0.0f || e < 0) ? 0u : (uint32_t)e;
}
__device__ __forceinline__ float e8m0_inverse(uint32_t E)  // 2^(127-E), exact (E <= 253)
{
    return __uint_as_float((254u - E) << 23);
}

// ---------------------------------------------------------------------------------------------
// pack
// ---------------------------------------------------------------------------------------------
// Q2 of a row of L or R: E4M3 with one fp32 scale
struct PackFp8Rows {
    __device__ void scale(float amax, float* s, float* inv) const { fp8_scales(amax, s, inv); }
    template <typename V>
    __device__ uint32_t quad(V v, float inv) const
    {
        return fp8_quad(__fmul_rn(v[0], inv), __fmul_rn(v[1], inv), __fmul_rn(v[2], inv), __fmul_rn(v[3], inv));
    }
    __device__ size_t r_offset(int j, int k, int r) const { return mx_rq_offset(j, k, r); }
};

// MXFP8e4 factors: one thread per (row, block of 32).  Rows of R, blocks along K, into the activation kernel's operand order;
// then rows of L, blocks along the rank, into the forward's.
// (Ks: row length of R's source; K: of the layout, a multiple of 128: blocks past the source are zero)
__global__ __launch_bounds__(256) void mxb_pack_rows_kernel(const float* L, const float* R, int N, int K, int Ks, int r, int rp,
                                                            uint8_t* lcodes, uint8_t* lscales, uint8_t* rcodes, uint8_t* rscales)
{
    size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t nr = (size_t)r * (K >> 5);
    const int mode = idx < nr ? 0 : 1;
    if (mode) idx -= nr;
    const int nb = mode ? r >> 5 : K >> 5, rows = mode ? N : r, src_len = mode ? r : Ks;
    if (idx >= (size_t)rows * nb) return;
    const float* A = mode ? L : R;
    uint8_t *codes = mode ? lcodes : rcodes, *scales = mode ? lscales : rscales;
    const int row = (int)(idx / nb), b = (int)(idx % nb);
    const bool in_src = 32 * b < src_len;
    const float* v = A + (size_t)row * src_len + 32 * b;
    float a = 0.f;
    if (in_src)
        for (int i = 0; i < 32; ++i) a = fmaxf(a, fabsf(v[i]));
    const uint32_t E = e8m0_of_fp8(a);
    const float inv = e8m0_inverse(E);
    for (int i = 0; i < 32; ++i) {
        const uint8_t c = in_src ? (uint8_t)fp8_byte(__fmul_rn(v[i], inv)) : (uint8_t)0;
        if (mode == 0)
            codes[mxb_rq_offset(row, 32 * b + i, r)] = c;
        else
            codes[mxb_frag8_offset(row, 32 * b + i, rp)] = c;
    }
    if (mode == 0)
        *(uint32_t*)(scales + mxb_re_offset(row, b, r)) = 0x7F7F7F00u | E;
    else
        scales[mxb_scale_offset(row, b)] = (uint8_t)E;
}

// Residual of a 64-chunk (two blocks of 32): MXFP4 codes and E8M0 bytes.  KIND of the factors: 0 as given, 1 E4M3 codes with
// fp32 row scales, 2 MXFP8e4 and 3 MXFP6e2 codes with E8M0 block scales (sl, sr hold le, re; element * 2^e is exact in fp32).
struct PackMxBlock4 {  // four codes and their block's scale byte
    uint32_t c, e;
};
typedef uint32_t u32_bytes __attribute__((aligned(1)));
// Four E2M3 codes of 24 bits (what is above is not looked at) as the E4M3 bytes of their values * 2^-6 (normal and subnormal alike)
__device__ __forceinline__ uint32_t e4m3_of_fp6(uint32_t c)
{
    const uint32_t h = (c & 0xFFFu) | (c << 4 & ~0xFFFu);                   // two codes to a half
    const uint32_t b = (h & 0x003F003Fu) | (h << 2 & ~0x003F003Fu);         // a code to a byte, bits 6 and 7 of no meaning
    return (b & 0x1F1F1F1Fu) | (b << 2 & 0x80808080u);
}
// Four E4M3 codes times 2^(E - 127), E <= 254 their block's scale byte: the converter multiplies by any such power, 2^-127 among them (checked
// against ldexp over all codes and scales; subnormal results are exact).  Codes of E2M3 give their values times 2^-6.  (With an ldexp per
// value, and ten instructions to spread the 6-bit codes, every wavefront's decoding of R cost more than reading it decoded from the LDS had: us a pack
// call, staged / ldexp / this: MXFP6 4608 x 1152 rank 32 21.5 / 22.5 / 20.8, 6720 x 2240 rank 96 92.0 / 99.2 / 78.5, MXFP8 8192 x 9216 rank 32 129 / 138 / 122.)
__device__ __forceinline__ void fp8_block_quad(uint32_t c, uint32_t E, float (&v)[4])
{
    const float s = __uint_as_float(E << 23);
    const auto lo = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c, s, false), hi = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c, s, true);
    v[0] = lo[0], v[1] = lo[1], v[2] = hi[0], v[3] = hi[1];
}
template <int KIND>
struct PackMxResidual {
    using Raw = std::conditional_t<KIND == 0, pack_v4f, std::conditional_t<KIND == 1, PackCodes4, PackMxBlock4>>;
    const float *L, *R;
    const uint8_t* l8;
    const float* sl;
    const uint8_t* r8;
    const float* sr;
    uint8_t *pc, *pe;
    int Ks, C64, r, rp;
    __device__ void lhat(int n, int j, int q, float (&v)[4]) const
    {
        if constexpr (KIND == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = L[(size_t)n * r + j + 4 * i + q];
        } else if constexpr (KIND <= 2) {
            const uint4 c = *(const uint4*)(l8 + (KIND == 1 ? (size_t)n * rp + j : mxb_frag8_offset(n, j, rp)));
            const uint32_t d[4] = {c.x, c.y, c.z, c.w};
            const float s = KIND == 1 ? sl[n] : e8m0_value(((const uint8_t*)sl)[mxb_scale_offset(n, j >> 5)]);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = __fmul_rn(fp8_value(d[i] >> (8 * q) & 0xFFu), s);
        } else {  // 16 codes in 96 bits, four in 24
            const uint32_t* p = (const uint32_t*)(l8 + mx6_lt_slot(n, j >> 5, rp) + 12 * ((j & 31) >> 4));
            const uint32_t w0 = p[0], w1 = p[1], w2 = p[2];
            const uint32_t d[4] = {w0, w0 >> 24 | w1 << 8, w1 >> 16 | w2 << 16, w2 >> 8};
            uint32_t c = 0u;  // the lane's four, in 24 bits
#pragma unroll
            for (int i = 0; i < 4; ++i) c |= (d[i] >> (6 * q) & 63u) << (6 * i);
            fp8_block_quad(e4m3_of_fp6(c), ((const uint8_t*)sl)[mxb_scale_offset(n, j >> 5)], v);
        }
    }
    __device__ Raw rload(int j, int k) const
    {
        if constexpr (KIND == 0) return *(const Raw*)(R + (size_t)j * Ks + k);
        else if constexpr (KIND == 1) return Raw{*(const uint32_t*)(r8 + mx_rq_offset(j, k, r)), sr[j]};
        else {
            const uint32_t E = ((const uint8_t*)sr)[mxb_re_offset(j, k >> 5, r)];
            if constexpr (KIND == 2) return Raw{*(const uint32_t*)(r8 + mxb_rq_offset(j, k, r)), E};
            else return Raw{*(const u32_bytes*)(r8 + mx6_rq_slot(j, k >> 5, r) + 3 * ((k & 31) >> 2)), E};  // (24 bits of the slot's 192)
        }
    }
    static constexpr double UNIT = KIND == 3 ? 4096.0 : 1.0;
    static constexpr bool PAD_CHECK = true;
    __device__ void rval(const Raw& x, float (&v)[4]) const
    {
        if constexpr (KIND >= 2) {
            fp8_block_quad(KIND == 3 ? e4m3_of_fp6(x.c) : x.c, x.e, v);
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if constexpr (KIND == 0) v[t] = x[t];
                else v[t] = __fmul_rn(fp8_value_of(x.c, t), x.s);
            }
        }
    }
    __device__ void encode(int n, int c, const float (&P)[1][16], int q) const
    {
        float a = pack_amax(P[0]);
        a = fmaxf(a, __shfl_xor(a, 16));  // lanes q, q ^ 1 hold the block
        const uint32_t E = e8m0_of(a);
        const float s = e8m0_value(E);
        uint32_t w[2] = {0u, 0u};
        if (a != 0.0f) {
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                w[d] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w[d], P[0][8 * d], P[0][8 * d + 1], s, 0);
                w[d] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w[d], P[0][8 * d + 2], P[0][8 * d + 3], s, 1);
                w[d] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w[d], P[0][8 * d + 4], P[0][8 * d + 5], s, 2);
                w[d] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w[d], P[0][8 * d + 6], P[0][8 * d + 7], s, 3);
            }
        }
        typedef uint32_t u2 __attribute__((ext_vector_type(2)));
        *(u2*)(pc + mx_code_offset(n, c * 64 + 16 * q, C64)) = u2{w[0], w[1]};
        if ((q & 1) == 0) pe[mx_scale_offset(n, c, q >> 1, (C64 + 3) >> 2)] = (uint8_t)E;
    }
};

hipError_t launch_pack_mx(const Dims& d, int from_q, const float* W, const float* L, const float* R, uint8_t* packed,
                          hipStream_t s)
{
    const PackedLayout pl = packed_layout(d);
    uint8_t* l8 = packed + pl.off_lq;
    float* sl = (float*)(packed + pl.off_sl);
    uint8_t* r8 = packed + pl.off_rq;
    float* sr = (float*)(packed + pl.off_sr);
    const int N = (int)d.N, K = (int)d.K, Ks = (int)d.Ks;
    uint8_t *pc = packed + pl.off_pq, *pe = packed + pl.off_sw;
    PackFill fill;
    fill.n = 0;
    if (d.C64 % 4) fill.add(pe, (size_t)(N / 32) * ((d.C64 + 3) / 4) * 256, 0x7F7F7F7Fu);  // padding chunks of the last quad: 2^0
    if (d.smooth) fill.add(packed + pl.off_rg, (size_t)K * 4, 0x3F800000u);                 // reciprocals start at 1
    if (d.mxb) {  // padding of the rank to 64: zero codes, scale 2^0
        if (d.rp != d.r) fill.add(l8, (size_t)N * d.rp, 0u);
        fill.add(sl, (size_t)N * 8, 0x7F7F7F7Fu);
    }
    hipError_t e = launch_pack_fill(fill, s);
    if (e != hipSuccess) return e;
    if (!d.mxb) {
        pack_row_factors(PackFp8Rows{}, L, R, N, Ks, K, d.r, d.rp, l8, sl, r8, sr, s);
    } else if (d.r > 0 && d.mxb_elem == 6) {
        e = launch_pack_rows_mx6(d, L, R, packed, s);
        if (e != hipSuccess) return e;
    } else if (d.r > 0) {
        const size_t nt = (size_t)d.r * (K / 32) + (size_t)N * (d.r / 32);
        hipLaunchKernelGGL(mxb_pack_rows_kernel, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, s, L, R, N, K, Ks, d.r, d.rp, l8, (uint8_t*)sl,
                           r8, (uint8_t*)sr);
    }
    e = hipGetLastError();
    auto residual = [&](auto kind) {
        return pack_residual<1>(e, PackMxResidual<decltype(kind)::value>{L, R, l8, sl, r8, sr, pc, pe, Ks, d.C64, d.r, d.rp}, W, N, Ks, d.r, d.C64, packed,
                                make_tag(d, LQ_BLOB_PACKED, 0), s);
    };
    if (!from_q || d.r == 0) return residual(std::integral_constant<int, 0>{});
    if (!d.mxb) return residual(std::integral_constant<int, 1>{});
    if (d.mxb_elem == 8) return residual(std::integral_constant<int, 2>{});
    return residual(std::integral_constant<int, 3>{});
}

// ---------------------------------------------------------------------------------------------
// plain views
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void mx_unpack_w_kernel(const uint8_t* packed, PackedLayout pl, int N, int K, int C64, int r,
                                                          int rp, int mxb, lq_weights_view out)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int CQ = (C64 + 3) >> 2, B = K >> 5;  // K: the caller's (views); C64: chunks of the layout
    if (idx < (size_t)N * K && out.pq) {
        const int n = (int)(idx / K), k = (int)(idx % K);
        const uint32_t w = *(const uint32_t*)(packed + pl.off_pq + mx_code_offset(n, k, C64));
        out.pq[idx] = (int8_t)((w >> (4 * (k & 7))) & 0xFu);
    }
    if (idx < (size_t)N * B && out.pe) {
        const int n = (int)(idx / B), b = (int)(idx % B);
        out.pe[idx] = packed[pl.off_sw + mx_scale_offset(n, b >> 1, b & 1, CQ)];
    }
    if (idx < (size_t)N * r && out.lq) {
        const int n = (int)(idx / r), j = (int)(idx % r);
        out.lq[idx] = (int8_t)packed[pl.off_lq + (mxb ? mxb_frag8_offset(n, j, rp) : (size_t)n * rp + j)];
    }
    if (idx < (size_t)r * K && out.rq) {
        const int j = (int)(idx / K), k = (int)(idx % K);
        out.rq[idx] = (int8_t)packed[pl.off_rq + (mxb ? mxb_rq_offset(j, k, r) : mx_rq_offset(j, k, r))];
    }
    if (mxb) {
        if (idx < (size_t)N * (r >> 5) && out.le) {
            const int n = (int)(idx / (r >> 5)), b = (int)(idx % (r >> 5));
            out.le[idx] = packed[pl.off_sl + mxb_scale_offset(n, b)];
        }
        if (idx < (size_t)r * B && out.re) {
            const int j = (int)(idx / B), b = (int)(idx % B);
            out.re[idx] = packed[pl.off_sr + mxb_re_offset(j, b, r)];
        }
    } else {
        if (idx < (size_t)N && out.sl) out.sl[idx] = ((const float*)(packed + pl.off_sl))[idx];
        if (idx < (size_t)r && out.sr) out.sr[idx] = ((const float*)(packed + pl.off_sr))[idx];
    }
}

hipError_t launch_unpack_weights_mx(const Dims& d, const uint8_t* packed, const lq_weights_view* out, hipStream_t s)
{
    if (d.mxb_elem == 6) return launch_unpack_weights_mx6(d, packed, out, s);
    const PackedLayout pl = packed_layout(d);
    const size_t n = (size_t)(d.N > d.r ? d.N : d.r) * (d.Ks > d.r ? d.Ks : d.r);  // covers N x K, r x K and N x r
    hipLaunchKernelGGL(mx_unpack_w_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, packed, pl, (int)d.N,
                       (int)d.Ks, d.C64, d.r, d.rp, d.mxb ? 1 : 0, *out);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void mx_unpack_a_kernel(const uint8_t* act, ActLayout al, int M, int K, int C64, int r, int rp,
                                                          int mxb, lq_act_view out)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int CQ = (C64 + 3) >> 2, B = K >> 5;
    if (idx < (size_t)M * K && out.xq) {
        const int m = (int)(idx / K), k = (int)(idx % K);
        const uint32_t w = *(const uint32_t*)(act + al.off_xq + mx_code_offset(m, k, C64));
        out.xq[idx] = (int8_t)((w >> (4 * (k & 7))) & 0xFu);
    }
    if (idx < (size_t)M * B && out.xe) {
        const int m = (int)(idx / B), b = (int)(idx % B);
        out.xe[idx] = act[al.off_sx + mx_scale_offset(m, b >> 1, b & 1, CQ)];
    }
    if (idx < (size_t)M && out.st && !mxb) out.st[idx] = ((const float*)(act + al.off_st))[idx];
    if (idx < (size_t)M * r && out.tq) {
        const int m = (int)(idx / r), j = (int)(idx % r);
        out.tq[idx] = (int8_t)act[al.off_tq + (mxb ? mxb_frag8_offset(m, j, rp) : (size_t)m * rp + j)];
    }
    if (mxb && idx < (size_t)M * (r >> 5) && out.te) {
        const int m = (int)(idx / (r >> 5)), b = (int)(idx % (r >> 5));
        out.te[idx] = act[al.off_st + mxb_scale_offset(m, b)];
    }
}

hipError_t launch_unpack_act_mx(const Dims& d, const uint8_t* act, int64_t M, const lq_act_view* out, hipStream_t s)
{
    if (d.mxb_elem == 6) return launch_unpack_act_mx6(d, act, M, out, s);
    const ActLayout al = act_layout(d, M);
    const size_t n = (size_t)M * (d.Ks > d.r ? d.Ks : d.r);
    hipLaunchKernelGGL(mx_unpack_a_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, act, al, (int)M,
                       (int)d.Ks, d.C64, d.r, d.rp, d.mxb ? 1 : 0, *out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// activation kernel: same decomposition as the INT one (16 token rows per workgroup, lane =
// (row l%16, 16-value quarter l/16 of each 64-chunk), chunks dealt round-robin to 4 or 8 wavefronts).
// Bound: X's bytes, then, all workgroups in step, coding and the way to the re-quantised intermediate.  us a call, four wavefronts, one of them
// re-quantising, and a clamp per value / this: 300 x 1152 rank 32 6.8 / 5.8, rank 128 7.9 / 6.5, 8192 x 4608 rank 128 42.3 / 36.4, smoothed 1000 x 4608
// rank 64 28.4 / 14.6, 6001 x 2240 rank 64 21.6 / 16.5.
// ---------------------------------------------------------------------------------------------
struct MxActParams {
    const void* X;
    int64_t ldx;
    int M, K, C64, C64s, CQ, r, rp;  // K, C64s: the caller's row length and its 64-chunks; C64: chunks of the layout
    const uint8_t* r8;
    const float* sr;
    uint8_t* xc;
    uint8_t* xe;
    uint8_t* tq8;
    float* st;
    int8_t* dbg_xb;
    float* dbg_sxb;
    float* dbg_T;
    const float* rg;  // reciprocals of the smoothing vector (smoothing variant only)
    BlobTag tag;        // header of the activation blob (written by the first workgroup)
    uint32_t* tag_dst;
};

template <bool BF16>
struct MxChunk;
template <>
struct MxChunk<true> {
    uint32_t w[8];
    __device__ __forceinline__ void load(const void* X, size_t elem, bool ok)
    {
        v4i a = {0, 0, 0, 0}, b = {0, 0, 0, 0};
        if (ok) {
            const v4i* p = (const v4i*)((const uint16_t*)X + elem);
            a = p[0];
            b = p[1];
        }
        w[0] = a[0]; w[1] = a[1]; w[2] = a[2]; w[3] = a[3];
        w[4] = b[0]; w[5] = b[1]; w[6] = b[2]; w[7] = b[3];
    }
    __device__ __forceinline__ float get(int i) const
    {
        return __uint_as_float((i & 1) ? (w[i >> 1] & 0xFFFF0000u) : (w[i >> 1] << 16));
    }
};
template <>
struct MxChunk<false> {
    float v[16];
    __device__ __forceinline__ void load(const void* X, size_t elem, bool ok)
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v4i a = {0, 0, 0, 0};
            if (ok) a = ((const v4i*)((const float*)X + elem))[q];
            v[4 * q] = __int_as_float(a[0]);
            v[4 * q + 1] = __int_as_float(a[1]);
            v[4 * q + 2] = __int_as_float(a[2]);
            v[4 * q + 3] = __int_as_float(a[3]);
        }
    }
    __device__ __forceinline__ float get(int i) const { return v[i]; }
};

// 16 values of a block and the block's scale -> 16 E4M3 bytes, nearest even, saturating at +-448 * 2^(E - 127): the scaled converters, from
// bf16 pairs with both magnitudes limited first (they return NaN past the range), without unpacking a value.
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void mxfp8_codes16(const MxChunk<true>& ch, uint32_t E, uint32_t* out)
{
    const uint32_t l1 = ((E + 8u) << 7) | 0x60u, lim = l1 | (l1 << 16);
    const float sc = e8m0_value(E);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        typedef short v2s __attribute__((ext_vector_type(2)));
        v2s r = {0, 0};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t w = ch.w[2 * g + h];
            const uint32_t m = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(us2, w & 0x7FFF7FFFu), __builtin_bit_cast(us2, lim)));
            const v2bf v = __builtin_bit_cast(v2bf, (w & 0x80008000u) | m);
            r = h ? __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(r, v, sc, true) : __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(r, v, sc, false);
        }
        out[g] = __builtin_bit_cast(uint32_t, r);
    }
}
__device__ __forceinline__ void mxfp8_codes16(const MxChunk<false>& ch, uint32_t E, uint32_t* out)
{
    const float inv = e8m0_inverse(E);
#pragma unroll
    for (int g = 0; g < 4; ++g)
        out[g] = fp8_quad(__fmul_rn(ch.get(4 * g), inv), __fmul_rn(ch.get(4 * g + 1), inv), __fmul_rn(ch.get(4 * g + 2), inv), __fmul_rn(ch.get(4 * g + 3), inv));
}
__device__ __forceinline__ void mxfp4_codes16(const MxChunk<true>& ch, float sc, uint32_t (&pk)[2])
{
#define LQ_CVT4(J) pk[(J) >> 2] = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(pk[(J) >> 2], __builtin_bit_cast(v2bf, ch.w[J]), sc, (J) & 3)
    LQ_CVT4(0); LQ_CVT4(1); LQ_CVT4(2); LQ_CVT4(3); LQ_CVT4(4); LQ_CVT4(5); LQ_CVT4(6); LQ_CVT4(7);
#undef LQ_CVT4
}
__device__ __forceinline__ void mxfp4_codes16(const MxChunk<false>& ch, float sc, uint32_t (&pk)[2])
{
#define LQ_CVT4(J) pk[(J) >> 2] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(pk[(J) >> 2], ch.get(2 * (J)), ch.get(2 * (J) + 1), sc, (J) & 3)
    LQ_CVT4(0); LQ_CVT4(1); LQ_CVT4(2); LQ_CVT4(3); LQ_CVT4(4); LQ_CVT4(5); LQ_CVT4(6); LQ_CVT4(7);
#undef LQ_CVT4
}
__device__ __forceinline__ float mx_amax16(const MxChunk<true>& ch)  // |bf16| is monotonic in its low 15 bits: packed unsigned maximum, two values per instruction
{
    us2 m2 = {0, 0};
#pragma unroll
    for (int d = 0; d < 8; ++d) m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(us2, ch.w[d] & 0x7FFF7FFFu));
    const uint32_t mm = m2[0] > m2[1] ? m2[0] : m2[1];
    return __uint_as_float(mm << 16);
}
__device__ __forceinline__ float mx_amax16(const MxChunk<false>& ch)
{
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) m = fmaxf(m, fabsf(ch.get(i)));
    return m;
}

// Wavefronts a SIMD is to hold.  Asked for one, the compiler keeps the eight sums of T beside the row's registers, and fewer workgroups fit than with four sums (us,
// one / two: fp32 8447 x 128 rank 64 7.4 / 6.1, 12327 x 1280 20.8 / 18.9, smoothed 16384 x 1600 rank 128 37.9 / 28.8).  Four wavefronts at rank 128 spill for two
// or are no faster (fp32 6125 x 1600 19.3 / 22.6, smoothed 6125 x 1280 11.6 / 12.1), but for smoothed rows of nine chunks and streamed ones.
constexpr int mx_act_waves(int maxc, int njb, bool sm, int nw)
{
    if (nw == 4 && njb == 8) return maxc == 0 || (maxc == 9 && sm) ? 2 : 1;
    return nw == 4 && maxc == 5 && njb == 1 ? 4 : 2;
}

// BF16IN: element type of X; SM: smoothing variant (X times the stored reciprocals, held as fp32).
template <bool BF16IN, int MAXC, int NJB, bool SM, int NW>
__global__ __launch_bounds__(64 * NW, mx_act_waves(MAXC, NJB, SM, NW)) void mx_act_kernel(MxActParams p)
{
    write_tag(p.tag_dst, p.tag);
    constexpr bool BF16 = BF16IN && !SM;  // representation of the row in registers
    constexpr int NJA = NJB > 0 ? NJB : 1;
    constexpr int NSUM = 8, SW = NSUM / NW;  // T is eight sums, over the chunks c = 0 .. 7 mod 8, added in order; SW of them to a wavefront
    __shared__ float s_amax[NW][16];
    __shared__ float s_sxb[16];
    __shared__ float s_acc[NSUM][NJA][64][4];
    __shared__ float s_tmax[NW][16];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, kq = lane >> 4;
    const int row = blockIdx.x * 16 + r16;
    const bool row_ok = row < p.M;
    const uint32_t rowmask = row_ok ? ~0u : 0u;
    const int C64 = p.C64;

    // MAXC = 0: rows too long for the registers are streamed twice through a two-chunk ring (amax pass, coding pass;
    // the second read comes from the caches)
    constexpr bool STREAM = MAXC == 0;
    constexpr int NS = STREAM ? 2 : MAXC;        // chunk slots in registers
    const int nmy = (C64 - wave + NW - 1) / NW;  // chunks of this wavefront: c = wave + NW * ci, ci < nmy
    MxChunk<BF16> xc[NS];
    const size_t xrow = (size_t)(row_ok ? row : p.M - 1) * p.ldx + kq * 16;
    // (in the ring no branch stands around the loads, which would end the compiler's count of those in flight: past the end they are clamped,
    // and masked where they are used)
    auto load_x = [&](MxChunk<BF16>& ch, int ci) {
        int c = wave + NW * ci;
        const bool ok = STREAM || c < p.C64s;  // wave-uniform
        c = c < p.C64s ? c : p.C64s - 1;
        if (!ok) ch = MxChunk<BF16>{};
        else if constexpr (SM)
            smooth_load<BF16IN, 16>(ch.v, p.X, xrow + (size_t)c * 64, p.rg + (size_t)c * 64 + kq * 16, true);
        else
            ch.load(p.X, xrow + (size_t)c * 64, true);
    };
    auto keep_of = [&](int ci, uint32_t m) { return wave + NW * ci < p.C64s ? m : 0u; };  // (rows past M and chunks past the row: zeros)
#pragma unroll
    for (int ci = 0; ci < NS; ++ci) load_x(xc[ci], ci);

    // Operands that do not depend on X are requested now (their latency overlaps the load of X):
    // the Q2(R) fragments of the first chunk (later ones one chunk ahead, in the loop), R's scales.
    v4i bvs[2][NJA];
    auto load_r8 = [&](v4i (&dst)[NJA], int ci) {
        int c = wave + NW * ci;
        c = c < C64 ? c : C64 - 1;  // clamped: a fragment past the end is fetched but not used
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) dst[jb] = *(const v4i*)(p.r8 + ((size_t)((size_t)c * NJB + jb) * 64 + lane) * 16);
    };
    load_r8(bvs[0], 0);
    constexpr int PW = NJB <= 2 ? 1 : NW;        // wavefronts that re-quantise the intermediate
    constexpr int NT = (NJA + PW - 1) / PW;      // 16-column groups each of them takes
    float srj[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) srj[t] = NJB > 0 ? p.sr[(wave + PW * t < NJB ? wave + PW * t : 0) * 16 + r16] : 0.f;

    // amax of the lane's 16 values per chunk (kept for the block scale when the row is resident) and of the whole row
    float a16[NS];
    float a = 0.f;
    auto amax_chunk = [&](const MxChunk<BF16>& ch, int ci) { return __uint_as_float(__float_as_uint(mx_amax16(ch)) & keep_of(ci, rowmask)); };
    if constexpr (STREAM) {
        for (int ci0 = 0; ci0 < nmy; ci0 += 2) {
#pragma unroll
            for (int sl = 0; sl < 2; ++sl) {
                a = fmaxf(a, amax_chunk(xc[sl], ci0 + sl));
                load_x(xc[sl], ci0 + sl + 2);
            }
        }
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) load_x(xc[sl], sl);  // second pass: the ring starts over
    } else {
#pragma unroll
        for (int ci = 0; ci < NS; ++ci) {
            a16[ci] = amax_chunk(xc[ci], ci);
            a = fmaxf(a, a16[ci]);
        }
    }
    a = max_xor16(a);
    a = max_xor32(a);
    if (kq == 0) s_amax[wave][r16] = a;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) a = fmaxf(a, s_amax[w][r16]);
    // Codes of the branch are fl(x * 448 / a) through the scaled converter with scale 1: at most 448 (1 + 2^-23) in magnitude, which its rounding saturates.  Below
    // 448 / FLT_MAX the factor is not finite and every value but zero saturates: 2^127 and a scale of 2^-40 take the smallest number past the range, where the
    // converter returns NaN (0x7F and the sign), which is 448 without its last bit.
    float invb = a == 0.0f ? 1.0f : 448.0f / a;
    const bool tiny = invb > 3.402823466e38f;
    const float cscale = tiny ? 0x1p-40f : 1.0f;
    const uint32_t codemask = tiny ? rowmask & 0xFEFEFEFEu : rowmask;
    invb = tiny ? 0x1p127f : invb;
    if (wave == NW - 1 && kq == 0) {  // (the scale itself: by the wavefront with the fewest chunks)
        const float sb = a == 0.0f ? 1.0f : a / 448.0f;
        s_sxb[r16] = sb;
        if (p.dbg_sxb && row_ok) p.dbg_sxb[row] = sb;
        if (NJB == 0) p.st[row] = 1.0f;
    }

    v4f acc[SW][NJA];
#pragma unroll
    for (int i = 0; i < SW; ++i)
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) acc[i][jb] = v4f{0.f, 0.f, 0.f, 0.f};

    // one 64-chunk: MXFP4 codes and block scales, FP8 branch codes, skinny contraction (am: amax of the lane's 16 values; odd: ci & 1)
    auto code_chunk = [&](const MxChunk<BF16>& ch, const int c, const uint32_t keep, const float am, auto odd) {
        // MXFP4: block of 32 = this lane's 16 values and its neighbour's (kq ^ 1)
        const float ab = max_xor16(am);
        const uint32_t E = e8m0_of(ab);
        const uint32_t nz = ab != 0.0f ? ~0u : 0u;  // (a block of zeros has codes 0, also where the zeros are negative)
        uint32_t pk[2] = {0u, 0u};
        mxfp4_codes16(ch, e8m0_value(E), pk);
        uint32_t x8[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            typedef short v2s __attribute__((ext_vector_type(2)));
            v2s c2 = {0, 0};
            c2 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(c2, __fmul_rn(ch.get(4 * q), invb), __fmul_rn(ch.get(4 * q + 1), invb), cscale, false);
            c2 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(c2, __fmul_rn(ch.get(4 * q + 2), invb), __fmul_rn(ch.get(4 * q + 3), invb), cscale, true);
            x8[q] = keep & __builtin_bit_cast(uint32_t, c2);
        }
        uint8_t* dst = p.xc + ((size_t)((size_t)(row >> 5) * C64 + c) * 64 + (row & 31) + 32 * (kq >> 1)) * 16 + (kq & 1) * 8;
        *(uint2*)dst = make_uint2(pk[0] & nz, pk[1] & nz);
        if ((kq & 1) == 0) p.xe[mx_scale_offset(row, c, kq >> 1, p.CQ)] = (uint8_t)E;
        if (p.dbg_xb && row_ok && c < p.C64s)
            *(v4i*)(p.dbg_xb + (size_t)row * p.K + c * 64 + kq * 16) = v4i{(int)x8[0], (int)x8[1], (int)x8[2], (int)x8[3]};
        if (NJB > 0) {
            constexpr int par = decltype(odd)::value, set = par % SW;
            const long alo = (long)(((unsigned long)x8[1] << 32) | x8[0]);
            const long ahi = (long)(((unsigned long)x8[3] << 32) | x8[2]);
#pragma unroll
            for (int jb = 0; jb < NJB; ++jb) {
                const v4i bv = bvs[par][jb];
                const long blo = (long)(((unsigned long)(uint32_t)bv[1] << 32) | (uint32_t)bv[0]);
                const long bhi = (long)(((unsigned long)(uint32_t)bv[3] << 32) | (uint32_t)bv[2]);
                acc[set][jb] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(alo, blo, acc[set][jb], 0, 0, 0);
                acc[set][jb] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(ahi, bhi, acc[set][jb], 0, 0, 0);
            }
        }
    };
    auto pad_chunk = [&](const int c) {  // padding chunk of the last quad: its scale bytes must be valid E8M0 values (2^0)
        if (c >= C64 && c < 4 * p.CQ && (kq & 1) == 0) p.xe[mx_scale_offset(row, c, kq >> 1, p.CQ)] = (uint8_t)127;
    };
    auto pair = [&](auto f) {  // f(0), f(1) with the argument as a compile-time constant
        f(std::integral_constant<int, 0>{});
        f(std::integral_constant<int, 1>{});
    };
    if constexpr (STREAM) {
        for (int ci0 = 0; ci0 < nmy; ci0 += 2) {
            pair([&](auto sl) {
                const int ci = ci0 + decltype(sl)::value, c = wave + NW * ci;
                load_r8(bvs[(decltype(sl)::value + 1) & 1], ci + 1);
                MxChunk<BF16>& x = xc[decltype(sl)::value];
                if (c < C64) code_chunk(x, c, keep_of(ci, codemask), amax_chunk(x, ci), sl);  // wave-uniform
                load_x(x, ci + 2);
            });
        }
        pad_chunk(wave + NW * nmy);
    } else {
#pragma unroll
        for (int ci0 = 0; ci0 < NS; ci0 += 2) {
            pair([&](auto sl) {
                constexpr int par = decltype(sl)::value;
                const int ci = ci0 + par, c = wave + NW * ci;
                if (ci >= NS) return;
                if (ci + 1 < NS) load_r8(bvs[par ^ 1], ci + 1);
                if (c < C64) code_chunk(xc[ci], c, keep_of(ci, codemask), a16[ci], sl);  // wave-uniform
                else pad_chunk(c);
            });
        }
    }
    if (NJB == 0) return;

    // ---- the eight sums, dequantised and re-quantised per token.  Up to two 16-column groups: the first wavefront; more: wavefront w takes the
    // groups w, w + NW, and the row maxima meet in LDS
#pragma unroll
    for (int i = 0; i < SW; ++i)
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) *(v4f*)&s_acc[wave + NW * i][jb][lane][0] = acc[i][jb];
    __syncthreads();
    if (wave >= PW) return;

    float T[NT][4];
    float tmax[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int jb = wave + PW * t;
        if (jb >= NJB) break;  // wave-uniform
        v4f s = *(const v4f*)&s_acc[0][jb][lane][0];
#pragma unroll
        for (int w = 1; w < NSUM; ++w) {
            const v4f o = *(const v4f*)&s_acc[w][jb][lane][0];
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = __fadd_rn(s[i], o[i]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int tok = 4 * kq + i;
            const float tv = __fmul_rn(__fmul_rn(s[i], s_sxb[tok]), srj[t]);
            T[t][i] = tv;
            tmax[i] = fmaxf(tmax[i], fabsf(tv));
            const int grow = blockIdx.x * 16 + tok;
            if (grow < p.M && p.dbg_T) p.dbg_T[(size_t)grow * p.r + jb * 16 + r16] = tv;
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        tmax[i] = max_row16(tmax[i]);
    }
    if constexpr (PW > 1) {
        if (r16 == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) s_tmax[wave][4 * kq + i] = tmax[i];
        }
        __syncthreads();  // (every wavefront: PW = NW)
#pragma unroll
        for (int w = 0; w < PW; ++w)
#pragma unroll
            for (int i = 0; i < 4; ++i) tmax[i] = fmaxf(tmax[i], s_tmax[w][4 * kq + i]);
    }
    // (a row's maximum is in 16 lanes: lane i & 3 divides for row i and hands both factors to the others)
    float sv, iv;
    fp8_scales(r16 & 2 ? (r16 & 1 ? tmax[3] : tmax[2]) : (r16 & 1 ? tmax[1] : tmax[0]), &sv, &iv);
    const float st4[4] = {row16_lane<0>(sv), row16_lane<1>(sv), row16_lane<2>(sv), row16_lane<3>(sv)};
    const float inv4t[4] = {row16_lane<0>(iv), row16_lane<1>(iv), row16_lane<2>(iv), row16_lane<3>(iv)};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int grow = blockIdx.x * 16 + 4 * kq + i;
        const float stv = st4[i], invt = inv4t[i];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int jb = wave + PW * t;
            if (jb >= NJB) break;
            p.tq8[(size_t)grow * p.rp + jb * 16 + r16] = (uint8_t)fp8_byte(__fmul_rn(T[t][i], invt));
        }
        if (wave == 0) {
            if (r16 == 0) p.st[grow] = stv;
            for (int j = p.r + r16; j < p.rp; j += 16) p.tq8[(size_t)grow * p.rp + j] = 0;
        }
    }
}

template <bool BF16, int MAXC, int NJB, bool SM, int NW>
static hipError_t mx_act_launch(const MxActParams& p, int64_t Mp, hipStream_t s)
{
    hipLaunchKernelGGL((mx_act_kernel<BF16, MAXC, NJB, SM, NW>), dim3((unsigned)(Mp / 16)), dim3(64 * NW), 0, s, p);
    return hipGetLastError();
}
template <bool BF16, int MAXC, bool SM, int NW>
static hipError_t mx_act_rank(const MxActParams& p, int64_t Mp, hipStream_t s)
{
    switch (p.r) {
        case 0: return mx_act_launch<BF16, MAXC, 0, SM, NW>(p, Mp, s);
        case 16: return mx_act_launch<BF16, MAXC, 1, SM, NW>(p, Mp, s);
        case 32: return mx_act_launch<BF16, MAXC, 2, SM, NW>(p, Mp, s);
        case 64: return mx_act_launch<BF16, MAXC, 4, SM, NW>(p, Mp, s);
        default: return mx_act_launch<BF16, MAXC, 8, SM, NW>(p, Mp, s);
    }
}
template <bool BF16, bool SM>
static hipError_t mx_act_len(const MxActParams& p, int64_t Mp, hipStream_t s)
{
    // Eight wavefronts while every 16 rows have a compute unit of their own (the time is one workgroup's chain: 2 x 1152 rank 32 4.5 us, four 5.1, 64 x
    // 4608 rank 128 13.7, 15.6, 4096 x 2240 rank 64 10.5, 11.5), and for long rows where they hold the row in few enough registers for two
    // workgroups to a compute unit, or four would have to stream it (8192 x 4608 rank 32 27.1, 28.8, rank 128 36.4, 40.0, 12000 x 2240 rank 16 19.7,
    // 20.8, smoothed 6001 x 4608 rank 128 36.0, 45.1); four elsewhere (16384 x 1152 rank 128 26.4, 21.8, 8192 x 4608 rank 64 32.3, 29.0, smoothed
    // 6001 x 2240 rank 64 18.3, 16.5, 16384 x 512 rank 32 10.8, 9.5).  Rank 64 is not among the long rows of bf16: eight wavefronts take 145 registers there and one
    // workgroup fits a compute unit, four (18 chunks each) 233 and two do; up to rank 32 eight take at most 122 and two fit, at rank 128 one fits either way.
    const bool fp32_rows = !BF16 || SM;
    // Rows beyond K = 4608 are streamed (MAXC = 0): by eight wavefronts where a chain is the time, but for fp32 input, whose reads bound it (us, four / eight: 400 x 4736
    // rank 32 bf16 16.0 / 15.6, fp32 23.2 / 25.8), and in a single part of a group (2 x 4736 fp32 13.1 / 11.9); by four beyond that, of which more
    // workgroups fit (8447 x 4736 rank 32 41.9 / 44.3, rank 128 54.2 / 59.8, smoothed fp32 12327 x 4736 rank 64 106.4 / 125.7).
    if (p.C64 > 72) {
        const bool eight = p.M < 16 || (BF16 && Mp <= 16 * compute_units());
        return eight ? mx_act_rank<BF16, 0, SM, 8>(p, Mp, s) : mx_act_rank<BF16, 0, SM, 4>(p, Mp, s);
    }
    const bool wide = Mp <= 16 * compute_units() || (p.C64 > 36 && (fp32_rows || p.r != 64)) || (!fp32_rows && p.r <= 32 && p.C64 > 20);
    if (wide) {
        const int mc = (p.C64 + 7) / 8;
        if (mc <= 3) return mx_act_rank<BF16, 3, SM, 8>(p, Mp, s);
        if (mc <= 5) return mx_act_rank<BF16, 5, SM, 8>(p, Mp, s);
        return mx_act_rank<BF16, 9, SM, 8>(p, Mp, s);
    }
    const int mc = (p.C64 + 3) / 4;  // (rows held as fp32 beyond K = 2304 went to eight wavefronts above)
    if (mc <= 5) return mx_act_rank<BF16, 5, SM, 4>(p, Mp, s);
    if constexpr (BF16 && !SM) {
        if (mc > 9) return mx_act_rank<BF16, 18, SM, 4>(p, Mp, s);
    }
    return mx_act_rank<BF16, 9, SM, 4>(p, Mp, s);
}

static hipError_t launch_quantize_act_mxb(const Dims& d, int x_dtype, const uint8_t* packed, const void* X, int64_t M,
                                          int64_t ldx, uint8_t* act, const lq_act_debug* dbg, hipStream_t s);

hipError_t launch_quantize_act_mx(const Dims& d, int x_dtype, const uint8_t* packed, const void* X, int64_t M,
                                  int64_t ldx, uint8_t* act, const lq_act_debug* dbg, hipStream_t s)
{
    if (d.mxb_elem == 6) return launch_quantize_act_mx6(d, x_dtype, packed, X, M, ldx, act, dbg, s);
    if (d.mxb) return launch_quantize_act_mxb(d, x_dtype, packed, X, M, ldx, act, dbg, s);
    const PackedLayout pl = packed_layout(d);
    const ActLayout al = act_layout(d, M);
    MxActParams p;
    p.tag = make_tag(d, LQ_BLOB_ACT, M);
    p.tag_dst = (uint32_t*)act;
    p.X = X;
    p.ldx = ldx;
    p.M = (int)M;
    p.K = (int)d.Ks;
    p.C64 = d.C64;
    p.C64s = (int)(d.Ks / 64);
    p.CQ = (d.C64 + 3) / 4;
    p.r = d.r;
    p.rp = d.rp;
    p.r8 = packed + pl.off_rq;
    p.sr = (const float*)(packed + pl.off_sr);
    p.xc = act + al.off_xq;
    p.xe = act + al.off_sx;
    p.tq8 = act + al.off_tq;
    p.st = (float*)(act + al.off_st);
    p.dbg_xb = dbg ? dbg->xb : nullptr;
    p.dbg_sxb = dbg ? dbg->sxb : nullptr;
    p.dbg_T = dbg ? dbg->T : nullptr;
    p.rg = d.smooth ? (const float*)(packed + pl.off_rg) : nullptr;
    if (d.smooth) return x_dtype == LQ_BF16 ? mx_act_len<true, true>(p, al.Mp, s) : mx_act_len<false, true>(p, al.Mp, s);
    return x_dtype == LQ_BF16 ? mx_act_len<true, false>(p, al.Mp, s) : mx_act_len<false, false>(p, al.Mp, s);
}

// ---------------------------------------------------------------------------------------------
// activation kernel with an MXFP8e4 branch.  Same decomposition as above, but K is walked in chunks
// of 128 (= one v_mfma_scale_f32_16x16x128_f8f6f4): lane (row l%16, q = l/16) holds the 16 values
// k = 16q.. of each 64-half of the chunk, which is both the fragment position of the 4-bit main codes
// and, as E4M3, bytes 0..15 / 16..31 of the lane's 8-bit MFMA operand.  A 32-block is shared by the
// lane pair (q, q^1); the MFMA takes the scale of block q from lane (row, q), so lanes 1 and 2 swap.
//
// No scale spans more than a block, so the row is streamed, two chunks of X in flight per wavefront; the chunk's R is requested before its X
// is coded and used after.  What bounds it: at one workgroup per compute unit the chain of a wavefront's chunks and the way of R (r K bytes)
// through one compute unit, at more R's traffic from the L2 beside X's from memory (mxb_act_form has the forms and their times).  us a call,
// four wavefronts with R a chunk ahead, values unpacked to fp32 and addresses in vector registers / this: 2 x 1152 rank 32 5.4 / 4.1, 300 x 1152
// rank 64 6.6 / 5.0, 64 x 4608 rank 128 17.2 / 9.1, 6001 x 2240 rank 64 17.8 / 15.7, 16384 x 1152 rank 64 20.1 / 16.3, rank 128 32.7 / 21.5.
// ---------------------------------------------------------------------------------------------
struct MxbActParams {
    const void* X;
    int64_t ldx;
    int M, K, C64, C64s, CQ, C128, r, rp;  // K, C64s: the caller's row length and its 64-chunks; C64, C128: of the layout
    const uint8_t* r8;
    const uint8_t* re;
    uint8_t* xc;
    uint8_t* xe;
    uint8_t* tq8;
    uint8_t* te;
    int8_t* dbg_xb;
    uint8_t* dbg_xbe;
    float* dbg_T;
    const float* rg;  // reciprocals of the smoothing vector (smoothing variant only)
    BlobTag tag;        // header of the activation blob (written by the first workgroup)
    uint32_t* tag_dst;
};

// BF16IN: element type of X; SM: smoothing variant (X times the stored reciprocals, held as fp32); DBG: parity taps; SHORT: rows of few chunks (mxb_act_short).
template <bool BF16IN, int NJB, bool SM, int NW, bool DBG, bool SHORT>
__global__ __launch_bounds__(64 * NW, 2) void mxb_act_kernel(MxbActParams p)
{
    write_tag(p.tag_dst, p.tag);
    constexpr bool BF16 = BF16IN && !SM;  // representation of a chunk in registers
    constexpr int NJA = NJB > 0 ? NJB : 1;
    constexpr int NS = 8, SW = NS / NW;  // T is eight sums, over the chunks c = 0 .. 7 mod 8, added in order; SW of them to a wavefront
    __shared__ float s_acc[NS][NJA][64][4];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, q = lane >> 4;
    const int row = blockIdx.x * 16 + r16;
    const bool row_ok = row < p.M;
    const uint32_t rowmask = row_ok ? ~0u : 0u;
    const int C64 = p.C64, C128 = p.C128;
    const int njb = p.r >> 4, jb0 = (int)blockIdx.y * NJB;  // this workgroup's 16-column groups of the rank; the first one stores the main codes
    const bool first = blockIdx.y == 0;

    const int nmy = (C128 - wave + NW - 1) / NW;  // chunks of this wavefront: c = wave + NW * ci, ci < nmy
    struct XSet { MxChunk<BF16> h[2]; };
    XSet xs[2];
    const size_t xrow = (size_t)(row_ok ? row : p.M - 1) * p.ldx + q * 16;
    // (no branch around the loads, which would end the compiler's count of those in flight: past the end they are clamped, and not used)
    auto load_x = [&](XSet& x, int ci) {
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            int c64 = 2 * (wave + NW * ci) + hh;
            c64 = c64 < p.C64s ? c64 : p.C64s - 1;
            if constexpr (SM)
                smooth_load<BF16IN, 16>(x.h[hh].v, p.X, xrow + (size_t)c64 * 64, p.rg + (size_t)c64 * 64 + q * 16, true);
            else
                x.h[hh].load(p.X, xrow + (size_t)c64 * 64, true);
        }
    };
    v4f acc[SW][NJA];
#pragma unroll
    for (int i = 0; i < SW; ++i)
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) acc[i][jb] = v4f{0.f, 0.f, 0.f, 0.f};

    // R, the codes and their scales go through descriptors (of R's sections and of this workgroup's block of 32 rows): a lane offset each and the
    // chunk in a scalar register, instead of 64-bit addresses in vector registers, of which three wavefronts per SIMD have none to spare.
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    const int rblk = (int)(blockIdx.x >> 1);
    const __amdgpu_buffer_rsrc_t rs_r = __builtin_amdgcn_make_buffer_rsrc((void*)p.r8, 0, (int)((unsigned)C128 * njb * 2048u), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_e = __builtin_amdgcn_make_buffer_rsrc((void*)p.re, 0, C128 * njb * 256, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_c = __builtin_amdgcn_make_buffer_rsrc(p.xc + (size_t)rblk * C64 * 1024, 0, C64 * 1024, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_s = __builtin_amdgcn_make_buffer_rsrc(p.xe + (size_t)rblk * p.CQ * 256, 0, p.CQ * 256, 0x00020000);
    const int off_c = ((row & 31) + 32 * (q >> 1)) * 16 + (q & 1) * 8, off_s = ((row & 31) + 32 * (q >> 1)) * 4;
    auto store_scales = [&](int c, uint32_t two) {  // of 64-chunks 2 c and 2 c + 1: neighbours in a dword
        if ((q & 1) == 0) __builtin_amdgcn_raw_buffer_store_b16((unsigned short)two, rs_s, off_s, (c >> 1) * 256 + (c & 1) * 2, 0);
    };

    // One chunk: request its R, code its X, request X of the chunk after the next (refill), multiply.
    auto step = [&](auto slot, int ci, auto refill) {
        constexpr int par = decltype(slot)::value, set = par % SW;  // (the chunks of a slot are those of one sum)
        XSet& x = xs[par];
        const int c = wave + NW * ci;
        v8i bv[NJA];
        int bs[NJA];
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) {
            const u4 lo = __builtin_amdgcn_raw_buffer_load_b128(rs_r, lane * 32, (c * njb + jb0 + jb) * 2048, 0);
            const u4 hi = __builtin_amdgcn_raw_buffer_load_b128(rs_r, lane * 32 + 16, (c * njb + jb0 + jb) * 2048, 0);
            bv[jb] = v8i{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
            bs[jb] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs_e, lane * 4, (c * njb + jb0 + jb) * 256, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        uint32_t x8[8], E4[2], Eh[2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const MxChunk<BF16>& xc = x.h[hh];
            const int c64 = 2 * c + hh;
            const uint32_t keep = c64 < p.C64s ? rowmask : 0u;  // (rows past M and the layout's padding chunk: amax and codes 0)
            const float ab = __uint_as_float(__float_as_uint(max_xor16(mx_amax16(xc))) & keep);  // amax of the 32-block (lanes q, q^1)
            E4[hh] = e8m0_of(ab);                        // main codes: MXFP4
            if (first) {
                uint32_t pk[2] = {0u, 0u};
                mxfp4_codes16(xc, e8m0_value(E4[hh]), pk);
                const uint32_t nz = ab != 0.0f ? ~0u : 0u;  // (a block of zeros has codes 0, also where the zeros are negative)
                __builtin_amdgcn_raw_buffer_store_b64(u2{pk[0] & nz, pk[1] & nz}, rs_c, off_c, c64 * 1024, 0);
            }
            if constexpr (NJB > 0 || DBG) {              // branch codes: MXFP8e4 of the same block
                Eh[hh] = e8m0_of_fp8(ab);
                mxfp8_codes16(xc, Eh[hh], x8 + 4 * hh);
#pragma unroll
                for (int g = 0; g < 4; ++g) x8[4 * hh + g] &= keep;
                if (DBG && p.dbg_xb && row_ok && c64 < p.C64s)
                    *(v4i*)(p.dbg_xb + (size_t)row * p.K + (size_t)c * 128 + hh * 64 + q * 16) =
                        v4i{(int)x8[4 * hh], (int)x8[4 * hh + 1], (int)x8[4 * hh + 2], (int)x8[4 * hh + 3]};
                if (DBG && p.dbg_xbe && row_ok && c64 < p.C64s && (q & 1) == 0) p.dbg_xbe[(size_t)row * (p.K >> 5) + 4 * c + 2 * hh + (q >> 1)] = (uint8_t)Eh[hh];
            }
        }
        if (first) store_scales(c, E4[0] | E4[1] << 8);
        // (the codes are formed before the slot is filled again: moved down to their use they would keep both rows of X in registers)
        if constexpr (NJB > 0) asm volatile("" : "+v"(x8[0]), "+v"(x8[1]), "+v"(x8[2]), "+v"(x8[3]), "+v"(x8[4]), "+v"(x8[5]), "+v"(x8[6]), "+v"(x8[7]));
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(refill)::value) {
            load_x(x, ci + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (NJB > 0) {
            // lane q knows blocks (q>>1) [first half] and 2+(q>>1) [second half]; it must supply block q
            const uint32_t send = (q == 1) ? Eh[1] : Eh[0];
            const auto h32 = __builtin_amdgcn_permlane32_swap(send, send, false, false);  // the value of lane ^ 48, without the LDS
            const uint32_t o32 = q < 2 ? h32[1] : h32[0];
            const auto h16 = __builtin_amdgcn_permlane16_swap(o32, o32, false, false);
            const uint32_t recv = (q & 1) ? h16[0] : h16[1];
            const int sa = (int)((q == 0) ? Eh[0] : (q == 3) ? Eh[1] : recv);
            const v8i a8 = {(int)x8[0], (int)x8[1], (int)x8[2], (int)x8[3], (int)x8[4], (int)x8[5], (int)x8[6], (int)x8[7]};
#pragma unroll
            for (int jb = 0; jb < NJB; ++jb)
                acc[set][jb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a8, bv[jb], acc[set][jb], 0, 0, 0, sa, 0, bs[jb]);
            // (the products stay ahead of the next chunk's request of R: moved behind it they would hold both chunks' R in registers)
#pragma unroll
            for (int jb = 0; jb < NJB; ++jb) asm volatile("" : "+v"(acc[set][jb]));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    constexpr std::integral_constant<int, 0> s0{};
    constexpr std::integral_constant<int, 1> s1{};
    if constexpr (SHORT) {
        if (nmy > 0) {
            load_x(xs[0], 0);
            if (NW == 4 && nmy > 1) load_x(xs[1], 1);
            step(s0, 0, std::false_type{});
            if (NW == 4 && nmy > 1) step(s1, 1, std::false_type{});
        }
    } else {
        load_x(xs[0], 0);
        __builtin_amdgcn_sched_barrier(0);
        load_x(xs[1], 1);
        __builtin_amdgcn_sched_barrier(0);
        int ci = 0;
        for (; ci + 3 < nmy; ci += 2) {
            step(s0, ci, std::true_type{});
            step(s1, ci + 1, std::true_type{});
        }
        if (ci + 2 < nmy) {
            step(s0, ci, std::true_type{});
            step(s1, ci + 1, std::false_type{});
            step(s0, ci + 2, std::false_type{});
        } else {
            if (ci < nmy) step(s0, ci, std::false_type{});
            if (ci + 1 < nmy) step(s1, ci + 1, std::false_type{});
        }
    }
    {   // padding 64-chunks of the last quad (at most one 128-chunk): valid E8M0 bytes (2^0)
        const int c = wave + NW * nmy;
        if (first && 2 * c < 4 * p.CQ) store_scales(c, 0x7F7Fu);
    }
    if (NJB == 0) return;

#pragma unroll
    for (int i = 0; i < SW; ++i)
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) *(v4f*)&s_acc[wave + NW * i][jb][lane][0] = acc[i][jb];
    __syncthreads();
    // The eight sums, re-quantised per token and per block of 32 along the rank: a task is a block (two 16-column groups) and two of a lane's
    // four token rows.  The lane holds columns (2 bb + g) * 16 + lane%16 of the intermediate for token rows 4*q + i.
    for (int task = wave; task < 2 * ((NJB + 1) / 2); task += NW) {
        const int bb = task >> 1, half = task & 1;
        float T[2][2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int jb = 2 * bb + g;
            typedef float v2f __attribute__((ext_vector_type(2)));
            v2f o[NS];
#pragma unroll
            for (int w = 0; w < NS; ++w) o[w] = *(const v2f*)&s_acc[w][jb][lane][2 * half];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                float sum = o[0][i];
#pragma unroll
                for (int w = 1; w < NS; ++w) sum = __fadd_rn(sum, o[w][i]);
                T[g][i] = sum;
                const int grow = blockIdx.x * 16 + 4 * q + 2 * half + i;
                if (DBG && grow < p.M && p.dbg_T) p.dbg_T[(size_t)grow * p.r + (jb0 + jb) * 16 + r16] = sum;
            }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            float tm = fmaxf(fabsf(T[0][i]), fabsf(T[1][i]));
            tm = max_row16(tm);
            const int grow = blockIdx.x * 16 + 4 * q + 2 * half + i;
            const uint32_t E = e8m0_of_fp8(tm);
            const float inv = e8m0_inverse(E);
            if (r16 == 0) p.te[mxb_scale_offset(grow, (jb0 >> 1) + bb)] = (uint8_t)E;
#pragma unroll
            for (int g = 0; g < 2; ++g)
                p.tq8[mxb_frag8_offset(grow, (jb0 + 2 * bb + g) * 16 + r16, p.rp)] = (uint8_t)fp8_byte(__fmul_rn(T[g][i], inv));
        }
    }
    if (wave != NW - 1 || !first) return;
    // padding of the rank to a multiple of 64: zero codes, scale 2^0
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int grow = blockIdx.x * 16 + 4 * q + i;
        for (int j = p.r + r16; j < p.rp; j += 16) p.tq8[mxb_frag8_offset(grow, j, p.rp)] = 0;
        if (r16 == 0)
            for (int bb = p.r >> 5; bb < (p.rp >> 5); ++bb) p.te[mxb_scale_offset(grow, bb)] = (uint8_t)127;
    }
}

template <bool BF16, int NJB, bool SM, int NW, bool DBG>
static hipError_t mxb_act_launch3(const MxbActParams& p, dim3 grid, hipStream_t s)
{
    if (!DBG && p.C128 <= mxb_act_short(NW))
        hipLaunchKernelGGL((mxb_act_kernel<BF16, NJB, SM, NW, false, true>), grid, dim3(64 * NW), 0, s, p);
    else
        hipLaunchKernelGGL((mxb_act_kernel<BF16, NJB, SM, NW, DBG, false>), grid, dim3(64 * NW), 0, s, p);
    return hipGetLastError();
}
template <bool BF16, int NJB, bool SM, bool DBG>
static hipError_t mxb_act_launch2(const MxbActParams& p, int64_t Mp, hipStream_t s)
{
    const dim3 rows((unsigned)(Mp / 16));
    switch (mxb_act_form(Mp, p.C128, NJB, !BF16 || SM)) {
        case 4: return mxb_act_launch3<BF16, NJB, SM, 4, DBG>(p, rows, s);
        case 8: return mxb_act_launch3<BF16, NJB, SM, 8, DBG>(p, rows, s);
        default: return mxb_act_launch3<BF16, NJB < 2 ? NJB : 2, SM, 8, DBG>(p, dim3(rows.x, NJB < 2 ? 1 : NJB / 2), s);
    }
}
template <bool BF16, int NJB, bool SM>
static hipError_t mxb_act_launch(const MxbActParams& p, int64_t Mp, hipStream_t s)
{
    return p.dbg_xb || p.dbg_xbe || p.dbg_T ? mxb_act_launch2<BF16, NJB, SM, true>(p, Mp, s) : mxb_act_launch2<BF16, NJB, SM, false>(p, Mp, s);
}
template <bool BF16, bool SM>
static hipError_t mxb_act_rank2(const MxbActParams& p, int64_t Mp, hipStream_t s)
{
    switch (p.r) {
        case 0: return mxb_act_launch<BF16, 0, SM>(p, Mp, s);
        case 32: return mxb_act_launch<BF16, 2, SM>(p, Mp, s);
        case 64: return mxb_act_launch<BF16, 4, SM>(p, Mp, s);
        case 96: return mxb_act_launch<BF16, 6, SM>(p, Mp, s);
        default: return mxb_act_launch<BF16, 8, SM>(p, Mp, s);
    }
}
template <bool BF16>
static hipError_t mxb_act_rank(const MxbActParams& p, int64_t Mp, hipStream_t s)
{
    return p.rg ? mxb_act_rank2<BF16, true>(p, Mp, s) : mxb_act_rank2<BF16, false>(p, Mp, s);
}

static hipError_t launch_quantize_act_mxb(const Dims& d, int x_dtype, const uint8_t* packed, const void* X, int64_t M,
                                          int64_t ldx, uint8_t* act, const lq_act_debug* dbg, hipStream_t s)
{
    const PackedLayout pl = packed_layout(d);
    const ActLayout al = act_layout(d, M);
    MxbActParams p;
    p.tag = make_tag(d, LQ_BLOB_ACT, M);
    p.tag_dst = (uint32_t*)act;
    p.X = X;
    p.ldx = ldx;
    p.M = (int)M;
    p.K = (int)d.Ks;
    p.C64 = d.C64;
    p.C64s = (int)(d.Ks / 64);
    p.CQ = (d.C64 + 3) / 4;
    p.C128 = d.C64 / 2;
    p.r = d.r;
    p.rp = d.rp;
    p.r8 = packed + pl.off_rq;
    p.re = packed + pl.off_sr;
    p.xc = act + al.off_xq;
    p.xe = act + al.off_sx;
    p.tq8 = act + al.off_tq;
    p.te = act + al.off_st;
    p.dbg_xb = dbg ? dbg->xb : nullptr;
    p.dbg_xbe = dbg ? dbg->xbe : nullptr;
    p.dbg_T = dbg ? dbg->T : nullptr;
    p.rg = d.smooth ? (const float*)(packed + pl.off_rg) : nullptr;
    return x_dtype == LQ_BF16 ? mxb_act_rank<true>(p, al.Mp, s) : mxb_act_rank<false>(p, al.Mp, s);
}

// ---------------------------------------------------------------------------------------------
// forward: 1 x 4 wavefronts per workgroup, 128 x 64 outputs per wavefront, K staged 128 at a time
// ---------------------------------------------------------------------------------------------
struct MxFwdParams {
    const uint8_t* xc;
    const uint8_t* xe;
    const uint8_t* tq8;
    const float* st;
    const uint8_t* pc;
    const uint8_t* pe;
    const uint8_t* l8;
    const float* sl;
    uint16_t* Y;
    int64_t ldy;
    int M, N, C64, CQ, S, rp, nrb;
    int tilesM, tilesN, panel;
    int n_full;  // workgroups that compute whole tiles; the rest of the grid are half tiles
    float* dbg_y32;
};

// NK = 64-deep chunks of the (padded) rank: 0 | 1 | 2.  BLK: the branch is MXFP8e4 (block scales,
// accumulated by the scaled MFMA straight into the main product's accumulators).
// BFMT: operand format code of the block-scaled branch (0 = E4M3, 2 = E2M3).
namespace mxf {
constexpr int WN = 4, RBT = 4;
constexpr int EPI_ROW = 136, EPI_WAVE = 32 * EPI_ROW;
constexpr int NBUF = 4;                          // LDS buffers of the activation stream (one stage each)
constexpr int LDS_MAIN = NBUF * 2 * RBT * 1024;  // [buffer][chunk in stage][row block][lane][16 B]
constexpr int LDS_BYTES = LDS_MAIN > 4 * EPI_WAVE ? LDS_MAIN : 4 * EPI_WAVE;
constexpr int LDS_TOTAL = LDS_BYTES + WN * 64 * 4;
}  // namespace mxf

// One output tile: row blocks rb0 .. rb0 + NRB - 1 (NRB = 4: a whole 128-row tile; 2: a half tile of the grid's last,
// sparse generation), columns tile_n * 256 ...  The four wavefronts always stage four row blocks (clamped).
template <int NK, bool DBG, bool BLK, int BFMT, int NRB>
__device__ __forceinline__ void mx_fwd_tile(const MxFwdParams& p, uint8_t* lds, const int rb0, const int tile_n)
{
    using namespace mxf;
    float* lds_sl = (float*)(lds + LDS_BYTES);  // + the tile's 256 per-channel scales of the fp32-scaled branch

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;

    const int cb0 = tile_n * (WN * 2) + wave * 2;
    const bool active = (cb0 * 32 < p.N) && (rb0 < p.nrb);
    const int C64 = p.C64, CQ = p.CQ, S = p.S;

    const uint32_t lane16 = (uint32_t)lane * 16u, lane4 = (uint32_t)lane * 4u;
    int rbs = rb0 + wave;  // row block staged by this wavefront
    rbs = rbs < p.nrb ? rbs : p.nrb - 1;
    const uint8_t* xc_base = p.xc + (size_t)rbs * C64 * 1024;
    const int cbw = (cb0 * 32 < p.N) ? cb0 : 0;
    const uint8_t* pc_base[2] = {p.pc + (size_t)cbw * C64 * 1024, p.pc + (size_t)(cbw + 1) * C64 * 1024};
    const uint8_t* pe_base[2] = {p.pe + (size_t)cbw * CQ * 256, p.pe + (size_t)(cbw + 1) * CQ * 256};
    const uint8_t* xe_base[NRB];
#pragma unroll
    for (int rbi = 0; rbi < NRB; ++rbi) {
        int rb = rb0 + rbi;
        rb = rb < p.nrb ? rb : p.nrb - 1;
        xe_base[rbi] = p.xe + (size_t)rb * CQ * 256;
    }

    struct AStage { v4i v[2]; };
    struct BStage { v4i v[2][2]; };
    // The streams are read with buffer loads: a wave-uniform descriptor and chunk offset in scalar registers plus the
    // 32-bit lane offsets all streams share, instead of a 64-bit vector address per stream (about 28 registers per
    // lane fewer).  Each descriptor spans exactly the bytes its stream may touch.
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    constexpr int RSRC_FLAGS = 0x00020000;
    const __amdgpu_buffer_rsrc_t rs_pe[2] = {__builtin_amdgcn_make_buffer_rsrc((void*)pe_base[0], 0, CQ * 256, RSRC_FLAGS),
                                             __builtin_amdgcn_make_buffer_rsrc((void*)pe_base[1], 0, CQ * 256, RSRC_FLAGS)};
    __amdgpu_buffer_rsrc_t rs_xe[NRB];
#pragma unroll
    for (int rbi = 0; rbi < NRB; ++rbi) rs_xe[rbi] = __builtin_amdgcn_make_buffer_rsrc((void*)xe_base[rbi], 0, CQ * 256, RSRC_FLAGS);
    // A load for a stage (or quad of chunks) past the end goes through a descriptor of zero bytes: every lane is out of
    // range, nothing is fetched and the (unused) result is zero; the loop body stays branch-free.
    auto load_a = [&](AStage& a, int stage) {
        const bool ok = stage < S;
        const int st = ok ? stage : S - 1;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)xc_base, 0, ok ? C64 * 1024 : 0, RSRC_FLAGS);
#pragma unroll
        for (int cc = 0; cc < 2; ++cc)
            a.v[cc] = __builtin_bit_cast(v4i, (u4)__builtin_amdgcn_raw_buffer_load_b128(rs, lane16, (st * 2 + cc) * 1024, 0));
    };
    auto store_a = [&](const AStage& a, int buf) {
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) *(v4i*)(lds + (size_t)(((buf * 2 + cc) * RBT + wave) * 1024) + lane16) = a.v[cc];
    };
    auto load_b = [&](BStage& b, int stage) {
        const bool ok = stage < S;
        const int st = ok ? stage : S - 1;
#pragma unroll
        for (int cbi = 0; cbi < 2; ++cbi) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)pc_base[cbi], 0, ok ? C64 * 1024 : 0, RSRC_FLAGS);
#pragma unroll
            for (int cc = 0; cc < 2; ++cc)
                b.v[cc][cbi] = __builtin_bit_cast(v4i, (u4)__builtin_amdgcn_raw_buffer_load_b128(rs, lane16, (st * 2 + cc) * 1024, 0));
        }
    };
    // scale dwords of one quad of chunks (= two stages)
    struct Scales { int a[NRB]; int b[2]; };
    auto load_s = [&](Scales& sc, int quad) {
        const int q = quad < CQ ? quad : CQ - 1;
#pragma unroll
        for (int rbi = 0; rbi < NRB; ++rbi) sc.a[rbi] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs_xe[rbi], lane4, q * 256, 0);
#pragma unroll
        for (int cbi = 0; cbi < 2; ++cbi) sc.b[cbi] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs_pe[cbi], lane4, q * 256, 0);
    };

    v16f t[NRB][2];
#pragma unroll
    for (int a = 0; a < NRB; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) t[a][b][i] = 0.f;

    // One stage = 128 values of K = two 64-chunks = eight activation fragments (chunk, row block), each the A operand of
    // two MFMAs.  P = stage index mod 4: LDS buffer P holds the stage's activation codes, buffer P+1 those of the next
    // stage (written one stage earlier, so they are visible without a barrier in between), buffer P+2 receives stage
    // s+2 during this one.  The fragments are read two ahead of their MFMAs into a ring of four register sets, across
    // the stage boundary as well, so that a wavefront on its own keeps the matrix core busy (the barrier at the end of
    // a stage orders LDS writes against reads two stages apart; nothing waits on it).  Loads past the last stage are
    // issued through an empty descriptor: at K = 1152 they would be a sixth of the wavefront's vector-memory work.
    // The op_sel immediates of the scale bytes are 2*(P&1) and 2*(P&1)+1.
    v4i fr[4];
    constexpr int NF = 2 * NRB;                    // fragments of a stage
    auto lds_frag = [&](int buf, int f) -> v4i {   // f = chunk * NRB + row block
        return *(const v4i*)(lds + (size_t)((buf * 2 * RBT + (f / NRB) * RBT + f % NRB) * 1024) + lane16);
    };
    auto do_stage = [&](auto pc, int s, AStage& a, BStage& b, const Scales& sc) {
        constexpr int P = decltype(pc)::value, PAR = P & 1;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const int cc = f / NRB, rbi = f % NRB;
            fr[(f + 2) & 3] = f + 2 < NF ? lds_frag(P, f + 2) : lds_frag((P + 1) & 3, f + 2 - NF);
            if (f == 0) store_a(a, (P + 2) & 3);
            if (f == 1) load_a(a, s + 4);
            const v4i av = fr[f & 3];
            const v8i a8 = {av[0], av[1], av[2], av[3], 0, 0, 0, 0};
#pragma unroll
            for (int cbi = 0; cbi < 2; ++cbi) {
                const v4i bq = b.v[cc][cbi];
                const v8i b8 = {bq[0], bq[1], bq[2], bq[3], 0, 0, 0, 0};
                // the weights are the first operand: a lane then holds one token and, per register quad, four
                // consecutive channels (the epilogue packs them into 8-byte LDS writes)
                if (cc == 0)
                    t[rbi][cbi] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(b8, a8, t[rbi][cbi], 4, 4, 2 * PAR,
                                                                                 sc.b[cbi], 2 * PAR, sc.a[rbi]);
                else
                    t[rbi][cbi] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(b8, a8, t[rbi][cbi], 4, 4, 2 * PAR + 1,
                                                                                 sc.b[cbi], 2 * PAR + 1, sc.a[rbi]);
            }
            if (f == NF - 1) load_b(b, s + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
    };

    // A wavefront whose columns lie past N (the last tile column of a layer whose width is no multiple of 256) only stages
    // its row block of the activation codes, barrier for barrier with the others: no matrix work, no
    // weight or scale loads that would compete with the wavefront it shares a SIMD with.
    if (cb0 * 32 >= p.N) {  // wave-uniform
        AStage x0, x1;
        load_a(x0, 0);
        load_a(x1, 1);
        store_a(x0, 0);
        store_a(x1, 1);
        load_a(x0, 2);
        load_a(x1, 3);
        __syncthreads();
        for (int s = 0; s < S; s += 2) {  // stage s sends stage s + 2 to its buffer and requests stage s + 4
            store_a(x0, (s + 2) & 3);
            load_a(x0, s + 4);
            __syncthreads();
            if (s + 1 >= S) break;
            store_a(x1, (s + 3) & 3);
            load_a(x1, s + 5);
            __syncthreads();
        }
        return;
    }
    AStage a0, a1;
    BStage b0, b1;
    Scales s0, s1;
    load_a(a0, 0);
    load_a(a1, 1);
    load_b(b0, 0);
    load_s(s0, 0);
    store_a(a0, 0);
    store_a(a1, 1);
    __builtin_amdgcn_sched_barrier(0);
    load_a(a0, 2);
    load_a(a1, 3);
    load_b(b1, 1);
    load_s(s1, 1);
    // Operands of the epilogue's first matrix instructions (the branch's channel codes, the intermediate codes of the
    // first row block) are requested here: asked for at the start of the epilogue, their round trip would open it.
    constexpr int NKF = BLK ? 0 : NK;  // chunks of the fp32-scaled branch handled in the epilogue
    constexpr int NKA = NKF > 0 ? NKF : 1;
    constexpr bool TQ_ALL = NKF <= 1;
    v8i lf[2][NKA];
    v8i tf[TQ_ALL ? NRB : 1][NKA];
    auto load_tq = [&](int rbi) {
        int rb = rb0 + rbi;
        rb = rb < p.nrb ? rb : p.nrb - 1;
#pragma unroll
        for (int kk = 0; kk < NKF; ++kk)
            tf[TQ_ALL ? rbi : 0][kk] = *(const v8i*)(p.tq8 + (size_t)(rb * 32 + l32) * p.rp + kk * 64 + half * 32);
    };
    auto load_lf = [&]() {
#pragma unroll
        for (int cbi = 0; cbi < 2; ++cbi)
#pragma unroll
            for (int kk = 0; kk < NKF; ++kk)
                lf[cbi][kk] = *(const v8i*)(p.l8 + (size_t)((cbw + cbi) * 32 + l32) * p.rp + kk * 64 + half * 32);
    };
    constexpr bool EARLY = NKF == 1;  // (two chunks: the registers are not there; the epilogue requests them itself)
    if constexpr (EARLY) {
        load_lf();
        load_tq(0);
    }
    // ... and, last, the branch's scales: of this lane's tokens, and of the wavefront's channel `lane`
    float stl[NRB], sl_lane = 0.f;
    if constexpr (!BLK && NK > 0) {
#pragma unroll
        for (int rbi = 0; rbi < NRB; ++rbi) {
            int rb = rb0 + rbi;
            rb = rb < p.nrb ? rb : p.nrb - 1;
            stl[rbi] = p.st[rb * 32 + l32];
        }
        sl_lane = p.sl[cbw * 32 + lane];
    }
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    fr[0] = lds_frag(0, 0);
    fr[1] = lds_frag(0, 1);

    // stages come in groups of four (two quads of chunks): quad q uses scale set q & 1
    int s = 0;
    for (; s + 3 < S; s += 4) {
        do_stage(std::integral_constant<int, 0>{}, s, a0, b0, s0);
        do_stage(std::integral_constant<int, 1>{}, s + 1, a1, b1, s0);
        load_s(s0, (s >> 1) + 2);
        do_stage(std::integral_constant<int, 2>{}, s + 2, a0, b0, s1);
        do_stage(std::integral_constant<int, 3>{}, s + 3, a1, b1, s1);
        load_s(s1, (s >> 1) + 3);
    }
    if (s < S) {
        do_stage(std::integral_constant<int, 0>{}, s, a0, b0, s0);
        if (s + 1 < S) do_stage(std::integral_constant<int, 1>{}, s + 1, a1, b1, s0);
        if (s + 2 < S) do_stage(std::integral_constant<int, 2>{}, s + 2, a0, b0, s1);
    }

    if (!active) return;

    if constexpr (BLK) {
        // ---- MXFP8e4 branch: tq . lq^T with both block scales, on top of the main accumulators.
        // Operands are stored in the 8-bit operand order of the instruction (32 bytes per lane and
        // 64-chunk of the rank); the scale dword of a lane holds the byte of chunk cc at position cc.
#pragma unroll
        for (int cc = 0; cc < NK; ++cc) {
            v8i lb[2];
            int lsc[2];
#pragma unroll
            for (int cbi = 0; cbi < 2; ++cbi) {
                lb[cbi] = *(const v8i*)(p.l8 + ((size_t)((size_t)(cb0 + cbi) * NK + cc) * 64 + lane) * 32);
                lsc[cbi] = *(const int*)((const uint8_t*)p.sl + ((size_t)(cb0 + cbi) * 64 + lane) * 4);
            }
#pragma unroll
            for (int rbi = 0; rbi < NRB; ++rbi) {
                int rb = rb0 + rbi;
                rb = rb < p.nrb ? rb : p.nrb - 1;
                const v8i ta = *(const v8i*)(p.tq8 + ((size_t)((size_t)rb * NK + cc) * 64 + lane) * 32);
                const int tsc = *(const int*)((const uint8_t*)p.st + ((size_t)rb * 64 + lane) * 4);
#pragma unroll
                for (int cbi = 0; cbi < 2; ++cbi) {
                    if (cc == 0)
                        t[rbi][cbi] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(lb[cbi], ta, t[rbi][cbi], BFMT, BFMT, 0, lsc[cbi], 0, tsc);
                    else
                        t[rbi][cbi] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(lb[cbi], ta, t[rbi][cbi], BFMT, BFMT, 1, lsc[cbi], 1, tsc);
                }
            }
        }
    }

    // ---- epilogue: FP8 rank-r expansion, scales, sum, bf16, full-line stores -------
    // A lane holds token l32 of a row block and, in registers 4g .. 4g+3 of a 32 x 32 tile, channels 8g + 4 half + 0..3:
    // four bf16 values = one 8-byte LDS write; the block is read back row-wise, 16 bytes per lane.
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    uint8_t* stage = lds + wave * EPI_WAVE;
    if constexpr (!BLK && NK > 0) lds_sl[wave * 64 + lane] = sl_lane;  // (read by this wavefront only)
    v4f slv[2][4];  // channel scales of the branch, in register order
#pragma unroll
    for (int cbi = 0; cbi < 2; ++cbi) {
        if (!BLK && NK > 0) {
#pragma unroll
            for (int g = 0; g < 4; ++g) slv[cbi][g] = *(const v4f*)(lds_sl + wave * 64 + cbi * 32 + 8 * g + 4 * half);
        }
    }
    const int wr_off = l32 * EPI_ROW + half * 8;
    const int rd_row = lane >> 3, rd_seg = lane & 7;
    // With one 64-chunk of the rank the intermediate codes of the other three row blocks are requested before the first
    // output store: the vector-memory counter retires in order, so a wait for a load issued after a store also waits for
    // that store's acknowledgement, and no such wait is left in the epilogue.  (Two chunks: one row block ahead; registers.)
    if constexpr (!EARLY) {
        load_lf();
        load_tq(0);
    }
    if constexpr (TQ_ALL) {
#pragma unroll
        for (int rbi = 1; rbi < NRB; ++rbi) load_tq(rbi);
    }
    // The stores are buffer stores through a descriptor that ends with the wavefront's 128 bytes of the tile's last valid
    // row: rows past M are out of range and dropped by the hardware, so the stores need no branch -- and only stores the
    // compiler can count let it wait for a load issued before them without waiting for the stores themselves.
    // They go through the caches: non-temporal stores make activation step and forward alone 1 to 15 % shorter and the kernel that reads Y
    // longer by as much or more (X written by the kernel before, the next layer's activation step behind, us, cached / non-temporal: 8192 x 2240
    // -> 11200 219.9 / 235.3, 16384 x 1152 -> 4608 146.1 / 150.2, 16384 x 1152 -> 3456 125.7 / 124.9, 2048 x 1152 -> 3456 37.1 / 36.0; with an
    // FP6 branch up to 10 % longer).
    const int rows_valid = p.M - rb0 * 32 < NRB * 32 ? p.M - rb0 * 32 : NRB * 32;
    const __amdgpu_buffer_rsrc_t rs_y = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(p.Y + (size_t)(rb0 * 32) * p.ldy + cb0 * 32), 0, (int)((rows_valid - 1) * p.ldy * 2 + 128), RSRC_FLAGS);
    uint32_t yoff = (uint32_t)(rd_row * (int)p.ldy * 2 + rd_seg * 16);
    const uint32_t ystep = (uint32_t)(8 * (int)p.ldy * 2);
    v4i ov[4];
#pragma unroll
    for (int rbi = 0; rbi < NRB; ++rbi) {
        const int rbase = (rb0 + rbi) * 32;
        v16f a2[2];
#pragma unroll
        for (int cbi = 0; cbi < 2; ++cbi) {
            a2[cbi] = v16f{0};
#pragma unroll
            for (int kk = 0; kk < NKF; ++kk)
                a2[cbi] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(lf[cbi][kk], tf[TQ_ALL ? rbi : 0][kk], a2[cbi], 0, 0, 0, 0, 0, 0);
        }
        if (!TQ_ALL && rbi + 1 < NRB) load_tq(rbi + 1);
        float y[2][16];
#pragma unroll
        for (int cbi = 0; cbi < 2; ++cbi)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                if (BLK) {
                    y[cbi][i] = t[rbi][cbi][i];
                } else if (NK == 0) {  // rank 0: the branch term is +0, whatever the (unused, possibly unwritten) scales hold
                    y[cbi][i] = __fadd_rn(t[rbi][cbi][i], 0.f);
                } else {
                    // two vector instructions per output: the scaled branch term enters through a fused multiply-add
                    // (the fp32 result is compared against a sum rounded once, within an accumulation bound)
                    y[cbi][i] = __builtin_fmaf(__fmul_rn(a2[cbi][i], stl[rbi]), slv[cbi][i >> 2][i & 3], t[rbi][cbi][i]);
                }
            }
#pragma unroll
        for (int cbi = 0; cbi < 2; ++cbi) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const bf16x2 h0 = __builtin_convertvector(f32x2{y[cbi][4 * g], y[cbi][4 * g + 1]}, bf16x2);
                const bf16x2 h1 = __builtin_convertvector(f32x2{y[cbi][4 * g + 2], y[cbi][4 * g + 3]}, bf16x2);
                *(v2i*)(stage + wr_off + cbi * 64 + g * 16) = v2i{__builtin_bit_cast(int, h0), __builtin_bit_cast(int, h1)};
            }
            if (DBG) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int row = rbase + l32;
                    const int col = (cb0 + cbi) * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
                    if (row < p.M && p.dbg_y32) p.dbg_y32[(size_t)row * p.N + col] = y[cbi][i];
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint8_t* src = stage + (q * 8 + rd_row) * EPI_ROW + rd_seg * 16;
            const v2i lo = *(const v2i*)src, hi = *(const v2i*)(src + 8);
            ov[q] = v4i{lo[0], lo[1], hi[0], hi[1]};
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, ov[q]), rs_y, yoff, 0, 0);
            yoff += ystep;
        }
    }
}

// Grid: the first n_full workgroups compute whole tiles (dealt round-robin to the XCDs, each XCD one contiguous run of the
// panel order); the tiles left over, if they were split (see the launcher), follow as two half tiles each.
template <int NK, bool DBG, bool BLK, int BFMT = 0>
__global__ __launch_bounds__(256, 2) void mx_fwd_kernel(MxFwdParams p)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[mxf::LDS_TOTAL];
    const int b = (int)blockIdx.x;
    auto xcd_order = [](int i, int n) {
        const int per = n >> 3, rem = n & 7, xcd = i & 7, loc = i >> 3;
        return xcd * per + (xcd < rem ? xcd : rem) + loc;
    };
    int tile_m, tile_n;
    if (b < p.n_full) {
        panel_tile(xcd_order(b, p.n_full), p.tilesM, p.tilesN, p.panel, tile_m, tile_n);
        mx_fwd_tile<NK, DBG, BLK, BFMT, 4>(p, lds, tile_m * 4, tile_n);
    } else {
        const int hh = xcd_order(b - p.n_full, 2 * (p.tilesM * p.tilesN - p.n_full));
        panel_tile(p.n_full + (hh >> 1), p.tilesM, p.tilesN, p.panel, tile_m, tile_n);
        const int rb0 = tile_m * 4 + (hh & 1) * 2;
        if (rb0 >= p.nrb) return;  // lower half of a partial last row tile
        mx_fwd_tile<NK, DBG, BLK, BFMT, 2>(p, lds, rb0, tile_n);
    }
}

// Small layers: a wavefront (a workgroup of its own) per tile of NRB*32 x NCB*32 outputs.  Where the 128 x 256 tiles leave most of the chip
// idle, the time of a call is one tile's serial chain of stages; here nothing is shared between wavefronts (no LDS staging, no
// barriers) and both operand streams are requested DEPTH quads of 64-chunks ahead straight into the registers the products
// read.  Bounded by that chain for a few tiles (128 x 1152 -> 3456: 7.6 -> 3.2 us, 128 x 4608 -> 1152: 16.2 -> 4.2 us), by the operands'
// L2 traffic for many.  Same products in the same order as mx_fwd_tile.
template <int NK, bool DBG, bool BLK, int BFMT, int NRB, int NCB>
__global__ __launch_bounds__(64, 2) void mx_fwd_small_kernel(MxFwdParams p)
{
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    constexpr int RSRC_FLAGS = 0x00020000;
    constexpr int DEPTH = NRB + NCB == 2 ? 4 : 2;  // quads in flight (17 registers per row or column block each)
    constexpr int ROW = 64 * NCB + 8;              // bytes per staged output row
    __shared__ __attribute__((aligned(16))) uint8_t stage[32 * ROW];

    const int lane = threadIdx.x, half = lane >> 5, l32 = lane & 31;
    // The tiles that share a block of the longer operand run together on one XCD: it is then read from memory once, the shorter one
    // stays in the L2.  (Row blocks always fastest, 31515 x 4608 -> 64: 25.2 us, now 15.4.)
    const int tiles = p.tilesM * p.tilesN, per = tiles >> 3, rem = tiles & 7, xcd = blockIdx.x & 7;
    const int tile = xcd * per + (xcd < rem ? xcd : rem) + ((int)blockIdx.x >> 3);
    const bool mfast = p.tilesM <= p.tilesN;
    const int slow = tile / (mfast ? p.tilesM : p.tilesN), fast = tile - slow * (mfast ? p.tilesM : p.tilesN);
    const int rb0 = (mfast ? fast : slow) * NRB, cb0 = (mfast ? slow : fast) * NCB;
    const int C64 = p.C64, CQ = p.CQ;
    const uint32_t lane16 = (uint32_t)lane * 16u, lane4 = (uint32_t)lane * 4u;

    int rbc[NRB];  // row blocks past the end are clamped; their results are not stored
#pragma unroll
    for (int i = 0; i < NRB; ++i) rbc[i] = rb0 + i < p.nrb ? rb0 + i : p.nrb - 1;
    __amdgpu_buffer_rsrc_t rs_x[NRB], rs_xe[NRB];
#pragma unroll
    for (int i = 0; i < NRB; ++i) {
        rs_x[i] = __builtin_amdgcn_make_buffer_rsrc((void*)(p.xc + (size_t)rbc[i] * C64 * 1024), 0, C64 * 1024, RSRC_FLAGS);
        rs_xe[i] = __builtin_amdgcn_make_buffer_rsrc((void*)(p.xe + (size_t)rbc[i] * CQ * 256), 0, CQ * 256, RSRC_FLAGS);
    }
    const __amdgpu_buffer_rsrc_t rs_p = __builtin_amdgcn_make_buffer_rsrc((void*)(p.pc + (size_t)cb0 * C64 * 1024), 0, NCB * C64 * 1024, RSRC_FLAGS);
    const __amdgpu_buffer_rsrc_t rs_pe = __builtin_amdgcn_make_buffer_rsrc((void*)(p.pe + (size_t)cb0 * CQ * 256), 0, NCB * CQ * 256, RSRC_FLAGS);

    struct Quad { v4i a[NRB][4], b[NCB][4]; int sa[NRB], sb[NCB]; };
    auto load = [&](Quad& t, int quad) {  // (quads and chunks past the end are clamped: fetched, not used)
        const int q = quad < CQ ? quad : CQ - 1;
#pragma unroll
        for (int i = 0; i < NRB; ++i) t.sa[i] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs_xe[i], lane4, q * 256, 0);
#pragma unroll
        for (int j = 0; j < NCB; ++j) t.sb[j] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs_pe, lane4, (j * CQ + q) * 256, 0);
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) {
            const int c = 4 * q + cc < C64 ? 4 * q + cc : C64 - 1;
#pragma unroll
            for (int j = 0; j < NCB; ++j) t.b[j][cc] = __builtin_bit_cast(v4i, (u4)__builtin_amdgcn_raw_buffer_load_b128(rs_p, lane16, (j * C64 + c) * 1024, 0));
#pragma unroll
            for (int i = 0; i < NRB; ++i) t.a[i][cc] = __builtin_bit_cast(v4i, (u4)__builtin_amdgcn_raw_buffer_load_b128(rs_x[i], lane16, c * 1024, 0));
        }
    };
    Quad qd[DEPTH];
#pragma unroll
    for (int i = 0; i < DEPTH; ++i) load(qd[i], i);

    v16f t[NRB][NCB];
#pragma unroll
    for (int i = 0; i < NRB; ++i)
#pragma unroll
        for (int j = 0; j < NCB; ++j) t[i][j] = v16f{0};
    auto chunk = [&](const Quad& c, auto cc_tag) {
        constexpr int CC = decltype(cc_tag)::value;
#pragma unroll
        for (int i = 0; i < NRB; ++i)
#pragma unroll
            for (int j = 0; j < NCB; ++j) {
                const v4i av = c.a[i][CC], bv = c.b[j][CC];
                const v8i a8 = {av[0], av[1], av[2], av[3], 0, 0, 0, 0}, b8 = {bv[0], bv[1], bv[2], bv[3], 0, 0, 0, 0};
                t[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(b8, a8, t[i][j], 4, 4, CC, c.sb[j], CC, c.sa[i]);
            }
    };
    auto multiply = [&](const Quad& c, int quad) {
        chunk(c, std::integral_constant<int, 0>{});
        chunk(c, std::integral_constant<int, 1>{});  // (the number of chunks is even)
        if (4 * quad + 2 < C64) {
            chunk(c, std::integral_constant<int, 2>{});
            chunk(c, std::integral_constant<int, 3>{});
        }
    };
    int q0 = 0;
    for (; q0 + DEPTH <= CQ; q0 += DEPTH) {
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) {
            multiply(qd[i], q0 + i);
            load(qd[i], q0 + i + DEPTH);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int i = 0; i < DEPTH - 1; ++i)
        if (q0 + i < CQ) multiply(qd[i], q0 + i);

    // ---- branch and epilogue as in mx_fwd_tile
    if constexpr (BLK) {
#pragma unroll
        for (int cc = 0; cc < NK; ++cc) {
            v8i lb[NCB];
            int lsc[NCB];
#pragma unroll
            for (int j = 0; j < NCB; ++j) {
                lb[j] = *(const v8i*)(p.l8 + ((size_t)((size_t)(cb0 + j) * NK + cc) * 64 + lane) * 32);
                lsc[j] = *(const int*)((const uint8_t*)p.sl + ((size_t)(cb0 + j) * 64 + lane) * 4);
            }
#pragma unroll
            for (int i = 0; i < NRB; ++i) {
                const v8i ta = *(const v8i*)(p.tq8 + ((size_t)((size_t)rbc[i] * NK + cc) * 64 + lane) * 32);
                const int tsc = *(const int*)((const uint8_t*)p.st + ((size_t)rbc[i] * 64 + lane) * 4);
#pragma unroll
                for (int j = 0; j < NCB; ++j) {
                    if (cc == 0)
                        t[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(lb[j], ta, t[i][j], BFMT, BFMT, 0, lsc[j], 0, tsc);
                    else
                        t[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(lb[j], ta, t[i][j], BFMT, BFMT, 1, lsc[j], 1, tsc);
                }
            }
        }
    }
    constexpr int NKF = BLK ? 0 : NK, NKA = NKF > 0 ? NKF : 1;
    v8i lf[NCB][NKA];
    v4f slv[NCB][4];
#pragma unroll
    for (int j = 0; j < NCB; ++j) {
#pragma unroll
        for (int kk = 0; kk < NKF; ++kk) lf[j][kk] = *(const v8i*)(p.l8 + (size_t)((cb0 + j) * 32 + l32) * p.rp + kk * 64 + half * 32);
        if constexpr (NKF > 0) {
#pragma unroll
            for (int g = 0; g < 4; ++g) slv[j][g] = *(const v4f*)(p.sl + (cb0 + j) * 32 + 8 * g + 4 * half);
        }
    }
    const int rows_valid = p.M - rb0 * 32 < NRB * 32 ? p.M - rb0 * 32 : NRB * 32;
    const __amdgpu_buffer_rsrc_t rs_y = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(p.Y + (size_t)(rb0 * 32) * p.ldy + cb0 * 32), 0, (int)((rows_valid - 1) * p.ldy * 2 + NCB * 64), RSRC_FLAGS);
#pragma unroll
    for (int i = 0; i < NRB; ++i) {
        v8i tf[NKA];
        float stl = 0.f;
        if constexpr (NKF > 0) {
#pragma unroll
            for (int kk = 0; kk < NKF; ++kk) tf[kk] = *(const v8i*)(p.tq8 + (size_t)(rbc[i] * 32 + l32) * p.rp + kk * 64 + half * 32);
            stl = p.st[rbc[i] * 32 + l32];
        }
#pragma unroll
        for (int j = 0; j < NCB; ++j) {
            v16f a2 = {0};
#pragma unroll
            for (int kk = 0; kk < NKF; ++kk)
                a2 = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(lf[j][kk], tf[kk], a2, 0, 0, 0, 0, 0, 0);
            float y[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                if (BLK) y[e] = t[i][j][e];
                else if (NK == 0) y[e] = __fadd_rn(t[i][j][e], 0.f);
                else y[e] = __builtin_fmaf(__fmul_rn(a2[e], stl), slv[j][e >> 2][e & 3], t[i][j][e]);
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const bf16x2 h0 = __builtin_convertvector(f32x2{y[4 * g], y[4 * g + 1]}, bf16x2);
                const bf16x2 h1 = __builtin_convertvector(f32x2{y[4 * g + 2], y[4 * g + 3]}, bf16x2);
                *(v2i*)(stage + l32 * ROW + half * 8 + j * 64 + g * 16) = v2i{__builtin_bit_cast(int, h0), __builtin_bit_cast(int, h1)};
            }
            if (DBG) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int row = (rb0 + i) * 32 + l32, col = (cb0 + j) * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
                    if (row < p.M && p.dbg_y32) p.dbg_y32[(size_t)row * p.N + col] = y[e];
                }
            }
        }
        // read back row-wise (LDS operations of one wavefront complete in order): 4 NCB lanes per row of 64 NCB bytes
        constexpr int LR = 4 * NCB, RP = 64 / LR;
#pragma unroll
        for (int q = 0; q < 32 / RP; ++q) {
            const int row = q * RP + lane / LR, seg = (lane % LR) * 16;
            const v2i lo = *(const v2i*)(stage + row * ROW + seg), hi = *(const v2i*)(stage + row * ROW + seg + 8);
            const v4i o = {lo[0], lo[1], hi[0], hi[1]};
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, o), rs_y, (i * 32 + row) * (int)p.ldy * 2 + seg, 0, 0);
        }
    }
}

template <int NK, bool DBG, bool BLK, int BFMT>
static void mx_fwd_small_launch(MxFwdParams p, int rbt, int cbt, hipStream_t s)
{
    p.tilesN = p.N / 32 / cbt;
    p.tilesM = (p.nrb + rbt - 1) / rbt;
    const dim3 grid((unsigned)(p.tilesM * p.tilesN)), block(64);
    if (rbt == 1) hipLaunchKernelGGL((mx_fwd_small_kernel<NK, DBG, BLK, BFMT, 1, 1>), grid, block, 0, s, p);
    else if (cbt == 1) hipLaunchKernelGGL((mx_fwd_small_kernel<NK, DBG, BLK, BFMT, 2, 1>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((mx_fwd_small_kernel<NK, DBG, BLK, BFMT, 2, 2>), grid, block, 0, s, p);
}

template <int NK, bool BLK, int BFMT = 0>
static void mx_fwd_launch(const MxFwdParams& p, hipStream_t s)
{
    // Small layers, by the number T of 32 x 32 tiles (the device holds 2048 wavefronts of these kernels): one tile to a
    // wavefront while that leaves no SIMD with two, larger ones as the L2 traffic of the operands (2, 1.5 and 1 KB per tile and
    // 64-chunk) begins to count, the 128 x 256 tiles once they occupy enough of the chip.  us, 1 x 1 / 2 x 1 / 2 x 2 / 128 x 256:
    //   T =  108 (   2 x 1152 -> 3456): 3.0 / 3.5 / 4.5 /  7.5        T = 1728 ( 512 x 1152 -> 3456):  6.4 /  5.5 /  5.8 /  7.8
    //   T =  720 ( 300 x 1152 -> 2304): 4.1 / 4.3 / 4.8 /  7.6        T = 2304 (2048 x 4608 -> 1152): 16.9 / 15.8 / 14.7 / 17.5
    //   T = 1080 ( 300 x 1152 -> 3456): 5.4 / 4.9 / 5.5 /  7.8        T = 3500 ( 300 x 2240 -> 11200): 16.4 / 12.1 / 10.7 / 11.7
    //   T =  576 ( 512 x 4608 -> 1152): 6.1 / 7.9 / 9.5 / 16.9        T = 4608 (4096 x 4608 -> 1152): 30.8 / 25.4 / 21.3 / 18.6
    //                                                               T = 3492 (3100 x 4608 -> 1152): 25.5 / 19.8 / 17.3 / 18.0
    const int64_t T = (int64_t)p.nrb * (p.N / 32);
    // More than 80 MB of X codes (a narrow layer): a stream over memory, which the large tiles' requests serve as well or better (37243 x
    // 4608 -> 64: 18.7 us against 17.9).
    if (T <= 3584 && (int64_t)p.nrb * p.C64 <= 80000) {
        const int rbt = T <= 800 ? 1 : 2, cbt = T <= 2000 ? 1 : 2;
        if (p.dbg_y32) mx_fwd_small_launch<NK, true, BLK, BFMT>(p, rbt, cbt, s);
        else mx_fwd_small_launch<NK, false, BLK, BFMT>(p, rbt, cbt, s);
        return;
    }
    dim3 grid((unsigned)(p.n_full + 2 * (p.tilesM * p.tilesN - p.n_full))), block(256);
    if (p.dbg_y32)
        hipLaunchKernelGGL((mx_fwd_kernel<NK, true, BLK, BFMT>), grid, block, 0, s, p);
    else
        hipLaunchKernelGGL((mx_fwd_kernel<NK, false, BLK, BFMT>), grid, block, 0, s, p);
}

static int mx_workgroup_slots() { return 2 * compute_units(); }  // two workgroups (of up to 256 registers per lane) per compute unit

hipError_t launch_fwd_mx(const Dims& d, const uint8_t* packed, const uint8_t* act, int64_t M, uint16_t* Y, int64_t ldy,
                         const lq_fwd_debug* dbg, hipStream_t s)
{
    const PackedLayout pl = packed_layout(d);
    const ActLayout al = act_layout(d, M);
    MxFwdParams p;
    p.xc = act + al.off_xq;
    p.xe = act + al.off_sx;
    p.tq8 = act + al.off_tq;
    p.st = (const float*)(act + al.off_st);
    p.pc = packed + pl.off_pq;
    p.pe = packed + pl.off_sw;
    p.l8 = packed + pl.off_lq;
    p.sl = (const float*)(packed + pl.off_sl);
    p.Y = Y;
    p.ldy = ldy;
    p.M = (int)M;
    p.N = (int)d.N;
    p.C64 = d.C64;
    p.CQ = (d.C64 + 3) / 4;
    p.S = d.C64 / 2;
    p.rp = d.rp;
    p.nrb = (int)(al.Mp / 32);
    p.tilesM = (p.nrb + 3) / 4;
    p.tilesN = (p.N + 255) / 256;
    p.panel = panel_width(p.tilesN, p.C64);
    // Whole generations of the grid (two workgroups per CU) use whole tiles.  A last generation that fills at most a
    // quarter of the slots is cut into half tiles: one per CU instead of one per second CU (16384 x 4608 -> 1152: 57.6 ->
    // 54.3 us, 16384 x 1152 -> 1152: 22.4 -> 21.3 us).
    {
        const int tiles = p.tilesM * p.tilesN, slots = mx_workgroup_slots() & ~7;
        const int rest = tiles % slots;
        p.n_full = (tiles > slots && 4 * rest <= slots) ? tiles - rest : tiles;
    }
    p.dbg_y32 = dbg ? dbg->y32 : nullptr;
    if (d.mxb_elem == 6) {
        switch (p.rp >> 6) {
            case 0: mx_fwd_launch<0, false>(p, s); break;
            case 1: mx_fwd_launch<1, true, 2>(p, s); break;
            default: mx_fwd_launch<2, true, 2>(p, s); break;
        }
    } else if (d.mxb) {  // sl / st hold the E8M0 scale dwords of L / of the intermediate
        switch (p.rp >> 6) {
            case 0: mx_fwd_launch<0, false>(p, s); break;
            case 1: mx_fwd_launch<1, true>(p, s); break;
            default: mx_fwd_launch<2, true>(p, s); break;
        }
    } else {
        switch (p.rp >> 6) {
            case 0: mx_fwd_launch<0, false>(p, s); break;
            case 1: mx_fwd_launch<1, false>(p, s); break;
            default: mx_fwd_launch<2, false>(p, s); break;
        }
    }
    return hipGetLastError();
}

}  // namespace lq
