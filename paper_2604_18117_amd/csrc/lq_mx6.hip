// MXFP6e2 branch of the MX family (App. A.3: E2M3 elements, blocks of 32, E8M0 scale; the 6-bit rows of
// the mixed-precision tables, Section 4.3): offline packing of L and R, the plain views, and the
// activation kernel.  The main product (MXFP4) and the forward kernel are those of lq_mx.hip; only the
// element format of the four branch operands differs (the scaled MFMA takes FP6 at the FP4 rate).
//
// Block exponent: floor(log2 amax) - 2 (2 = largest E2M3 exponent, the same rule as for E2M1, so the main
// and the branch codes of an activation block share one scale byte); elements saturate at +-7.5; codes
// come from the hardware converters (round to nearest even), checked against the oracle's encoder.
#include "lq_internal.h"

namespace lq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef unsigned v6u __attribute__((ext_vector_type(6)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v32bf __attribute__((ext_vector_type(32)));
typedef unsigned short us2 __attribute__((ext_vector_type(2)));

// layouts shared with lq_mx.hip (same formulas there)
__device__ __forceinline__ size_t m6_code_offset(int row, int k, int C64)  // dword holding main code (row, k)
{
    const int blk = row >> 5, c = k >> 6, half = (k & 63) >> 5, d = (k & 31) >> 3;
    return ((size_t)((size_t)blk * C64 + c) * 64 + (row & 31) + 32 * half) * 16 + d * 4;
}
__device__ __forceinline__ size_t m6_scale_offset(int row, int c, int half, int CQ)  // main scale byte of block (row, c, half)
{
    return ((size_t)((size_t)(row >> 5) * CQ + (c >> 2)) * 64 + (row & 31) + 32 * half) * 4 + (c & 3);
}
__device__ __forceinline__ size_t m6_lt_scale_offset(int row, int rb)  // scale byte (row, rank block rb) of le / te
{
    return ((size_t)(row >> 5) * 64 + (row & 31) + 32 * (rb & 1)) * 4 + (rb >> 1);
}
__device__ __forceinline__ size_t m6_re_offset(int j, int kb, int r)  // scale dword (rank row j, K block kb) of re
{
    return ((size_t)((size_t)(kb >> 2) * (r >> 4) + (j >> 4)) * 64 + (j & 15) + 16 * (kb & 3)) * 4;
}
__device__ __forceinline__ uint32_t m6_e8m0_of(float amax)  // floor(log2 amax) - 2 + 127, clamped at 0
{
    const int e = (int)((__float_as_uint(amax) >> 23) & 0xFFu) - 2;
    return (amax == 0.0f || e < 0) ? 0u : (uint32_t)e;
}
__device__ __forceinline__ float m6_e8m0_value(uint32_t E)  // 2^(E-127) as a float (E >= 1), 2^-127 for E = 0
{
    return E ? __uint_as_float(E << 23) : __uint_as_float(0x00400000u);
}

// 32 fp32 values -> 32 E2M3 codes (6 dwords).  The two-source converter interleaves its sources (result
// position 2j holds a[j], 2j+1 holds b[j]), so it is fed the even and the odd elements.
__device__ __forceinline__ v6u fp6_block_from_f32(const float* v, float sc)
{
    v16f a, b;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        a[j] = v[2 * j];
        b[j] = v[2 * j + 1];
    }
    v6u c = __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(a, b, sc);
    // The converter writes its six result registers over several passes while still reading its sources,
    // and the register allocator is not told: without the sources being live past it, it has been seen
    // to place the result on top of the scale register (positions 0 and 1 right, the rest garbage).  The result passes
    // through the statement: one that only reads the sources may be moved ahead of the conversion.
    asm volatile("" : "+v"(c) : "v"(a), "v"(b), "v"(sc));
    return c;
}
__device__ __forceinline__ v6u fp6_block_from_bf16(v32bf h, float sc)
{
    v6u c = __builtin_amdgcn_cvt_scalef32_pk32_fp6_bf16(h, sc);
    asm volatile("" : "+v"(c) : "v"(h), "v"(sc));  // as above
    return c;
}

// ---------------------------------------------------------------------------------------------
// offline packing of the factors: one thread per (row, block of 32)
// ---------------------------------------------------------------------------------------------
// Rows of R, then rows of L.  (Ks: row length of R's source; K: of the layout, a multiple of 128: blocks past the source are zero)
__global__ __launch_bounds__(256) void mx6_pack_rows_kernel(const float* L, const float* R, int N, int K, int Ks, int r, int rp,
                                                            uint8_t* lslots, uint8_t* lscales, uint8_t* rslots, uint8_t* rscales)
{
    size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t nr = (size_t)r * (K >> 5);
    const int mode = idx < nr ? 0 : 1;
    if (mode) idx -= nr;
    const int nb = mode ? r >> 5 : K >> 5, rows = mode ? N : r, src_len = mode ? r : Ks;
    if (idx >= (size_t)rows * nb) return;
    const float* A = mode ? L : R;
    uint8_t *slots = mode ? lslots : rslots, *scales = mode ? lscales : rscales;
    const int row = (int)(idx / nb), b = (int)(idx % nb);
    float v[32];
    float a = 0.f;
    for (int i = 0; i < 32; ++i) {
        v[i] = 32 * b < src_len ? A[(size_t)row * src_len + 32 * b + i] : 0.0f;
        a = fmaxf(a, fabsf(v[i]));
    }
    const uint32_t E = m6_e8m0_of(a);
    v6u c = {0u, 0u, 0u, 0u, 0u, 0u};
    if (a != 0.0f) c = fp6_block_from_f32(v, m6_e8m0_value(E));
    uint32_t* dst = (uint32_t*)(slots + (mode == 0 ? mx6_rq_slot(row, b, r) : mx6_lt_slot(row, b, rp)));
#pragma unroll
    for (int i = 0; i < 6; ++i) dst[i] = c[i];
    dst[6] = 0u;
    dst[7] = 0u;
    if (mode == 0)
        *(uint32_t*)(scales + m6_re_offset(row, b, r)) = 0x7F7F7F00u | E;
    else
        scales[m6_lt_scale_offset(row, b)] = (uint8_t)E;
}

hipError_t launch_pack_rows_mx6(const Dims& d, const float* L, const float* R, uint8_t* packed, hipStream_t s)
{
    const PackedLayout pl = packed_layout(d);
    if (d.r == 0) return hipSuccess;
    const int N = (int)d.N, K = (int)d.K;
    const size_t nt = (size_t)d.r * (K / 32) + (size_t)N * (d.r / 32);
    hipLaunchKernelGGL(mx6_pack_rows_kernel, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, s, L, R, N, K, (int)d.Ks, d.r, d.rp,
                       packed + pl.off_lq, packed + pl.off_sl, packed + pl.off_rq, packed + pl.off_sr);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// plain views
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void mx6_unpack_w_kernel(const uint8_t* packed, PackedLayout pl, int N, int K, int C64, int r,
                                                           int rp, lq_weights_view out)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int CQ = (C64 + 3) >> 2, B = K >> 5, BR = r >> 5;  // K: the caller's (views); C64: chunks of the layout
    if (idx < (size_t)N * K && out.pq) {
        const int n = (int)(idx / K), k = (int)(idx % K);
        const uint32_t w = *(const uint32_t*)(packed + pl.off_pq + m6_code_offset(n, k, C64));
        out.pq[idx] = (int8_t)((w >> (4 * (k & 7))) & 0xFu);
    }
    if (idx < (size_t)N * B && out.pe) {
        const int n = (int)(idx / B), b = (int)(idx % B);
        out.pe[idx] = packed[pl.off_sw + m6_scale_offset(n, b >> 1, b & 1, CQ)];
    }
    if (idx < (size_t)N * r && out.lq) {
        const int n = (int)(idx / r), j = (int)(idx % r);
        out.lq[idx] = (int8_t)fp6_get(packed + pl.off_lq + mx6_lt_slot(n, j >> 5, rp), j & 31);
    }
    if (idx < (size_t)N * BR && out.le) {
        const int n = (int)(idx / BR), b = (int)(idx % BR);
        out.le[idx] = packed[pl.off_sl + m6_lt_scale_offset(n, b)];
    }
    if (idx < (size_t)r * K && out.rq) {
        const int j = (int)(idx / K), k = (int)(idx % K);
        out.rq[idx] = (int8_t)fp6_get(packed + pl.off_rq + mx6_rq_slot(j, k >> 5, r), k & 31);
    }
    if (idx < (size_t)r * B && out.re) {
        const int j = (int)(idx / B), b = (int)(idx % B);
        out.re[idx] = packed[pl.off_sr + m6_re_offset(j, b, r)];
    }
}

hipError_t launch_unpack_weights_mx6(const Dims& d, const uint8_t* packed, const lq_weights_view* out, hipStream_t s)
{
    const PackedLayout pl = packed_layout(d);
    const size_t n = (size_t)(d.N > d.r ? d.N : d.r) * (d.Ks > d.r ? d.Ks : d.r);  // covers N x K, r x K and N x r
    hipLaunchKernelGGL(mx6_unpack_w_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, packed, pl, (int)d.N, (int)d.Ks,
                       d.C64, d.r, d.rp, *out);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void mx6_unpack_a_kernel(const uint8_t* act, ActLayout al, int M, int K, int C64, int r, int rp,
                                                           lq_act_view out)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int CQ = (C64 + 3) >> 2, B = K >> 5, BR = r >> 5;
    if (idx < (size_t)M * K && out.xq) {
        const int m = (int)(idx / K), k = (int)(idx % K);
        const uint32_t w = *(const uint32_t*)(act + al.off_xq + m6_code_offset(m, k, C64));
        out.xq[idx] = (int8_t)((w >> (4 * (k & 7))) & 0xFu);
    }
    if (idx < (size_t)M * B && out.xe) {
        const int m = (int)(idx / B), b = (int)(idx % B);
        out.xe[idx] = act[al.off_sx + m6_scale_offset(m, b >> 1, b & 1, CQ)];
    }
    if (idx < (size_t)M * r && out.tq) {
        const int m = (int)(idx / r), j = (int)(idx % r);
        out.tq[idx] = (int8_t)fp6_get(act + al.off_tq + mx6_lt_slot(m, j >> 5, rp), j & 31);
    }
    if (idx < (size_t)M * BR && out.te) {
        const int m = (int)(idx / BR), b = (int)(idx % BR);
        out.te[idx] = act[al.off_st + m6_lt_scale_offset(m, b)];
    }
}

hipError_t launch_unpack_act_mx6(const Dims& d, const uint8_t* act, int64_t M, const lq_act_view* out, hipStream_t s)
{
    const ActLayout al = act_layout(d, M);
    const size_t n = (size_t)M * (d.Ks > d.r ? d.Ks : d.r);
    hipLaunchKernelGGL(mx6_unpack_a_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, act, al, (int)M, (int)d.Ks,
                       d.C64, d.r, d.rp, *out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// activation kernel.  16 token rows per workgroup; K is walked in chunks of 128 (= one
// v_mfma_scale_f32_16x16x128_f8f6f4), dealt round-robin to the 4 wavefronts; lane (row l%16, q = l/16)
// owns block q of the chunk: its 32 values are one lane's FP4 operand of the main product (16 bytes),
// one lane's FP6 operand of the skinny contraction (24 bytes), and share one scale byte, which the
// lane itself supplies to the instruction.  No scale spans more than a block, so the row is streamed.
// ---------------------------------------------------------------------------------------------
struct Mx6ActParams {
    const void* X;
    int64_t ldx;
    int M, K, C64, C64s, CQ, C128, r, rp;  // K, C64s: the caller's row length and its 64-chunks; C64, C128: of the layout
    const uint8_t* rs;   // R slots
    const uint8_t* re;   // R scale dwords
    uint8_t* xc;
    uint8_t* xe;
    uint8_t* ts;         // intermediate slots
    uint8_t* te;
    int8_t* dbg_xb;
    uint8_t* dbg_xbe;
    float* dbg_T;
    const float* rg;  // reciprocals of the smoothing vector (smoothing variant only)
    BlobTag tag;        // header of the activation blob (written by the first workgroup)
    uint32_t* tag_dst;
};

template <bool BF16>
struct Mx6Block;
template <>
struct Mx6Block<true> {  // 32 bf16 values = 16 dwords
    uint32_t w[16];
    __device__ __forceinline__ void load(const void* X, size_t elem, bool ok)
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v4i a = {0, 0, 0, 0};
            if (ok) a = ((const v4i*)((const uint16_t*)X + elem))[q];
            w[4 * q] = a[0]; w[4 * q + 1] = a[1]; w[4 * q + 2] = a[2]; w[4 * q + 3] = a[3];
        }
    }
    __device__ __forceinline__ float get(int i) const
    {
        return __uint_as_float((i & 1) ? (w[i >> 1] & 0xFFFF0000u) : (w[i >> 1] << 16));
    }
};
template <>
struct Mx6Block<false> {  // 32 fp32 values
    float v[32];
    __device__ __forceinline__ void load(const void* X, size_t elem, bool ok)
    {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            v4i a = {0, 0, 0, 0};
            if (ok) a = ((const v4i*)((const float*)X + elem))[q];
            v[4 * q] = __int_as_float(a[0]); v[4 * q + 1] = __int_as_float(a[1]);
            v[4 * q + 2] = __int_as_float(a[2]); v[4 * q + 3] = __int_as_float(a[3]);
        }
    }
    __device__ __forceinline__ float get(int i) const { return v[i]; }
};

// The 32 values of a block and their scale -> FP4 codes (16 bytes) and FP6 codes (24 bytes).
__device__ __forceinline__ void mx6_codes(const Mx6Block<true>& x, float sc, uint32_t (&pk)[4], v6u& c6, bool main_codes, bool branch)
{
    if (main_codes) {
#define LQ_CVT4B(J) pk[(J) >> 2] = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(pk[(J) >> 2], __builtin_bit_cast(v2bf, x.w[J]), sc, (J) & 3)
        LQ_CVT4B(0); LQ_CVT4B(1); LQ_CVT4B(2); LQ_CVT4B(3); LQ_CVT4B(4); LQ_CVT4B(5); LQ_CVT4B(6); LQ_CVT4B(7);
        LQ_CVT4B(8); LQ_CVT4B(9); LQ_CVT4B(10); LQ_CVT4B(11); LQ_CVT4B(12); LQ_CVT4B(13); LQ_CVT4B(14); LQ_CVT4B(15);
#undef LQ_CVT4B
    }
    if (branch) {
        v32bf h;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const v2bf two = __builtin_bit_cast(v2bf, x.w[j]);
            h[2 * j] = two[0];
            h[2 * j + 1] = two[1];
        }
        c6 = fp6_block_from_bf16(h, sc);
    }
}
__device__ __forceinline__ void mx6_codes(const Mx6Block<false>& x, float sc, uint32_t (&pk)[4], v6u& c6, bool main_codes, bool branch)
{
    if (main_codes) {
#define LQ_CVT4F(J) pk[(J) >> 2] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(pk[(J) >> 2], x.get(2 * (J)), x.get(2 * (J) + 1), sc, (J) & 3)
        LQ_CVT4F(0); LQ_CVT4F(1); LQ_CVT4F(2); LQ_CVT4F(3); LQ_CVT4F(4); LQ_CVT4F(5); LQ_CVT4F(6); LQ_CVT4F(7);
        LQ_CVT4F(8); LQ_CVT4F(9); LQ_CVT4F(10); LQ_CVT4F(11); LQ_CVT4F(12); LQ_CVT4F(13); LQ_CVT4F(14); LQ_CVT4F(15);
#undef LQ_CVT4F
    }
    if (branch) c6 = fp6_block_from_f32(x.v, sc);
}

// BF16IN: element type of X; SM: smoothing variant (X times the stored reciprocals, held as fp32); DBG: parity taps.  The forms, the order of
// T's sums and the way of the operands are those of mxb_act_kernel.
template <bool BF16IN, int NJB, bool SM, int NW, bool DBG, bool SHORT>
__global__ __launch_bounds__(64 * NW, 2) void mx6_act_kernel(Mx6ActParams p)
{
    write_tag(p.tag_dst, p.tag);
    constexpr bool BF16 = BF16IN && !SM;  // representation of a block in registers
    constexpr int NJA = NJB > 0 ? NJB : 1;
    constexpr int NS = 8, SW = NS / NW;  // T is eight sums, over the chunks c = 0 .. 7 mod 8, added in order; SW of them to a wavefront
    __shared__ float s_acc[NS][NJA][64][4];
    __shared__ float s_T[16][NJA * 16 + 1];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, q = lane >> 4;
    const int row = blockIdx.x * 16 + r16;
    const bool row_ok = row < p.M;
    const int C128 = p.C128;
    const int njb = p.r >> 4, jb0 = (int)blockIdx.y * NJB;  // this workgroup's 16-column groups of the rank; the first one stores the main codes
    const bool first = blockIdx.y == 0;
    const int nmy = (C128 - wave + NW - 1) / NW;  // chunks of this wavefront: c = wave + NW * ci, ci < nmy

    Mx6Block<BF16> xs[2];
    const size_t xrow = (size_t)(row_ok ? row : p.M - 1) * p.ldx;
    auto load_x = [&](Mx6Block<BF16>& x, int ci) {  // (no branch around the loads: past the end they are clamped, and not used)
        int b = 4 * (wave + NW * ci) + q;
        b = b < 2 * p.C64s ? b : 2 * p.C64s - 1;
        if constexpr (SM)
            smooth_load<BF16IN, 32>(x.v, p.X, xrow + (size_t)b * 32, p.rg + (size_t)b * 32, true);
        else
            x.load(p.X, xrow + (size_t)b * 32, true);
    };
    v4f acc[SW][NJA];
#pragma unroll
    for (int i = 0; i < SW; ++i)
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) acc[i][jb] = v4f{0.f, 0.f, 0.f, 0.f};

    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    const int rblk = (int)(blockIdx.x >> 1);
    const __amdgpu_buffer_rsrc_t rs_r = __builtin_amdgcn_make_buffer_rsrc((void*)p.rs, 0, (int)((unsigned)C128 * njb * 2048u), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_e = __builtin_amdgcn_make_buffer_rsrc((void*)p.re, 0, C128 * njb * 256, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_c = __builtin_amdgcn_make_buffer_rsrc(p.xc + (size_t)rblk * p.C64 * 1024, 0, p.C64 * 1024, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_s = __builtin_amdgcn_make_buffer_rsrc(p.xe + (size_t)rblk * p.CQ * 256, 0, p.CQ * 256, 0x00020000);
    // the lane's block is K block q & 1 of 64-chunk 2 c + (q >> 1)
    const int off_c = ((row & 31) + 32 * (q & 1)) * 16 + (q >> 1) * 1024, off_s = ((row & 31) + 32 * (q & 1)) * 4 + (q >> 1);

    // One chunk: request its R, code its X, request X of the chunk after the next (refill), multiply.
    auto step = [&](auto slot, int ci, auto refill) {
        constexpr int par = decltype(slot)::value, set = par % SW;  // (the chunks of a slot are those of one sum)
        Mx6Block<BF16>& x = xs[par];
        const int c = wave + NW * ci;
        v8i bv[NJA];
        int bs[NJA];
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) {
            const u4 lo = __builtin_amdgcn_raw_buffer_load_b128(rs_r, lane * 32, (c * njb + jb0 + jb) * 2048, 0);
            const u2 hi = __builtin_amdgcn_raw_buffer_load_b64(rs_r, lane * 32 + 16, (c * njb + jb0 + jb) * 2048, 0);
            bv[jb] = v8i{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], 0, 0};
            bs[jb] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs_e, lane * 4, (c * njb + jb0 + jb) * 256, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        float m = 0.f;
        if constexpr (BF16) {
            us2 m2 = {0, 0};
#pragma unroll
            for (int d = 0; d < 16; ++d) m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(us2, x.w[d] & 0x7FFF7FFFu));
            const uint32_t mm = m2[0] > m2[1] ? m2[0] : m2[1];
            m = __uint_as_float(mm << 16);
        } else {
#pragma unroll
            for (int i = 0; i < 32; ++i) m = fmaxf(m, fabsf(x.get(i)));
        }
        if (!row_ok || 4 * c + q >= 2 * p.C64s) m = 0.f;  // (rows past M and the layout's padding chunk)
        const uint32_t E = m6_e8m0_of(m), nz = m != 0.0f ? ~0u : 0u;  // (a block of zeros has codes 0, also where the zeros are negative)
        uint32_t pk[4] = {0u, 0u, 0u, 0u};
        v6u c6 = {0u, 0u, 0u, 0u, 0u, 0u};
        mx6_codes(x, m6_e8m0_value(E), pk, c6, first, NJB > 0 || DBG);
        if (first) {
            __builtin_amdgcn_raw_buffer_store_b128(u4{pk[0] & nz, pk[1] & nz, pk[2] & nz, pk[3] & nz}, rs_c, off_c, c * 2048, 0);
            __builtin_amdgcn_raw_buffer_store_b8((unsigned char)E, rs_s, off_s, (c >> 1) * 256 + (c & 1) * 2, 0);
        }
#pragma unroll
        for (int i = 0; i < 6; ++i) c6[i] &= nz;
        if constexpr (DBG) {  // (codes taken out at constant positions: an array indexed at run time ends up in the LDS or in scratch)
            if (p.dbg_xb && row_ok && 4 * c + q < 2 * p.C64s) {
                int8_t* o = p.dbg_xb + (size_t)row * p.K + (size_t)c * 128 + q * 32;
#pragma unroll
                for (int i = 0; i < 32; ++i) {
                    const int w = 6 * i / 32, sh = 6 * i % 32;
                    const uint32_t hi = sh > 26 ? c6[w + 1] << (32 - sh) : 0u;
                    o[i] = (int8_t)(((c6[w] >> sh) | hi) & 63u);
                }
            }
            if (p.dbg_xbe && row_ok && 4 * c + q < 2 * p.C64s) p.dbg_xbe[(size_t)row * (p.K >> 5) + 4 * c + q] = (uint8_t)E;
        }
        // (the codes are formed before the slot is filled again: moved down to their use they would keep both rows of X in registers)
        if constexpr (NJB > 0) asm volatile("" : "+v"(c6));
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(refill)::value) {
            load_x(x, ci + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (NJB > 0) {
            const v8i a8 = {(int)c6[0], (int)c6[1], (int)c6[2], (int)c6[3], (int)c6[4], (int)c6[5], 0, 0};
#pragma unroll
            for (int jb = 0; jb < NJB; ++jb)
                acc[set][jb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a8, bv[jb], acc[set][jb], 2, 2, 0, (int)E, 0, bs[jb]);
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
        if (first && 2 * c < 4 * p.CQ) __builtin_amdgcn_raw_buffer_store_b8((unsigned char)127, rs_s, off_s, (c >> 1) * 256 + (c & 1) * 2, 0);
    }
    if (NJB == 0) return;

#pragma unroll
    for (int i = 0; i < SW; ++i)
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) *(v4f*)&s_acc[wave + NW * i][jb][lane][0] = acc[i][jb];
    __syncthreads();
    // the eight sums, a 16-column group and two of a lane's four token rows to a wavefront at a time: lane holds column j = jb*16 + lane%16 of
    // the intermediate for token rows 4*q + i
    for (int task = wave; task < 2 * NJB; task += NW) {
        const int jb = task >> 1, half = task & 1;
        typedef float v2f __attribute__((ext_vector_type(2)));
        v2f o[NS];
#pragma unroll
        for (int w = 0; w < NS; ++w) o[w] = *(const v2f*)&s_acc[w][jb][lane][2 * half];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            float sum = o[0][i];
#pragma unroll
            for (int w = 1; w < NS; ++w) sum = __fadd_rn(sum, o[w][i]);
            s_T[4 * q + 2 * half + i][jb * 16 + r16] = sum;
            const int grow = blockIdx.x * 16 + 4 * q + 2 * half + i;
            if (DBG && grow < p.M && p.dbg_T) p.dbg_T[(size_t)grow * p.r + (jb0 + jb) * 16 + r16] = sum;
        }
    }
    __syncthreads();
    // re-quantise: one thread per (token row, block of 32 along the rank); the first workgroup adds the blocks that pad the rank to a
    // multiple of 64: zero codes and scale 2^0
    const int own = NJB / 2, pad = first ? (p.rp >> 5) - (p.r >> 5) : 0;
    if (tid < 16 * (own + pad)) {
        const int trow = tid & 15, b = tid >> 4;
        const int blk = b < own ? (jb0 >> 1) + b : (p.r >> 5) + b - own;
        const int grow = blockIdx.x * 16 + trow;
        float v[32];
        float a = 0.f;
        v6u c6 = {0u, 0u, 0u, 0u, 0u, 0u};
        uint32_t E = 127u;
        if (b < own) {
            for (int i = 0; i < 32; ++i) {
                v[i] = s_T[trow][32 * b + i];
                a = fmaxf(a, fabsf(v[i]));
            }
            E = m6_e8m0_of(a);
            if (a != 0.0f) c6 = fp6_block_from_f32(v, m6_e8m0_value(E));
        }
        uint4* dst = (uint4*)(p.ts + mx6_lt_slot(grow, blk, p.rp));
        dst[0] = make_uint4(c6[0], c6[1], c6[2], c6[3]);
        dst[1] = make_uint4(c6[4], c6[5], 0u, 0u);
        p.te[m6_lt_scale_offset(grow, blk)] = (uint8_t)E;
    }
}

template <bool BF16, int NJB, bool SM, int NW, bool DBG>
static hipError_t mx6_act_launch3(const Mx6ActParams& p, dim3 grid, hipStream_t s)
{
    if (!DBG && p.C128 <= mxb_act_short(NW))
        hipLaunchKernelGGL((mx6_act_kernel<BF16, NJB, SM, NW, false, true>), grid, dim3(64 * NW), 0, s, p);
    else
        hipLaunchKernelGGL((mx6_act_kernel<BF16, NJB, SM, NW, DBG, false>), grid, dim3(64 * NW), 0, s, p);
    return hipGetLastError();
}
template <bool BF16, int NJB, bool SM, bool DBG>
static hipError_t mx6_act_launch2(const Mx6ActParams& p, int64_t Mp, hipStream_t s)
{
    const dim3 rows((unsigned)(Mp / 16));
    switch (mxb_act_form(Mp, p.C128, NJB, !BF16 || SM)) {
        case 4: return mx6_act_launch3<BF16, NJB, SM, 4, DBG>(p, rows, s);
        case 8: return mx6_act_launch3<BF16, NJB, SM, 8, DBG>(p, rows, s);
        default: return mx6_act_launch3<BF16, NJB < 2 ? NJB : 2, SM, 8, DBG>(p, dim3(rows.x, NJB < 2 ? 1 : NJB / 2), s);
    }
}
template <bool BF16, int NJB, bool SM>
static hipError_t mx6_act_launch(const Mx6ActParams& p, int64_t Mp, hipStream_t s)
{
    return p.dbg_xb || p.dbg_xbe || p.dbg_T ? mx6_act_launch2<BF16, NJB, SM, true>(p, Mp, s) : mx6_act_launch2<BF16, NJB, SM, false>(p, Mp, s);
}
template <bool BF16, bool SM>
static hipError_t mx6_act_rank2(const Mx6ActParams& p, int64_t Mp, hipStream_t s)
{
    switch (p.r) {
        case 0: return mx6_act_launch<BF16, 0, SM>(p, Mp, s);
        case 32: return mx6_act_launch<BF16, 2, SM>(p, Mp, s);
        case 64: return mx6_act_launch<BF16, 4, SM>(p, Mp, s);
        case 96: return mx6_act_launch<BF16, 6, SM>(p, Mp, s);
        default: return mx6_act_launch<BF16, 8, SM>(p, Mp, s);
    }
}
template <bool BF16>
static hipError_t mx6_act_rank(const Mx6ActParams& p, int64_t Mp, hipStream_t s)
{
    return p.rg ? mx6_act_rank2<BF16, true>(p, Mp, s) : mx6_act_rank2<BF16, false>(p, Mp, s);
}

hipError_t launch_quantize_act_mx6(const Dims& d, int x_dtype, const uint8_t* packed, const void* X, int64_t M,
                                   int64_t ldx, uint8_t* act, const lq_act_debug* dbg, hipStream_t s)
{
    const PackedLayout pl = packed_layout(d);
    const ActLayout al = act_layout(d, M);
    Mx6ActParams p;
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
    p.rs = packed + pl.off_rq;
    p.re = packed + pl.off_sr;
    p.xc = act + al.off_xq;
    p.xe = act + al.off_sx;
    p.ts = act + al.off_tq;
    p.te = act + al.off_st;
    p.dbg_xb = dbg ? dbg->xb : nullptr;
    p.dbg_xbe = dbg ? dbg->xbe : nullptr;
    p.dbg_T = dbg ? dbg->T : nullptr;
    p.rg = d.smooth ? (const float*)(packed + pl.off_rg) : nullptr;
    return x_dtype == LQ_BF16 ? mx6_act_rank<true>(p, al.Mp, s) : mx6_act_rank<false>(p, al.Mp, s);
}

}  // namespace lq
