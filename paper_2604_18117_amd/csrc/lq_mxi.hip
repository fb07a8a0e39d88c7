// MXI family: integer MX formats (App. A.3: "MXINT4 and MXINT8 quantize to a signed int4 and int8
// format", blocks of 32, E8M0 scale; the integer rows of the mixed-precision tables, Section 4.3).
//
//   main   : X and P = W - deq(Q2 L) deq(Q2 R) in MXINT4, blocks of 32 along K
//   branch : X and X R^T in MXINT8, L and R in MXINT8 or MXINT4, blocks of 32 along the contraction axis
//
// Element of width b: integer code c in [-(2^(b-1)-1), 2^(b-1)-1], value c * 2^(s-(b-2)) with the
// block's shared exponent s = floor(log2 amax) (E8M0 byte s + 127; 0 for an all-zero block).
//
// Main product: the 4-bit codes are fed to v_mfma_scale_f32_32x32x64_f8f6f4 as 6-bit fields s00mmm, the
// E2M3 (FP6) patterns of +-m/8, which run at twice the rate of 8-bit operands; the instruction applies
// both E8M0 block scales itself, so there is NO vector-ALU dequantisation: the stored scale byte is
// s + 127 + 1 (2^-3 * 2^(s+1) = 2^(s-2), one code step).  Inside a block every product and partial sum is
// exact; across blocks the matrix core accumulates in fp32.
// Branch: a power-of-two block scale times an integer of at most 7 bits is exactly a bf16 value, so
// the dequantised MXINT elements are stored as bf16 and both contractions run on the bf16 MFMA with
// fp32 accumulation (products exact); the rank-r expansion accumulates straight into the main
// product's accumulators.
//
// Contract beyond the general one: block maxima are zero or lie in [2^-100, 2^120].
#include "lq_pack.h"

#include <type_traits>

namespace lq {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned short us2 __attribute__((ext_vector_type(2)));

// ---- layouts -------------------------------------------------------------------------------
// Main codes, "fragment order": [block of 32 rows][64-chunk of K][lane = row%32 + 32*h][16 bytes].
// With 6-bit operands lane (row, h) of the scaled MFMA holds block h of its row's chunk, code i at bits 6i .. 6i+5 of six
// dwords; two of the six bits of every field are zero, so three dwords (16 codes) are kept in two (f6_pack / f6_unpack):
// bytes 0..7 hold k = 32h .. 32h+15, bytes 8..15 the other half of the block.
__device__ __forceinline__ size_t mxi_frag_offset(int row, int k, int C64)  // the 8 bytes that hold code (row, k)
{
    return ((size_t)((size_t)(row >> 5) * C64 + (k >> 6)) * 64 + (row & 31) + 32 * ((k >> 5) & 1)) * 16 + ((k >> 4) & 1) * 8;
}
// Three dwords of fields have 64 bits in use (sign, three of magnitude per code).  a keeps the 22 of dword 0 in place and, where that
// has its zeros, 10 bits of dword 2; b the 21 of dword 1 and the other 11 of dword 2: no bit changes its position, two and
// an and-or apart the three dwords come back in four instructions (expanding nibbles to bytes takes six for 16 codes).
constexpr uint32_t F6_A = 0xE79E79E7u, F6_B = 0x79E79E79u;  // the bits of dwords 0 and 1 that fields use
__device__ __forceinline__ uint2 f6_pack(uint32_t d0, uint32_t d1, uint32_t d2) { return make_uint2(d0 | (d2 & ~F6_A), d1 | (d2 & ~F6_B)); }
__device__ __forceinline__ void f6_unpack(uint32_t a, uint32_t b, uint32_t (&d)[3])
{
    d[0] = a & F6_A;
    d[1] = b & F6_B;
    d[2] = (a & ~F6_A) | (b & ~F6_B);
}
__device__ __forceinline__ int f6_code(const uint8_t* at, int e)  // code e (0..15) of the 8 bytes at `at`
{
    uint32_t d[3];
    f6_unpack(*(const uint32_t*)at, *(const uint32_t*)(at + 4), d);
    const int bit = 6 * e;
    const uint64_t lo = d[bit >> 5] | (bit < 64 ? (uint64_t)d[(bit >> 5) + 1] << 32 : 0ull);
    const uint32_t c = (uint32_t)(lo >> (bit & 31)) & 63u;
    return (c & 32u) ? -(int)(c & 7u) : (int)(c & 7u);
}

// The 6-bit fields of values |v| <= 7 sc / 8 (clamped before): the hardware FP6 converter applied to v / sc, round to nearest even,
// on the grid of E2M3's subnormals = one code step.  The converters write their six result registers over several passes while still
// reading their sources, and the register allocator is not told: the sources are kept live past them so that the result
// cannot land on them.  (The result passes through the statement: one that only reads the sources may be moved ahead.)
typedef unsigned int v6u __attribute__((ext_vector_type(6)));
__device__ __forceinline__ v6u f6_from_bf16(const uint32_t (&w)[16], float sc)  // bf16 pairs, in order
{
    typedef unsigned int v16u __attribute__((ext_vector_type(16)));
    typedef __bf16 v32bf __attribute__((ext_vector_type(32)));
    const v16u h = {w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7], w[8], w[9], w[10], w[11], w[12], w[13], w[14], w[15]};
    v6u c = __builtin_amdgcn_cvt_scalef32_pk32_fp6_bf16(__builtin_bit_cast(v32bf, h), sc);
    asm volatile("" : "+v"(c) : "v"(h), "v"(sc));
    return c;
}
// 16 values: the sources' upper halves are not defined, the codes they give (result dwords 3..5) not used
__device__ __forceinline__ uint2 f6_pack16_bf16(const uint32_t (&w)[8], float sc)
{
    typedef unsigned int v8u __attribute__((ext_vector_type(8)));
    typedef __bf16 v32bf __attribute__((ext_vector_type(32)));
    const v8u h8 = {w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7]};
    const auto h = __builtin_shufflevector(h8, h8, 0, 1, 2, 3, 4, 5, 6, 7, -1, -1, -1, -1, -1, -1, -1, -1);
    v6u c = __builtin_amdgcn_cvt_scalef32_pk32_fp6_bf16(__builtin_bit_cast(v32bf, h), sc);
    asm volatile("" : "+v"(c) : "v"(h), "v"(sc));
    return f6_pack(c[0], c[1], c[2]);
}
__device__ __forceinline__ uint2 f6_pack16_f32(const float (&v)[16], float sc)  // (the converter interleaves its two sources)
{
    typedef float v8f __attribute__((ext_vector_type(8)));
    const v8f ev = {v[0], v[2], v[4], v[6], v[8], v[10], v[12], v[14]}, od = {v[1], v[3], v[5], v[7], v[9], v[11], v[13], v[15]};
    const v16f a = __builtin_shufflevector(ev, ev, 0, 1, 2, 3, 4, 5, 6, 7, -1, -1, -1, -1, -1, -1, -1, -1);
    const v16f b = __builtin_shufflevector(od, od, 0, 1, 2, 3, 4, 5, 6, 7, -1, -1, -1, -1, -1, -1, -1, -1);
    v6u c = __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(a, b, sc);
    asm volatile("" : "+v"(c) : "v"(a), "v"(b), "v"(sc));
    return f6_pack(c[0], c[1], c[2]);
}
// bf16 pair with both magnitudes at most those of `lim` (7 code steps, in both halves)
__device__ __forceinline__ uint32_t clamp_pair(uint32_t w, uint32_t lim)
{
    const uint32_t m = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(us2, w & 0x7FFF7FFFu), __builtin_bit_cast(us2, lim)));
    return (w & 0x80008000u) | m;
}
// 7 code steps (1.75 * 2^s) and the converter's scale 2^(s+1) of a block with exponent field `field`; blocks below 2^-125 have codes 0
__device__ __forceinline__ uint32_t f6_limit(uint32_t field) { return field >= 2u ? (field << 23) | 0x00600000u : 0u; }  // as fp32 bits
__device__ __forceinline__ float f6_scale(uint32_t field) { return __uint_as_float((field + 1u) << 23); }
// Scale bytes: one dword per (block of 32 rows, quad of 64-chunks, lane); lane (row, h) holds the
// scale of K block h of its row, byte c%4 for chunk c (the instruction's op_sel picks the byte).
__device__ __forceinline__ size_t mxi_scale_offset(int row, int c, int blk, int CQ)
{
    return ((size_t)((size_t)(row >> 5) * CQ + (c >> 2)) * 64 + (row & 31) + 32 * blk) * 4 + (c & 3);
}
// bf16 element (rank row j, k) of the dequantised R, operand order of v_mfma_f32_16x16x32_bf16 in the
// activation kernel: [64-chunk][j/16][u = (k%16)/8][lane = j%16 + 16*((k%64)/16)][k%8]
__device__ __forceinline__ size_t mxi_rq_offset(int j, int k, int r)
{
    const int c = k >> 6, q = (k & 63) >> 4, u = (k & 15) >> 3;
    return ((((size_t)((size_t)c * (r >> 4) + (j >> 4)) * 2 + u) * 64 + (j & 15) + 16 * q) * 8 + (k & 7)) * 2;
}
// bf16 element (row, rank index j) of the dequantised L / intermediate, operand order of
// v_mfma_f32_32x32x16_bf16: [block of 32 rows][j/16][lane = row%32 + 32*((j%16)/8)][j%8]
__device__ __forceinline__ size_t mxi_lt_offset(int row, int j, int rp)
{
    return (((size_t)((size_t)(row >> 5) * (rp >> 4) + (j >> 4)) * 64 + (row & 31) + 32 * ((j >> 3) & 1)) * 8 + (j & 7)) * 2;
}

__device__ __forceinline__ float bf16_value(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// shared exponent byte of a block: floor(log2 amax) + 127 clamped at 0 = the fp32 exponent field
__device__ __forceinline__ uint32_t exp_field(float amax) { return (__float_as_uint(amax) >> 23) & 0xFFu; }

// One element: code = clamp(rne(v * 2^(frac - s)), -qmax, qmax) with s = field - 127.
__device__ __forceinline__ int mxint_code(float v, uint32_t field, int bits)
{
    const float qmax = (float)((1 << (bits - 1)) - 1);
    const float q = rintf(ldexpf(v, (bits - 2) - ((int)field - 127)));
    return (int)fminf(fmaxf(q, -qmax), qmax);
}
__device__ __forceinline__ float mxint_value(int code, uint32_t field, int bits)
{
    return ldexpf((float)code, ((int)field - 127) - (bits - 2));
}

// ---------------------------------------------------------------------------------------------
// offline packing
// ---------------------------------------------------------------------------------------------
// Factors: one thread per (row, block of 32).  Rows of R, blocks along K, then rows of L, blocks along the rank.
// Stores the dequantised elements as bf16 in operand order and the E8M0 bytes row-major.
__global__ __launch_bounds__(256) void mxi_pack_rows_kernel(const float* L, const float* R, int N, int K, int bits, int r, int rp,
                                                            uint8_t* lvals, uint8_t* lebytes, uint8_t* rvals, uint8_t* rebytes)
{
    size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t nr = (size_t)r * (K >> 5);
    const int mode = idx < nr ? 0 : 1;
    if (mode) idx -= nr;
    const int nb = mode ? r >> 5 : K >> 5, rows = mode ? N : r;
    if (idx >= (size_t)rows * nb) return;
    uint8_t *vals = mode ? lvals : rvals, *ebytes = mode ? lebytes : rebytes;
    const int row = (int)(idx / nb), b = (int)(idx % nb);
    const float* v = (mode ? L : R) + (size_t)row * (mode ? r : K) + 32 * b;
    float a = 0.f;
    for (int i = 0; i < 32; ++i) a = fmaxf(a, fabsf(v[i]));
    const uint32_t field = exp_field(a);
    ebytes[(size_t)row * nb + b] = (uint8_t)field;
    for (int i = 0; i < 32; ++i) {
        const float val = mxint_value(mxint_code(v[i], field, bits), field, bits);
        const uint16_t h = (uint16_t)(__float_as_uint(val) >> 16);  // at most 7 significant bits: exact
        const size_t off = mode == 0 ? mxi_rq_offset(row, 32 * b + i, r) : mxi_lt_offset(row, 32 * b + i, rp);
        *(uint16_t*)(vals + off) = h;
    }
}

// Residual of a 64-chunk (two blocks of 32): MXINT4 codes and scale bytes.  Factors: the dequantised elements (exact in
// bf16) or, from_q = 0, as given.
template <bool FROMQ>
struct PackMxiResidual {
    using Raw = std::conditional_t<FROMQ, uint2, pack_v4f>;
    const float *L, *R;
    const uint8_t *lv, *rv;
    uint8_t *pq, *pe;
    int K, r, rp;
    __device__ void lhat(int n, int j, int q, float (&v)[4]) const
    {
        if constexpr (FROMQ) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint4 c = *(const uint4*)(lv + mxi_lt_offset(n, j + 8 * h, rp));  // 8 elements; the lane's are q and q + 4
                v[2 * h] = bf16_value((uint16_t)((q & 2 ? c.y : c.x) >> (16 * (q & 1))));
                v[2 * h + 1] = bf16_value((uint16_t)((q & 2 ? c.w : c.z) >> (16 * (q & 1))));
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = L[(size_t)n * r + j + 4 * i + q];
        }
    }
    __device__ Raw rload(int j, int k) const
    {
        if constexpr (FROMQ) return *(const Raw*)(rv + mxi_rq_offset(j, k, r));
        else return *(const Raw*)(R + (size_t)j * K + k);
    }
    static constexpr double UNIT = 1.0;
    static constexpr bool PAD_CHECK = true;
    __device__ void rval(const Raw& x, float (&v)[4]) const
    {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if constexpr (FROMQ) v[t] = bf16_value((uint16_t)((t < 2 ? x.x : x.y) >> (16 * (t & 1))));
            else v[t] = x[t];
        }
    }
    __device__ void encode(int n, int c, const float (&P)[1][16], int q) const
    {
        float a = pack_amax(P[0]);
        a = fmaxf(a, __shfl_xor(a, 16));  // lanes q, q ^ 1 hold the block
        const uint32_t field = exp_field(a);
        uint32_t d[3] = {0u, 0u, 0u};
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const uint32_t f = f6_field(mxint_code(P[0][e], field, 4));
            const int bit = 6 * e, at = bit >> 5, sh = bit & 31;
            d[at] |= f << sh;
            if (sh > 26) d[at + 1] |= f >> (32 - sh);
        }
        *(uint2*)(pq + mxi_frag_offset(n, c * 64 + 16 * q, K >> 6)) = f6_pack(d[0], d[1], d[2]);
        if ((q & 1) == 0) pe[mxi_scale_offset(n, c, q >> 1, ((K >> 6) + 3) >> 2)] = (uint8_t)(field + 1);
    }
};

struct MxiPackedPtrs {
    uint8_t *pq, *pe, *lv, *le, *rv, *re;
};
static MxiPackedPtrs mxi_packed_ptrs(const Dims& d, uint8_t* packed)
{
    const PackedLayout pl = packed_layout(d);
    return {packed + pl.off_pq, packed + pl.off_sw, packed + pl.off_lq, packed + pl.off_sl, packed + pl.off_rq,
            packed + pl.off_sr};
}

hipError_t launch_pack_mxi(const Dims& d, int from_q, const float* W, const float* L, const float* R, uint8_t* packed,
                           hipStream_t s)
{
    const MxiPackedPtrs pp = mxi_packed_ptrs(d, packed);
    const int N = (int)d.N, K = (int)d.K;
    PackFill fill;
    fill.n = 0;
    if (d.C64 % 4) fill.add(pp.pe, (size_t)(N / 32) * ((d.C64 + 3) / 4) * 256, 0x7F7F7F7Fu);        // padding chunks of the last quad: 2^0
    if (d.smooth) fill.add(packed + packed_layout(d).off_rg, (size_t)K * 4, 0x3F800000u);            // reciprocals start at 1
    const hipError_t e = launch_pack_fill(fill, s);
    if (e != hipSuccess) return e;
    if (d.r > 0) {
        const size_t nt = (size_t)d.r * (K / 32) + (size_t)N * (d.r / 32);
        hipLaunchKernelGGL(mxi_pack_rows_kernel, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, s, L, R, N, K, d.bw_bits, d.r, d.rp, pp.lv,
                           pp.le, pp.rv, pp.re);
    }
    auto residual = [&](auto fq) {
        return pack_residual<1>(hipGetLastError(), PackMxiResidual<decltype(fq)::value>{L, R, pp.lv, pp.rv, pp.pq, pp.pe, K, d.r, d.rp}, W, N, K, d.r, d.C64,
                                packed, make_tag(d, LQ_BLOB_PACKED, 0), s);
    };
    return from_q && d.r > 0 ? residual(std::true_type{}) : residual(std::false_type{});
}

// ---------------------------------------------------------------------------------------------
// plain views
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ int8_t mxi_code_of(uint16_t bf, uint32_t field, int bits)
{
    return (int8_t)(int)ldexpf(bf16_value(bf), (bits - 2) - ((int)field - 127));  // exact: the value is on the grid
}

__global__ __launch_bounds__(256) void mxi_unpack_w_kernel(MxiPackedPtrs pp, int N, int K, int r, int rp, int bits,
                                                           lq_weights_view out)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int C64 = K >> 6, CQ = (C64 + 3) >> 2, B = K >> 5, BR = r >> 5;
    if (idx < (size_t)N * K && out.pq) {
        const int n = (int)(idx / K), k = (int)(idx % K);
        out.pq[idx] = (int8_t)f6_code(pp.pq + mxi_frag_offset(n, k, C64), k & 15);
    }
    if (idx < (size_t)N * B && out.pe) {
        const int n = (int)(idx / B), b = (int)(idx % B);
        out.pe[idx] = (uint8_t)(pp.pe[mxi_scale_offset(n, b >> 1, b & 1, CQ)] - 1);
    }
    if (idx < (size_t)N * r && out.lq) {
        const int n = (int)(idx / r), j = (int)(idx % r);
        out.lq[idx] = mxi_code_of(*(const uint16_t*)(pp.lv + mxi_lt_offset(n, j, rp)), pp.le[(size_t)n * BR + (j >> 5)], bits);
    }
    if (idx < (size_t)N * BR && out.le) out.le[idx] = pp.le[idx];
    if (idx < (size_t)r * K && out.rq) {
        const int j = (int)(idx / K), k = (int)(idx % K);
        out.rq[idx] = mxi_code_of(*(const uint16_t*)(pp.rv + mxi_rq_offset(j, k, r)), pp.re[(size_t)j * B + (k >> 5)], bits);
    }
    if (idx < (size_t)r * B && out.re) out.re[idx] = pp.re[idx];
}

hipError_t launch_unpack_weights_mxi(const Dims& d, const uint8_t* packed, const lq_weights_view* out, hipStream_t s)
{
    const MxiPackedPtrs pp = mxi_packed_ptrs(d, const_cast<uint8_t*>(packed));
    const size_t n = (size_t)(d.N > d.r ? d.N : d.r) * (d.K > d.r ? d.K : d.r);  // covers N x K, r x K and N x r
    hipLaunchKernelGGL(mxi_unpack_w_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, pp, (int)d.N, (int)d.K,
                       d.r, d.rp, d.bw_bits, *out);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void mxi_unpack_a_kernel(const uint8_t* act, ActLayout al, int M, int K, int r, int rp,
                                                           lq_act_view out)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int C64 = K >> 6, CQ = (C64 + 3) >> 2, B = K >> 5, BR = r >> 5;
    if (idx < (size_t)M * K && out.xq) {
        const int m = (int)(idx / K), k = (int)(idx % K);
        out.xq[idx] = (int8_t)f6_code(act + al.off_xq + mxi_frag_offset(m, k, C64), k & 15);
    }
    if (idx < (size_t)M * B && out.xe) {
        const int m = (int)(idx / B), b = (int)(idx % B);
        out.xe[idx] = (uint8_t)(act[al.off_sx + mxi_scale_offset(m, b >> 1, b & 1, CQ)] - 1);
    }
    if (idx < (size_t)M * r && out.tq) {
        const int m = (int)(idx / r), j = (int)(idx % r);
        out.tq[idx] = mxi_code_of(*(const uint16_t*)(act + al.off_tq + mxi_lt_offset(m, j, rp)),
                                  act[al.off_st + (size_t)m * BR + (j >> 5)], 8);
    }
    if (idx < (size_t)M * BR && out.te) out.te[idx] = act[al.off_st + idx];
}

hipError_t launch_unpack_act_mxi(const Dims& d, const uint8_t* act, int64_t M, const lq_act_view* out, hipStream_t s)
{
    const ActLayout al = act_layout(d, M);
    const size_t n = (size_t)M * (d.K > d.r ? d.K : d.r);
    hipLaunchKernelGGL(mxi_unpack_a_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, act, al, (int)M, (int)d.K,
                       d.r, d.rp, *out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// activation kernel.  Every scale is local to a block of 32, so there is no pass over the whole row before coding: the row
// is streamed and K is not limited by the register file.  A workgroup is ROWG x 4 wavefronts; wavefront (rg, w) owns RPW
// groups of 16 token rows and the chunks c = w mod 4 of K; lane l works on row l%16 of each group and on the 16-value
// quarter l/16 of a 64-chunk.
//
// What bounds it: the dequantised R (2 r K bytes) passes through every workgroup, at rank 128 several times the bytes of X.
// Large batches (ROWG = 2) copy each super-step of 4 chunks of it to LDS once per workgroup, directly and one super-step
// ahead, and a fragment read from there serves RPW groups of rows; small ones (ROWG = 1) have each wavefront read its own
// chunks' fragments from the L2 while it codes X.  X is requested two super-steps ahead.  Chain of 16384 x 1152 -> 4608 -> 1152 at
// rank 128: first activation step 31.5 -> 20.4 us, step from codes 60.7 -> 31.7 us (without LDS and with R requested a fragment
// ahead); 64 rows of 4608, rank 128: 19.5 -> 17.6 us.  (Eight wavefronts along K take 16.2 us there, but then T is another sum.)
// T is defined as four sums, each over the chunks c = w mod 4 in ascending order, added in the order of w: every form forms
// these, so a token's codes do not depend on the batch it is in, and a hand-off gives the bits of the two-call path.
// ---------------------------------------------------------------------------------------------
struct MxiActParams {
    const void* X;
    const int8_t* cb;    // from-codes variant: M x K MXINT8 codes of a quantized hand-off, row-major
    const uint8_t* cbe;  // ... and their E8M0 bytes, M x K/32
    int64_t ldx;
    int M, Mp, K, C64, CQ, r, rp;
    const uint8_t* rv;
    uint8_t* xq;
    uint8_t* xe;
    uint8_t* tv;
    uint8_t* te;
    int8_t* dbg_xb;
    uint8_t* dbg_xbe;
    float* dbg_T;
    const float* rg;  // reciprocals of the smoothing vector (smoothing variant only)
    BlobTag tag;        // header of the activation blob (written by the first workgroup)
    uint32_t* tag_dst;
};

template <bool BF16>
struct MxiChunk;
template <>
struct MxiChunk<true> {  // 16 bf16 values = 8 dwords
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
struct MxiChunk<false> {  // 16 fp32 values
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

// Round v to the MXINT8 grid of a block with exponent field `field`: multiples of 2^(s-6), ties to
// even, clamped to +-127 steps.  Adding 1.5 * 2^(17+s) leaves exactly that granularity in the sum's
// significand (|v| < 2^(s+1)); the result has at most 7 significant bits, so its upper 16 bits are
// the exact bf16 value.
__device__ __forceinline__ float mxint8_round(float v, uint32_t field)
{
    const float magic = __uint_as_float(((field + 17u) << 23) | 0x00400000u);
    const float lim = __uint_as_float((field << 23) | 0x007E0000u);  // 127 * 2^(s-6) = 1.984375 * 2^s
    const float q = __fsub_rn(__fadd_rn(v, magic), magic);
    return fminf(fmaxf(q, -lim), lim);
}
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi)  // upper halves of two floats
{
    return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}

// BF16IN: element type of X; SM: smoothing variant (X times the stored reciprocals, held as fp32).
// FROMC: the branch half of the step alone, from the MXINT8 codes of a quantized hand-off (the producing layer's
// epilogue has already written this layer's main codes and scales): 16 code bytes and a scale byte replace the 16 values
// of X, code * 2^(s-6) is the dequantised bf16 element; the contraction and the re-quantisation are the same code.
template <bool BF16IN, int NJB, bool SM, bool FROMC, int RPW, int ROWG, bool DBG, bool SPLIT>
__global__ __launch_bounds__(ROWG * 256, 2) void mxi_act_kernel(MxiActParams p)
{
    write_tag(p.tag_dst, p.tag);
    constexpr bool BF16 = BF16IN && !SM;  // representation of a chunk in registers
    constexpr int NJA = NJB > 0 ? NJB : 1;
    constexpr int KW = 4;                        // wavefronts along K: part of T's order of summation, the same in every form
    constexpr int NG = RPW * ROWG;               // groups of 16 rows per workgroup
    constexpr int RCHUNK = NJB * 2048;           // bytes of this workgroup's columns of R per 64-chunk
    constexpr int RBUF = KW * RCHUNK;            // ... per super-step
    constexpr bool STAGE = NJB > 0 && ROWG > 1;  // R goes through LDS
    constexpr int RED = NG * KW * NJA * 1024;    // partial sums of the wavefronts of a row group
    constexpr int LDS_BYTES = NJB == 0 ? 16 : STAGE && 2 * RBUF > RED ? 2 * RBUF : RED;
    __shared__ __attribute__((aligned(16))) uint8_t lds[LDS_BYTES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = wid & (KW - 1), rgrp = wid / KW;
    const int r16 = lane & 15, kq = lane >> 4;
    const int row0 = blockIdx.x * (16 * NG) + rgrp * (16 * RPW);  // first row of this wavefront
    const int C64 = p.C64;
    const int Mp = p.Mp;
    const int nss = (C64 + KW - 1) / KW;
    // SPLIT (small batches): a workgroup per 16 rows and 32 columns of the rank (grid.y); the first stores the main codes.  Every block of the intermediate
    // is 32 columns, and no sum runs across them.  (A flag of the kernel's: decided at run time, the forms without it were up to 6 % slower, smoothed fp32 rows above all.)
    if (SPLIT && row0 >= Mp) return;  // (grid.x is rounded up)
    const int jb0 = SPLIT ? (int)blockIdx.y * NJB : 0, rchunk = SPLIT ? p.r * 128 : RCHUNK;  // bytes of all of R per 64-chunk
    const bool first = !SPLIT || blockIdx.y == 0;

    // Rows past M count as zeros, chunks past the end are clamped and not used: the loads are unconditional (the wait
    // below counts them).  Groups past Mp (the last workgroup) are not stored.
    struct XSet { MxiChunk<BF16> g[RPW]; };
    XSet xs[2];
    auto load_x = [&](XSet& st, int ss) {
        int c = KW * ss + wave;
        c = c < C64 ? c : C64 - 1;
#pragma unroll
        for (int g = 0; g < RPW; ++g) {
            MxiChunk<BF16>& ch = st.g[g];
            int row = row0 + 16 * g + r16;
            row = row < p.M ? row : p.M - 1;
            const size_t koff = (size_t)c * 64 + kq * 16;
            if constexpr (FROMC) {  // 16 code bytes in w[0..3], the block's scale byte in w[4]
                static_assert(!FROMC || (BF16IN && !SM), "the from-codes variant reuses the packed chunk registers");
                const v4i a = *(const v4i*)(p.cb + (size_t)row * p.K + koff);
                ch.w[0] = a[0]; ch.w[1] = a[1]; ch.w[2] = a[2]; ch.w[3] = a[3];
                ch.w[4] = p.cbe[(size_t)row * (p.K >> 5) + (koff >> 5)];
            } else if constexpr (SM)
                smooth_load<BF16IN, 16>(ch.v, p.X, (size_t)row * p.ldx + koff, p.rg + koff, true);
            else
                ch.load(p.X, (size_t)row * p.ldx + koff, true);
        }
    };
    // R of super-step ss -> LDS buffer: lane l of an instruction writes 16 bytes at 16 l behind the wave-uniform address
    constexpr int RI = RBUF / 1024 / (KW * ROWG);  // 1 KB instructions per wavefront, all of one chunk
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    auto chunk_r = [&](int c) {  // R of one chunk (a descriptor for all of it would end at 4 GB: K = 2^24 at rank 128 has as much)
        return __builtin_amdgcn_make_buffer_rsrc((void*)(p.rv + (size_t)c * rchunk + jb0 * 2048), 0, RCHUNK, 0x00020000);
    };
    auto load_r = [&](int ss) {
        if constexpr (STAGE) {
            static_assert(RCHUNK / 1024 % RI == 0, "a wavefront's share of a super-step lies in one chunk");
            const int c = KW * ss + wid * RI / (RCHUNK / 1024);    // (a chunk past the end is clamped: fetched, not used)
            const __amdgpu_buffer_rsrc_t rs_r = chunk_r(c < C64 ? c : C64 - 1);
#pragma unroll
            for (int i = 0; i < RI; ++i) {
                const int piece = wid * RI + i;              // of RBUF / 1024
                uint8_t* dst = lds + (ss & 1) * RBUF + piece * 1024;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_r, (__attribute__((address_space(3))) void*)dst, 16, lane * 16,
                                                         (piece % (RCHUNK / 1024)) * 1024, 0, 0);
            }
        }
    };

    v4f acc[RPW][NJA];
#pragma unroll
    for (int g = 0; g < RPW; ++g)
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) acc[g][jb] = v4f{0.f, 0.f, 0.f, 0.f};

    // Fragment pairs of R, RD ahead of their products: an LDS round trip is longer than a pair's products, an L2 round trip much
    // longer.  Without STAGE they are requested before X is coded, up to rank 64 a super-step ahead (ROLL; us without / with it: rank 32,
    // 4096 x 4608 16.5 / 14.7, rank 64 18.7 / 15.8, smoothed fp32 rank 32, 8192 x 2240 21.0 / 18.5, though 64 x 2240 10.1 / 11.0;
    // but rank 128, 64 x 1152 7.1 / 7.5, smoothed bf16 rank 64, 4096 x 2240 12.4 / 13.9, from codes rank 64, 2 x 4608 7.6 / 10.3).
    constexpr bool ROLL = !STAGE && !FROMC && (!SM || !BF16IN) && NJB <= 4;
    constexpr int RD = STAGE ? (NJA < 3 ? NJA : 3) : NJA < 4 ? NJA : 4;
    v4i rf[RD][2];
    auto read_pair = [&](int ss, int jb) {
        const int c = KW * ss + wave;  // (past the end: clamped, fetched, not used)
        const __amdgpu_buffer_rsrc_t rs_r = chunk_r(c < C64 ? c : C64 - 1);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if constexpr (STAGE)
                rf[jb % RD][u] = *(const v4i*)(lds + (ss & 1) * RBUF + wave * RCHUNK + lane * 16 + (jb * 2 + u) * 1024);
            else
                rf[jb % RD][u] = __builtin_bit_cast(v4i, (u4)__builtin_amdgcn_raw_buffer_load_b128(rs_r, lane * 16, (jb * 2 + u) * 1024, 0));
        }
    };

    // One super-step: request R of the next one, code this one's X, request X of the one after the next, multiply.
    auto step = [&](XSet& st, int ss) {
        const int c = KW * ss + wave;
        const bool have = c < C64;  // wave-uniform
        load_r(ss + 1);
        if constexpr (NJB > 0 && !STAGE && !ROLL) {
#pragma unroll
            for (int jb = 0; jb < RD; ++jb) read_pair(ss, jb);
        }
        __builtin_amdgcn_sched_barrier(0);
        v4i au[RPW][2];
#pragma unroll
        for (int g = 0; g < RPW; ++g) {
            MxiChunk<BF16> ch = st.g[g];
            const int row = row0 + 16 * g + r16;
            const bool row_ok = row < p.M;
            // zeros: a row past M (only in the last workgroup); ROLL: a chunk past the end, whose products are formed (a branch around
            // them would end the compiler's count of the loads in flight)
            if ((row0 + 16 * g + 16 > p.M && !row_ok) || (ROLL && !have)) {
                if constexpr (BF16) {
#pragma unroll
                    for (int d = 0; d < 8; ++d) ch.w[d] = 0u;
                } else {
#pragma unroll
                    for (int d = 0; d < 16; ++d) ch.v[d] = 0.f;
                }
            }
            uint32_t field;
            if constexpr (FROMC) {
                field = ch.w[4];
            } else {
                float m = 0.f;
                if constexpr (BF16) {
                    // |bf16| is monotonic in its low 15 bits: packed unsigned 16-bit max, two values per op
                    us2 m2 = {0, 0};
#pragma unroll
                    for (int d = 0; d < 8; ++d) m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(us2, ch.w[d] & 0x7FFF7FFFu));
                    const uint32_t mm = m2[0] > m2[1] ? m2[0] : m2[1];
                    m = __uint_as_float(mm << 16);
                } else {
#pragma unroll
                    for (int i = 0; i < 16; ++i) m = fmaxf(m, fabsf(ch.get(i)));
                }
                const float ab = max_xor16(m);  // block of 32 = lanes kq, kq ^ 1
                field = exp_field(ab);
                // ---- main codes: MXINT4, clamp(rne(x * 2^(2-s)), +-7) by the FP6 converter
                const float sc = f6_scale(field);
                uint2 pk = {0u, 0u};
                if (!first) {
                } else if constexpr (BF16) {
                    const uint32_t l1 = f6_limit(field), l2 = l1 | (l1 >> 16);
                    uint32_t cw[8];
#pragma unroll
                    for (int d = 0; d < 8; ++d) cw[d] = clamp_pair(ch.w[d], l2);
                    pk = f6_pack16_bf16(cw, sc);
                } else {
                    const float lim = __uint_as_float(f6_limit(field));
                    float cv[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i) cv[i] = __builtin_amdgcn_fmed3f(ch.get(i), -lim, lim);
                    pk = f6_pack16_f32(cv, sc);
                }
                // lane (row, kq): half kq & 1 of block kq >> 1 of the chunk
                uint8_t* dst = p.xq + ((size_t)((size_t)(row >> 5) * C64 + c) * 64 + (row & 31) + 32 * (kq >> 1)) * 16 + (kq & 1) * 8;
                if (first && have && row0 + 16 * g < Mp) {
                    *(uint2*)dst = pk;
                    if ((kq & 1) == 0) p.xe[mxi_scale_offset(row, c, kq >> 1, p.CQ)] = (uint8_t)(field + 1u);
                }
            }
            if (NJB > 0) {
                // ---- branch: MXINT8 of the same block, kept as dequantised bf16
                float v8[16];
                if constexpr (FROMC) {  // code * 2^(s-6): exact, at most 7 significant bits
                    const float step = field >= 7u ? __uint_as_float((field - 6u) << 23) : 0.0f;
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        v8[i] = __fmul_rn((float)(int)(int8_t)((ch.w[i >> 2] >> (8 * (i & 3))) & 0xFFu), step);
                } else {
#pragma unroll
                    for (int i = 0; i < 16; ++i) v8[i] = mxint8_round(ch.get(i), field);
                }
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int d = 0; d < 4; ++d) au[g][u][d] = (int)bf16_pair(v8[8 * u + 2 * d], v8[8 * u + 2 * d + 1]);
                if (DBG && p.dbg_xb && row_ok && have) {
                    uint32_t cb[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        cb[i >> 2] |= ((uint32_t)(int)ldexpf(v8[i], 6 - ((int)field - 127)) & 0xFFu) << (8 * (i & 3));
                    *(v4i*)(p.dbg_xb + (size_t)row * p.K + c * 64 + kq * 16) = v4i{(int)cb[0], (int)cb[1], (int)cb[2], (int)cb[3]};
                }
                if (DBG && p.dbg_xbe && row_ok && have && (kq & 1) == 0) p.dbg_xbe[(size_t)row * (p.K >> 5) + 2 * c + (kq >> 1)] = (uint8_t)field;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (STAGE || NJB == 0) {
            load_x(st, ss + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (NJB > 0) {
            if (ROLL || have) {
                if constexpr (STAGE) {
#pragma unroll
                    for (int jb = 0; jb < RD; ++jb) read_pair(ss, jb);
                }
#pragma unroll
                for (int jb = 0; jb < NJB; ++jb) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int g = 0; g < RPW; ++g)
                            acc[g][jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, au[g][u]),
                                                                                 __builtin_bit_cast(v8bf, rf[jb % RD][u]), acc[g][jb], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    if (jb + RD < NJB) read_pair(ss, jb + RD);
                    else if constexpr (ROLL) read_pair(ss + 1, jb + RD - NJB);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (STAGE) {
                // this wavefront's share of R for the next super-step has arrived once at most the loads issued after it are
                // outstanding: X of super-step ss + 2, at least two per row group
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * RPW) : "memory");
            } else {
                load_x(st, ss + 2);
            }
        }
    };
    load_x(xs[0], 0);
    __builtin_amdgcn_sched_barrier(0);
    load_r(0);
    if constexpr (NJB > 0 && ROLL) {
#pragma unroll
        for (int jb = 0; jb < RD; ++jb) read_pair(0, jb);
    }
    __builtin_amdgcn_sched_barrier(0);
    load_x(xs[1], 1);
    if constexpr (STAGE) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * RPW) : "memory");
    }
    int ss = 0;
    for (; ss + 1 < nss; ss += 2) {
        step(xs[0], ss);
        step(xs[1], ss + 1);
    }
    if (ss < nss) step(xs[0], ss);
    if constexpr (!FROMC) {   // padding chunks of the last quad: their scale bytes must be valid E8M0 values (2^0)
        const int c = C64 + wave;
        if (first && c < 4 * p.CQ && (kq & 1) == 0) {
#pragma unroll
            for (int g = 0; g < RPW; ++g)
                if (row0 + 16 * g < Mp) p.xe[mxi_scale_offset(row0 + 16 * g + r16, c, kq >> 1, p.CQ)] = (uint8_t)127;
        }
    }
    if constexpr (NJB > 0) {
        const int BR = p.r >> 5;
        constexpr int NBB = (NJB + 1) / 2;   // blocks of 32 along the rank
        if constexpr (STAGE) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the last super-step's request (clamped, unused) has landed
            __syncthreads();
        }
        v4f* red = (v4f*)lds;                // [row group][wavefront][jb][lane]
#pragma unroll
        for (int g = 0; g < RPW; ++g)
#pragma unroll
            for (int jb = 0; jb < NJB; ++jb) red[(((rgrp * RPW + g) * KW + wave) * NJB + jb) * 64 + lane] = acc[g][jb];
        __syncthreads();
        // one (row group, block of 32 of the rank) per wavefront at a time: sum over the wavefronts, re-quantise to
        // MXINT8; the lane holds columns (2 bb + h) * 16 + lane%16 of the intermediate for token rows 4*kq + i
        for (int task = wid; task < NG * NBB; task += KW * ROWG) {
            const int g = task / NBB, bb = task - g * NBB;
            const int rbase = blockIdx.x * (16 * NG) + 16 * g;
            if (rbase >= Mp) continue;
            float T[2][4];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                v4f sum = red[(g * KW * NJB + 2 * bb + h) * 64 + lane];
#pragma unroll
                for (int w = 1; w < KW; ++w) {
                    const v4f o = red[((g * KW + w) * NJB + 2 * bb + h) * 64 + lane];
#pragma unroll
                    for (int i = 0; i < 4; ++i) sum[i] = __fadd_rn(sum[i], o[i]);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    T[h][i] = sum[i];
                    const int grow = rbase + 4 * kq + i;
                    if (DBG && grow < p.M && p.dbg_T) p.dbg_T[(size_t)grow * p.r + (jb0 + 2 * bb + h) * 16 + r16] = sum[i];
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float tm = fmaxf(fabsf(T[0][i]), fabsf(T[1][i]));
                tm = max_row16(tm);
                const int grow = rbase + 4 * kq + i;
                const uint32_t field = exp_field(tm);
                if (r16 == 0) p.te[(size_t)grow * BR + (jb0 >> 1) + bb] = (uint8_t)field;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float v = mxint8_round(T[h][i], field);
                    *(uint16_t*)(p.tv + mxi_lt_offset(grow, (jb0 + 2 * bb + h) * 16 + r16, p.rp)) = (uint16_t)(__float_as_uint(v) >> 16);
                }
            }
        }
    }
}

// Rows per workgroup: 64 (two groups of 32, R through LDS), 32 (two groups of 16, R through LDS) or 16 (each wavefront reads its R
// from the L2).  All sum T in the same order, so a token's bits depend on none of this.  The forms with R in LDS run one workgroup to
// a compute unit: they pay where the rounds they take are nearly full and there is R enough (rank times K) for its traffic to
// count; the step from codes, which reads half as much and codes nothing, is earlier at that point.
// Measured (us, bf16 X, act / from codes; 64-, 32-, 16-row form):
//   16384 x 4608, rank 128: 50.4 / 31.7, 61.5 / 45.4, 65.8 / 55.6      16384 x 4608, rank  64: 42.0 / 24.1, 40.0 / 28.5, 47.1 / 37.3
//   16384 x 1152, rank 128: 20.4 / 12.8, 24.2 / 15.6, 21.5 / 16.3      16384 x 1152, rank  32: 15.8 /  7.5, 14.3 /  7.9, 13.3 /  8.6
//   10240 x 4608, rank 128: 48.3 / 30.3, 58.6 / 43.0, 49.9 / 42.2       8192 x 4608, rank 128: 47.7 / 30.0, 32.1 / 23.8, 35.5 / 29.6
//    8192 x 1152, rank 128: 18.9 / 12.1, 12.7 /  8.5, 12.1 /  9.4       8192 x 2240, rank  32: 21.5 /   - , 14.9 /   - , 12.2 /   -
//    1024 x 4608, rank 128: 46.3 / 27.9, 29.9 / 19.1, 18.1 / 14.0        300 x 1152, rank  64: 14.6 /  8.1,  9.5 /  5.9,  6.5 /  4.6
static int mxi_act_rows(int r, int64_t K, int64_t Mp, bool from_codes)
{
    const int64_t cus = compute_units();
    auto full = [&](int rows) {  // the share of its rounds that a form of one workgroup per compute unit fills
        const int64_t wgs = (Mp + rows - 1) / rows;
        return (double)wgs / (double)((wgs + cus - 1) / cus * cus);
    };
    const bool large = r * K >= 128 * 1152, one_round = Mp <= 32 * cus;  // (of the 32-row form)
    if (r < 32) return 16;
    if (from_codes) {
        if (one_round) return r >= 64 && full(32) >= 0.6 ? 32 : 16;
        if (full(64) >= (large && r >= 64 ? 0.55 : 0.7)) return 64;
        return full(32) >= 0.75 ? 32 : 16;
    }
    if (!large) return 16;
    if (r <= 64) return !one_round && full(32) >= 0.85 ? 32 : 16;
    if (full(64) >= (r * K >= 96 * 4096 ? 0.7 : 0.8)) return 64;
    return one_round && full(32) >= 0.6 && K >= 2240 ? 32 : 16;
}

template <bool BF16, int NJB, bool SM, bool FROMC, bool DBG>
static hipError_t mxi_act_launch2(const MxiActParams& p, hipStream_t s)
{
    switch (mxi_act_rows(p.r, p.K, p.Mp, FROMC)) {
        case 64: hipLaunchKernelGGL((mxi_act_kernel<BF16, NJB, SM, FROMC, 2, 2, DBG, false>), dim3((unsigned)((p.Mp + 63) / 64)), dim3(512), 0, s, p); break;
        case 32: hipLaunchKernelGGL((mxi_act_kernel<BF16, NJB, SM, FROMC, 1, 2, DBG, false>), dim3((unsigned)(p.Mp / 32)), dim3(512), 0, s, p); break;
        default: {
            // A workgroup per 32 columns of the rank while compute units are left over for them: R passes through a compute unit each (us, one / this:
            // 300 x 1152 rank 128 7.1 / 5.1, 64 x 4608 rank 128 18.9 / 10.6, rank 64 12.9 / 12.3, 300 x 2240 fp32 rank 96 11.8 / 8.3, 2000 x 1152 rank 64
            // 7.3 / 6.3; with two workgroups to a compute unit 2000 x 1152 rank 128 8.7 / 8.1, 3000 x 2240 rank 64 11.4 / 12.0, 3000 x 512 4.5 / 5.3).
            // Whole eights of row groups, so that the workgroups of a group are on one of the 8 XCDs and X is read from memory once (smoothed 600 x 6144 rank 64
            // 24.8 us without, 20.8 unsplit, 18.6 so; 1500 x 4608 rank 64 13.7, 13.2, 11.8; 783 x 4608 rank 128 14.0, 17.0, 11.8).
            constexpr int NB = NJB / 2;
            const unsigned groups = (unsigned)(p.Mp / 16);
            if constexpr (NB > 1) {
                if ((int64_t)groups * NB <= compute_units()) {
                    const dim3 grid(groups > 8 ? (groups + 7) / 8 * 8 : groups, NB);
                    hipLaunchKernelGGL((mxi_act_kernel<BF16, 2, SM, FROMC, 1, 1, DBG, true>), grid, dim3(256), 0, s, p);
                    break;
                }
            }
            hipLaunchKernelGGL((mxi_act_kernel<BF16, NJB, SM, FROMC, 1, 1, DBG, false>), dim3(groups), dim3(256), 0, s, p);
            break;
        }
    }
    return hipGetLastError();
}
template <bool BF16, int NJB, bool SM, bool FROMC>
static hipError_t mxi_act_launch(const MxiActParams& p, hipStream_t s)
{
    if constexpr (!FROMC) {
        if (p.dbg_xb || p.dbg_xbe || p.dbg_T) return mxi_act_launch2<BF16, NJB, SM, FROMC, true>(p, s);
    }
    return mxi_act_launch2<BF16, NJB, SM, FROMC, false>(p, s);
}
template <bool BF16, bool SM, bool FROMC>
static hipError_t mxi_act_rank(const MxiActParams& p, hipStream_t s)
{
    switch (p.r) {
        case 0: return mxi_act_launch<BF16, 0, SM, FROMC>(p, s);
        case 32: return mxi_act_launch<BF16, 2, SM, FROMC>(p, s);
        case 64: return mxi_act_launch<BF16, 4, SM, FROMC>(p, s);
        case 96: return mxi_act_launch<BF16, 6, SM, FROMC>(p, s);
        default: return mxi_act_launch<BF16, 8, SM, FROMC>(p, s);
    }
}

// The branch half of the activation step from the codes of a quantized hand-off (see mxi_act_kernel, FROMC).
hipError_t launch_branch_from_codes_mxi(const Dims& d, const uint8_t* packed, const uint8_t* codes, int64_t M, uint8_t* act,
                                        hipStream_t s)
{
    const PackedLayout pl = packed_layout(d);
    const ActLayout al = act_layout(d, M);
    MxiActParams p = {};
    p.tag = make_tag(d, LQ_BLOB_ACT, M);
    p.tag_dst = (uint32_t*)act;
    p.cb = (const int8_t*)codes;
    p.cbe = codes + handoff_codes_bytes(d, M);
    p.M = (int)M;
    p.Mp = (int)al.Mp;
    p.K = (int)d.K;
    p.C64 = d.C64;
    p.CQ = (d.C64 + 3) / 4;
    p.r = d.r;
    p.rp = d.rp;
    p.rv = packed + pl.off_rq;
    p.xq = act + al.off_xq;
    p.xe = act + al.off_sx;
    p.tv = act + al.off_tq;
    p.te = act + al.off_st;
    if (d.r == 0) return hipSuccess;  // the next layer has no branch: its blob is complete after the producing layer's epilogue
    return mxi_act_rank<true, false, true>(p, s);
}

hipError_t launch_quantize_act_mxi(const Dims& d, int x_dtype, const uint8_t* packed, const void* X, int64_t M,
                                   int64_t ldx, uint8_t* act, const lq_act_debug* dbg, hipStream_t s)
{
    const PackedLayout pl = packed_layout(d);
    const ActLayout al = act_layout(d, M);
    MxiActParams p;
    p.tag = make_tag(d, LQ_BLOB_ACT, M);
    p.tag_dst = (uint32_t*)act;
    p.X = X;
    p.cb = nullptr;
    p.cbe = nullptr;
    p.ldx = ldx;
    p.M = (int)M;
    p.Mp = (int)al.Mp;
    p.K = (int)d.K;
    p.C64 = d.C64;
    p.CQ = (d.C64 + 3) / 4;
    p.r = d.r;
    p.rp = d.rp;
    p.rv = packed + pl.off_rq;
    p.xq = act + al.off_xq;
    p.xe = act + al.off_sx;
    p.tv = act + al.off_tq;
    p.te = act + al.off_st;
    p.dbg_xb = dbg ? dbg->xb : nullptr;
    p.dbg_xbe = dbg ? dbg->xbe : nullptr;
    p.dbg_T = dbg ? dbg->T : nullptr;
    p.rg = d.smooth ? (const float*)(packed + pl.off_rg) : nullptr;
    if (d.smooth) return x_dtype == LQ_BF16 ? mxi_act_rank<true, true, false>(p, s) : mxi_act_rank<false, true, false>(p, s);
    return x_dtype == LQ_BF16 ? mxi_act_rank<true, false, false>(p, s) : mxi_act_rank<false, false, false>(p, s);
}

// ---------------------------------------------------------------------------------------------
// forward: 1 x 4 wavefronts per workgroup, 128 x 64 outputs per wavefront, one 64-chunk of K per step
// ---------------------------------------------------------------------------------------------
struct MxiFwdParams {
    const uint8_t* xq;
    const uint8_t* xe;
    const uint8_t* tv;
    const uint8_t* pq;
    const uint8_t* pe;
    const uint8_t* lv;
    uint16_t* Y;
    int64_t ldy;
    int M, N, C64, CQ, nrb;
    int tilesM, tilesN, panel;
    float* dbg_y32;
    // quantized hand-off to a next MXINT layer whose K is this layer's N (HO variant): its main codes and scale bytes
    // (sections of its activation blob) and its MXINT8 branch codes and scale bytes (row-major, for the from-codes step)
    uint8_t* ho_xq;
    uint8_t* ho_xe;
    int8_t* ho_cb;
    uint8_t* ho_cbe;
    int ho_C64, ho_CQ;
    BlobTag ho_tag;      // header of the consumer's activation blob
    uint32_t* ho_tag_dst;
};

__device__ __forceinline__ v8i mxi_expand(v4i p)  // 32 packed codes -> the lane's FP6 operand (six dwords; FP6 mode reads no more)
{
    uint32_t lo[3], hi[3];
    f6_unpack((uint32_t)p[0], (uint32_t)p[1], lo);
    f6_unpack((uint32_t)p[2], (uint32_t)p[3], hi);
    typedef int v6i __attribute__((ext_vector_type(6)));
    const v6i o = {(int)lo[0], (int)lo[1], (int)lo[2], (int)hi[0], (int)hi[1], (int)hi[2]};
    return __builtin_shufflevector(o, o, 0, 1, 2, 3, 4, 5, -1, -1);
}

// MXINT8 codes of eight values (bf16 pairs) by one fused multiply-add each: scaling by a power of two is exact, so fma(x, 2^-step, magic)
// rounds the scaled value to the nearest integer (ties to even) in one step -- the same integer the
// activation kernel reaches by rounding on the block's grid and scaling afterwards -- and leaves it in
// the low mantissa bits of the magic number.  Clamping after the rounding equals clamping before it.
__device__ __forceinline__ void mxi_handoff_codes8(const uint32_t* w, const float to8, uint32_t* c8)
{
    uint32_t ub[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float x = __uint_as_float((e & 1) ? (w[e >> 1] & 0xFFFF0000u) : (w[e >> 1] << 16));
        // 1.5 * 2^23 + code, code in [-127, 127]: the low byte is the two's-complement MXINT8 code
        ub[e] = __float_as_uint(__builtin_amdgcn_fmed3f(__builtin_fmaf(x, to8, 12582912.0f), 12582785.0f, 12583039.0f));
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t lo = __builtin_amdgcn_perm(ub[4 * h + 1], ub[4 * h], 0x0c0c0400u);      // bytes 0 of two dwords
        const uint32_t hi = __builtin_amdgcn_perm(ub[4 * h + 3], ub[4 * h + 2], 0x04000c0cu);  // ... in the upper half
        c8[h] = lo | hi;
    }
}
__device__ __forceinline__ float mxint8_unscale(uint32_t field) { return field >= 7u ? __uint_as_float((260u - field) << 23) : 0.0f; }  // 2^(6-s)

// Hand-off codes of 8 consecutive channels (k0 = this layer's channel = the next layer's k) of one token, given as bf16: a
// block of 32 of the next layer's K axis is the 4 lanes that differ in the two low lane bits.  Codes as in the activation
// kernel: shared exponent from the block maximum, MXINT4 main codes (6-bit fields), MXINT8 branch codes.
__device__ __forceinline__ void mxi_handoff_emit(const MxiFwdParams& p, const v4i v, const int row, const int k0)
{
    const uint32_t w[4] = {(uint32_t)v[0], (uint32_t)v[1], (uint32_t)v[2], (uint32_t)v[3]};
    us2 m2 = {0, 0};
#pragma unroll
    for (int d = 0; d < 4; ++d) m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(us2, w[d] & 0x7FFF7FFFu));
    const uint32_t mm = m2[0] > m2[1] ? m2[0] : m2[1];
    float am = __uint_as_float(mm << 16);
    am = max_dpp<0xB1>(am);  // quad_perm [1,0,3,2], then [2,3,0,1]
    am = max_dpp<0x4E>(am);
    const uint32_t field = exp_field(am);
    uint32_t c8[2];
    mxi_handoff_codes8(w, mxint8_unscale(field), c8);
    // the neighbour's 8 values are the other half of the 16 codes that share 8 bytes: both lanes convert all of them, each stores a dword
    const uint32_t l1 = f6_limit(field), l2 = l1 | (l1 >> 16);
    const bool odd = (k0 >> 3) & 1;
    uint32_t cw[8];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const uint32_t own = clamp_pair(w[d], l2), other = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xF, 0xF, true);
        cw[d] = odd ? other : own;
        cw[4 + d] = odd ? own : other;
    }
    const uint2 pk = f6_pack16_bf16(cw, f6_scale(field));
    if (row < p.nrb * 32) {
        *(uint32_t*)(p.ho_xq + mxi_frag_offset(row, k0, p.ho_C64) + (odd ? 4 : 0)) = odd ? pk.y : pk.x;
        *(uint2*)(p.ho_cb + (size_t)row * p.N + k0) = make_uint2(c8[0], c8[1]);
        if ((k0 & 31) == 0) {
            p.ho_xe[mxi_scale_offset(row, k0 >> 6, (k0 >> 5) & 1, p.ho_CQ)] = (uint8_t)(field + 1u);
            p.ho_cbe[(size_t)row * (p.N >> 5) + (k0 >> 5)] = (uint8_t)field;
            // padding chunks of the next layer's last quad: valid E8M0 bytes (2^0), written with the last real chunk
            if ((k0 >> 6) == p.ho_C64 - 1)
                for (int c = p.ho_C64; c < 4 * p.ho_CQ; ++c) p.ho_xe[mxi_scale_offset(row, c, (k0 >> 5) & 1, p.ho_CQ)] = (uint8_t)127;
        }
    }
}

// The same from the registers of mxi_fwd_kernel: a row block of 32 tokens and 64 channels (one chunk of the next layer's K); lane (row, h)
// holds channels 16 h .. 16 h + 15 of both blocks of 32 as bf16 pairs.  Eight row-swap instructions leave it block h whole, the unit of
// the consumer's operands: the block's maximum and both kinds of codes need no other lane; 16 bytes of main codes (1 KB contiguous per
// wavefront), 32 of branch codes, and the block's scale bytes.
__device__ __forceinline__ void mxi_handoff_rows(const MxiFwdParams& p, const uint32_t (&w)[2][8], const int rb, const int cb0, const int lane)
{
    const int half = lane >> 5, row = rb * 32 + (lane & 31), c = cb0 >> 1;
    uint32_t x[16], cw[16];
#pragma unroll
    for (int d = 0; d < 8; ++d) {  // the upper half of w[0] and the lower half of w[1] change places
        const auto sw = __builtin_amdgcn_permlane32_swap(w[0][d], w[1][d], false, false);
        x[d] = sw[0];
        x[8 + d] = sw[1];
    }
    us2 m2 = {0, 0};
#pragma unroll
    for (int d = 0; d < 16; ++d) m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(us2, x[d] & 0x7FFF7FFFu));
    const uint32_t field = exp_field(__uint_as_float((uint32_t)(m2[0] > m2[1] ? m2[0] : m2[1]) << 16));
    const float to8 = mxint8_unscale(field);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t c8[4];
        mxi_handoff_codes8(&x[8 * h], to8, c8);
        mxi_handoff_codes8(&x[8 * h + 4], to8, c8 + 2);
        *(v4i*)(p.ho_cb + (size_t)row * p.N + (cb0 + half) * 32 + 16 * h) = v4i{(int)c8[0], (int)c8[1], (int)c8[2], (int)c8[3]};
    }
    const uint32_t l1 = f6_limit(field), l2 = l1 | (l1 >> 16);
#pragma unroll
    for (int d = 0; d < 16; ++d) cw[d] = clamp_pair(x[d], l2);
    const v6u f6 = f6_from_bf16(cw, f6_scale(field));
    const uint2 lo = f6_pack(f6[0], f6[1], f6[2]), hi = f6_pack(f6[3], f6[4], f6[5]);
    *(v4i*)(p.ho_xq + ((size_t)((size_t)rb * p.ho_C64 + c) * 64 + lane) * 16) = v4i{(int)lo.x, (int)lo.y, (int)hi.x, (int)hi.y};
    p.ho_xe[mxi_scale_offset(row, c, half, p.ho_CQ)] = (uint8_t)(field + 1u);
    p.ho_cbe[(size_t)row * (p.N >> 5) + cb0 + half] = (uint8_t)field;
    // padding chunks of the next layer's last quad: valid E8M0 bytes (2^0), written with the last real chunk
    if (c == p.ho_C64 - 1)
        for (int cc = p.ho_C64; cc < 4 * p.ho_CQ; ++cc) p.ho_xe[mxi_scale_offset(row, cc, half, p.ho_CQ)] = (uint8_t)127;
}

namespace mxif {
constexpr int RBT = 4, NBUF = 4;              // row blocks of a tile, LDS buffers of the activation stream (one 64-chunk each)
constexpr int EPI_ROW = 144, EPI_WAVE = 32 * EPI_ROW;
constexpr int SLOT = 2064;                    // of one staged operand: [lane][16 B], [lane][8 B]; the stride keeps the compiler from merging reads of two slots
constexpr int LDS_MAIN = NBUF * RBT * SLOT;   // [buffer][row block]
constexpr int LDS_BYTES = LDS_MAIN > 4 * EPI_WAVE ? LDS_MAIN : 4 * EPI_WAVE;
}  // namespace mxif

// One tile of 128 rows: WN = 4 wavefronts side by side of 128 x 64 outputs each, or, for a last column of tiles of at most 128 channels,
// 2 x 2 wavefronts of 64 x 64 (side by side two of the four would have no columns).  Inside the K loop the 6-bit matrix
// rate (512 cycles a step for the two wavefronts of a SIMD) is the largest of several: a step takes 790 (K = 4608) to 870 cycles (K = 1152), with
// 24 instructions that unpack codes and 9 KB through the LDS per wavefront; around it instruction latency.  Codes as 8-bit operands (FP8
// subnormals) took 1024 cycles of the matrix core a step: us with those / as it is, rank 64: 16384 x 1152 -> 3456 68.3 / 64.5, 5000 x 2240 -> 6720
// 63.9 / 53.9, 16384 x 1152 -> 1152 23.8 / 21.9, rank 128 16384 x 4608 -> 1152 68.7 / 59.8, 16384 x 1152 -> 4608 with hand-off 105.5 / 98.1 (38 -> 30
// thousand cycles a tile: prologue 3.0, loop 15.2, branch 4.7, epilogue with the hand-off 7.2).  The fences in the loop
// hold every load two steps ahead of its use: left to itself the compiler sinks them to the end of their step and waits for all of
// them in the next (us without the fences / without the narrow tiles / as it is: 16384 x 4608 -> 1152 rank 128 66.4 / 64.5 / 59.8, 16384 x
// 1152 -> 3456 69.7 / 63.2 / 64.5, 16384 x 1152 -> 1152 22.9 / 22.8 / 21.9, 5000 x 2240 -> 6720 56.5 / 54.3 / 53.9).
// NK16 = 16-deep chunks of the rank: 0 | 2 | 4 | 6 | 8.  HO: quantized hand-off (Section 4.5): the epilogue also emits
// the next layer's activation codes from the bf16 values it has just formed; Y itself is optional then.
template <int NK16, bool DBG, bool HO, int WN>
__device__ __forceinline__ void mxi_fwd_tile(const MxiFwdParams& p, uint8_t* lds, const int rb0, const int tile_n)
{
    using namespace mxif;
    constexpr int NRB = WN == 4 ? 4 : 2;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int rw = NRB * (wave / WN), rbw = rb0 + rw;   // this wavefront's first row block, in the tile and in the layer
    const int cb0 = tile_n * 8 + (wave % WN) * 2;
    const bool active = (cb0 * 32 < p.N) && (rbw < p.nrb);
    const int C64 = p.C64, CQ = p.CQ;

    const uint32_t lane16 = (uint32_t)lane * 16u, lane8 = 1024u + (uint32_t)lane * 8u, lane4 = (uint32_t)lane * 4u;
    // The weights are the first operand, and lane l32 of it takes row c(l32) of its block of 32: the accumulator of row 8 g + 4 h + i is
    // register 4 g + i of the lanes of half h, so with c(8 g + 4 h + i) = 16 h + 4 g + i a lane ends up with one token and 16
    // consecutive channels of it -- 32 bytes of Y, and the unit in which the next layer's codes are laid out.
    const uint32_t lanep = (uint32_t)((l32 & 3) + ((l32 >> 3) << 2) + (((l32 >> 2) & 1) << 4) + 32 * half);
    int rbs = rb0 + wave;  // row block staged by this wavefront
    rbs = rbs < p.nrb ? rbs : p.nrb - 1;
    const int cbw = (cb0 * 32 < p.N) ? cb0 : 0;  // wavefronts past the last column read block 0 (unused)
    // The streams are read with buffer loads: a wave-uniform descriptor and step offset in scalar registers, the lane offset shared
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    constexpr int RSRC_FLAGS = 0x00020000;
    auto rsrc = [](const void* base, size_t bytes) { return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, RSRC_FLAGS); };
    const __amdgpu_buffer_rsrc_t rs_x = rsrc(p.xq + (size_t)rbs * C64 * 1024, (size_t)C64 * 1024);
    const __amdgpu_buffer_rsrc_t rs_p[2] = {rsrc(p.pq + (size_t)cbw * C64 * 1024, (size_t)C64 * 1024), rsrc(p.pq + (size_t)(cbw + 1) * C64 * 1024, (size_t)C64 * 1024)};
    const __amdgpu_buffer_rsrc_t rs_pe[2] = {rsrc(p.pe + (size_t)cbw * CQ * 256, (size_t)CQ * 256), rsrc(p.pe + (size_t)(cbw + 1) * CQ * 256, (size_t)CQ * 256)};
    __amdgpu_buffer_rsrc_t rs_xe[NRB];
#pragma unroll
    for (int rbi = 0; rbi < NRB; ++rbi) {
        int rb = rbw + rbi;
        rb = rb < p.nrb ? rb : p.nrb - 1;
        rs_xe[rbi] = rsrc(p.xe + (size_t)rb * CQ * 256, (size_t)CQ * 256);
    }

    // Steps (and quads of steps) past the end are clamped instead of predicated: the loads stay
    // unconditional, what they fetch is never used.
    auto load_a = [&](v4i& a, int step) {
        const int st = step < C64 ? step : C64 - 1;
        a = __builtin_bit_cast(v4i, (u4)__builtin_amdgcn_raw_buffer_load_b128(rs_x, lane16, st * 1024, 0));
    };
    auto store_a = [&](const v4i& a, int buf) {
        const v8i e = mxi_expand(a);
        uint8_t* base = lds + (size_t)((buf * RBT + wave) * SLOT);
        *(v4i*)(base + lane16) = v4i{e[0], e[1], e[2], e[3]};
        *(v2i*)(base + lane8) = v2i{e[4], e[5]};
    };
    struct BStage { v4i v[2]; };
    auto load_b = [&](BStage& b, int step) {
        const int st = step < C64 ? step : C64 - 1;
#pragma unroll
        for (int cbi = 0; cbi < 2; ++cbi) b.v[cbi] = __builtin_bit_cast(v4i, (u4)__builtin_amdgcn_raw_buffer_load_b128(rs_p[cbi], lanep * 16u, st * 1024, 0));
    };
    struct Scales { int a[NRB]; int b[2]; };
    auto load_s = [&](Scales& sc, int quad) {
        const int q = quad < CQ ? quad : CQ - 1;
#pragma unroll
        for (int rbi = 0; rbi < NRB; ++rbi) sc.a[rbi] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs_xe[rbi], lane4, q * 256, 0);
#pragma unroll
        for (int cbi = 0; cbi < 2; ++cbi) sc.b[cbi] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs_pe[cbi], lanep * 4u, q * 256, 0);
    };

    v16f t[NRB][2];
#pragma unroll
    for (int a = 0; a < NRB; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) t[a][b][i] = 0.f;

    v8i bu[2][2];  // expanded weight operands: [step parity][column block]

    // One step = one 64-chunk.  On entry: LDS buffers s & 3 and (s + 1) & 3 hold the activation operands of steps s and s + 1, af[0] the
    // first of step s, bu[s & 1] its weight operands, `a` / `b` the packed data of steps s + 2 / s + 1.  During the step the activations
    // of step s + 2 are expanded into their LDS buffer and the weights of step s + 1 into bu[(s + 1) & 1], and the loads of steps
    // s + 4 and s + 3 are issued.  Operands are read across the step's end: what the barrier there orders is written and read two steps
    // apart, so nothing waits for it.  SEL = s % 4 picks the scale byte and the buffer.
    v8i af[2];
    auto lds_a = [&](int buf, int rbi) -> v8i {
        const uint8_t* base = lds + (size_t)((buf * RBT + rw + rbi) * SLOT);
        const v4i lo = *(const v4i*)(base + lane16);
        const v2i hi = *(const v2i*)(base + lane8);
        typedef int v6i __attribute__((ext_vector_type(6)));
        const v6i o = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1]};
        return __builtin_shufflevector(o, o, 0, 1, 2, 3, 4, 5, -1, -1);
    };
    auto do_step = [&](auto sel, int s, v4i& a, BStage& b, const Scales& sc) {
        constexpr int SEL = decltype(sel)::value;
        constexpr int PAR = SEL & 1;
#pragma unroll
        for (int rbi = 0; rbi < NRB; ++rbi) {
            af[(rbi + 1) & 1] = rbi + 1 < NRB ? lds_a(SEL, rbi + 1) : lds_a((SEL + 1) & 3, 0);
#pragma unroll
            for (int cbi = 0; cbi < 2; ++cbi)
                t[rbi][cbi] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(bu[PAR][cbi], af[rbi & 1], t[rbi][cbi], 2, 2, SEL,
                                                                             sc.b[cbi], SEL, sc.a[rbi]);
            if (rbi == 0) {
                store_a(a, (SEL + 2) & 3);
                load_a(a, s + 4);
            }
            if (rbi == 1) {
#pragma unroll
                for (int cbi = 0; cbi < 2; ++cbi) bu[PAR ^ 1][cbi] = mxi_expand(b.v[cbi]);
                load_b(b, s + 3);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
    };

    v4i a0, a1;
    BStage b0, b1;
    Scales s0, s1;
    load_a(a0, 0);
    load_a(a1, 1);
    load_b(b0, 0);
    load_s(s0, 0);
    store_a(a0, 0);
    store_a(a1, 1);
#pragma unroll
    for (int cbi = 0; cbi < 2; ++cbi) bu[0][cbi] = mxi_expand(b0.v[cbi]);
    __builtin_amdgcn_sched_barrier(0);
    load_b(b1, 1);
    load_a(a0, 2);
    load_b(b0, 2);
    load_a(a1, 3);
    load_s(s1, 1);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    af[0] = lds_a(0, 0);

    // steps in groups of eight (two quads of chunks): quad q uses scale set q & 1; step s uses the
    // register sets a(s & 1) and b((s + 1) & 1)
    int s = 0;
    for (; s + 7 < C64; s += 8) {
        do_step(std::integral_constant<int, 0>{}, s, a0, b1, s0);
        do_step(std::integral_constant<int, 1>{}, s + 1, a1, b0, s0);
        do_step(std::integral_constant<int, 2>{}, s + 2, a0, b1, s0);
        do_step(std::integral_constant<int, 3>{}, s + 3, a1, b0, s0);
        load_s(s0, (s >> 2) + 2);
        do_step(std::integral_constant<int, 0>{}, s + 4, a0, b1, s1);
        do_step(std::integral_constant<int, 1>{}, s + 5, a1, b0, s1);
        do_step(std::integral_constant<int, 2>{}, s + 6, a0, b1, s1);
        do_step(std::integral_constant<int, 3>{}, s + 7, a1, b0, s1);
        load_s(s1, (s >> 2) + 3);
    }
    if (s < C64) do_step(std::integral_constant<int, 0>{}, s, a0, b1, s0);
    if (s + 1 < C64) do_step(std::integral_constant<int, 1>{}, s + 1, a1, b0, s0);
    if (s + 2 < C64) do_step(std::integral_constant<int, 2>{}, s + 2, a0, b1, s0);
    if (s + 3 < C64) do_step(std::integral_constant<int, 3>{}, s + 3, a1, b0, s0);
    if (s + 4 < C64) do_step(std::integral_constant<int, 0>{}, s + 4, a0, b1, s1);
    if (s + 5 < C64) do_step(std::integral_constant<int, 1>{}, s + 5, a1, b0, s1);
    if (s + 6 < C64) do_step(std::integral_constant<int, 2>{}, s + 6, a0, b1, s1);

    if (!active) return;

    // ---- rank-r expansion on the bf16 MFMA, accumulated on top of the main product: operands of BD chunks of the rank requested
    // ahead (the registers of the K loop's operands are free; with each chunk's requested at its turn these products took 10500
    // cycles at rank 128, of which the matrix core needs 2048)
    constexpr int BD = NK16 < 3 ? NK16 : 3;
    if constexpr (NK16 > 0) {
        const __amdgpu_buffer_rsrc_t rs_l = __builtin_amdgcn_make_buffer_rsrc((void*)(p.lv + (size_t)cb0 * NK16 * 1024), 0, 2 * NK16 * 1024, RSRC_FLAGS);
        __amdgpu_buffer_rsrc_t rs_t[NRB];
#pragma unroll
        for (int rbi = 0; rbi < NRB; ++rbi) {
            int rb = rbw + rbi;
            rb = rb < p.nrb ? rb : p.nrb - 1;
            rs_t[rbi] = __builtin_amdgcn_make_buffer_rsrc((void*)(p.tv + (size_t)rb * NK16 * 1024), 0, NK16 * 1024, RSRC_FLAGS);
        }
        v8bf lf[BD][2], tf[BD][NRB];
        auto load_branch = [&](int ch) {
#pragma unroll
            for (int cbi = 0; cbi < 2; ++cbi)
                lf[ch % BD][cbi] = __builtin_bit_cast(v8bf, (u4)__builtin_amdgcn_raw_buffer_load_b128(rs_l, lanep * 16u, (cbi * NK16 + ch) * 1024, 0));
#pragma unroll
            for (int rbi = 0; rbi < NRB; ++rbi)
                tf[ch % BD][rbi] = __builtin_bit_cast(v8bf, (u4)__builtin_amdgcn_raw_buffer_load_b128(rs_t[rbi], lane16, ch * 1024, 0));
        };
#pragma unroll
        for (int ch = 0; ch < BD; ++ch) load_branch(ch);
#pragma unroll
        for (int ch = 0; ch < NK16; ++ch) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int rbi = 0; rbi < NRB; ++rbi)
#pragma unroll
                for (int cbi = 0; cbi < 2; ++cbi)
                    t[rbi][cbi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lf[ch % BD][cbi], tf[ch % BD][rbi], t[rbi][cbi], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (ch + BD < NK16) load_branch(ch + BD);
        }
    }

    // ---- epilogue: bf16; with the hand-off the next layer's codes straight from the registers; Y transposed through the wavefront's
    // own LDS slice, full-line stores ------
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    uint8_t* stage = lds + wave * EPI_WAVE;
    const int wr_off = l32 * EPI_ROW + half * 32;
    const int rd_row = lane >> 3, rd_seg = lane & 7;
    // The stores are buffer stores through a descriptor that ends with the wavefront's 128 bytes of the tile's last valid
    // row (rows past M are out of range and dropped by the hardware): no branch, so
    // the compiler can count the stores and need not wait for them when it waits for an older load.
    const int rows_valid = p.M - rbw * 32 < NRB * 32 ? p.M - rbw * 32 : NRB * 32;
    const bool have_y = !HO || p.Y;
    const __amdgpu_buffer_rsrc_t rs_y = __builtin_amdgcn_make_buffer_rsrc(
        have_y ? (void*)(p.Y + (size_t)(rbw * 32) * p.ldy + cb0 * 32) : (void*)p.ho_xq, 0,
        have_y ? (int)((rows_valid - 1) * p.ldy * 2 + 128) : 0, RSRC_FLAGS);
    uint32_t yoff = (uint32_t)(rd_row * (int)p.ldy * 2 + rd_seg * 16);
    const uint32_t ystep = (uint32_t)(8 * (int)p.ldy * 2);
    v4i ov[4];
#pragma unroll
    for (int rbi = 0; rbi < NRB; ++rbi) {
        uint32_t w[2][8];
#pragma unroll
        for (int cbi = 0; cbi < 2; ++cbi) {
#pragma unroll
            for (int i = 0; i < 16; i += 2)
                w[cbi][i >> 1] = __builtin_bit_cast(uint32_t, (bf16x2)__builtin_convertvector(f32x2{t[rbi][cbi][i], t[rbi][cbi][i + 1]}, bf16x2));
            if (DBG) {
                const int row = (rbw + rbi) * 32 + l32;
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (row < p.M && p.dbg_y32) p.dbg_y32[(size_t)row * p.N + (cb0 + cbi) * 32 + 16 * half + i] = t[rbi][cbi][i];
            }
        }
        if constexpr (HO) {
            if (rbw + rbi < p.nrb) mxi_handoff_rows(p, w, rbw + rbi, cb0, lane);
        }
        if (have_y) {
#pragma unroll
            for (int cbi = 0; cbi < 2; ++cbi)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    *(v4i*)(stage + wr_off + cbi * 64 + h * 16) = v4i{(int)w[cbi][4 * h], (int)w[cbi][4 * h + 1], (int)w[cbi][4 * h + 2], (int)w[cbi][4 * h + 3]};
#pragma unroll
            for (int q = 0; q < 4; ++q) ov[q] = *(const v4i*)(stage + (q * 8 + rd_row) * EPI_ROW + rd_seg * 16);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, ov[q]), rs_y, yoff, 0, 0);
                yoff += ystep;
            }
        }
    }
}

template <int NK16, bool DBG, bool HO = false>
__global__ __launch_bounds__(256, 2) void mxi_fwd_kernel(MxiFwdParams p)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[mxif::LDS_BYTES];
    if constexpr (HO) write_tag(p.ho_tag_dst, p.ho_tag);
    // XCD-aware tile order: workgroup ids are dealt round-robin to the 8 XCDs, each gets one run of tiles
    // of the panel order; a last column of tiles of at most 128 channels comes last of all: half the work each, these tiles fill the
    // last generation of the grid.
    auto xcd_order = [](int i, int n) {
        const int per = n >> 3, rem = n & 7, xcd = i & 7, loc = i >> 3;
        return xcd * per + (xcd < rem ? xcd : rem) + loc;
    };
    const int wide = (p.N + 127) / 256, n_wide = p.tilesM * wide, b = (int)blockIdx.x;
    if (b < n_wide) {
        int tile_m, tile_n;
        panel_tile(xcd_order(b, n_wide), p.tilesM, wide, p.panel < wide ? p.panel : wide, tile_m, tile_n);
        mxi_fwd_tile<NK16, DBG, HO, 4>(p, lds, tile_m * mxif::RBT, tile_n);
    } else {
        mxi_fwd_tile<NK16, DBG, HO, 2>(p, lds, xcd_order(b - n_wide, p.tilesM) * mxif::RBT, wide);
    }
}

// Small layers: a wavefront (a workgroup of its own) per tile of NRB*32 x NCB*32 outputs.  Where the 128 x 256 tiles leave most of the
// chip idle, the time of a call is one tile's serial chain of steps; here nothing is shared between wavefronts (no LDS staging, no
// barriers) and both operand streams are requested DEPTH quads of 64-chunks ahead, as packed codes, and unpacked in registers.
// Bounded by that chain for a few tiles (128 x 1152 -> 3456 and 128 x 4608 -> 1152, large tiles / this, both with codes as 8-bit operands: 10.6 /
// 4.2 and 30.3 / 8.6 us; this with 8-bit / 6-bit operands, calls of one captured graph: 4.1 / 3.8 and 8.4 / 7.4 with the operands in the caches,
// 5.1 / 4.8 and 10.7 / 9.6 with them from memory), by the operands' L2 traffic for many.  Same products in the same order as mxi_fwd_kernel.  HO: as there.
template <int NK16, bool DBG, bool HO, int NRB, int NCB>
__global__ __launch_bounds__(64, 2) void mxi_fwd_small_kernel(MxiFwdParams p)
{
    if constexpr (HO) write_tag(p.ho_tag_dst, p.ho_tag);
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    constexpr int RSRC_FLAGS = 0x00020000;
    constexpr int DEPTH = NRB + NCB == 2 ? 4 : NRB + NCB == 3 ? 2 : 1;  // quads in flight (17 registers per row or column block each)
    constexpr int ROW = 64 * NCB + 16;                                  // bytes per staged output row
    __shared__ __attribute__((aligned(16))) uint8_t stage[32 * ROW];

    const int lane = threadIdx.x, half = lane >> 5, l32 = lane & 31;
    // The tiles that share a block of the longer operand run together on one XCD: it is then read from memory once, the shorter one
    // stays in the L2.  (Row blocks always fastest, 50395 x 4608 -> 64: 40.3 us, now 24.9.)
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
        rs_x[i] = __builtin_amdgcn_make_buffer_rsrc((void*)(p.xq + (size_t)rbc[i] * C64 * 1024), 0, C64 * 1024, RSRC_FLAGS);
        rs_xe[i] = __builtin_amdgcn_make_buffer_rsrc((void*)(p.xe + (size_t)rbc[i] * CQ * 256), 0, CQ * 256, RSRC_FLAGS);
    }
    const __amdgpu_buffer_rsrc_t rs_p = __builtin_amdgcn_make_buffer_rsrc((void*)(p.pq + (size_t)cb0 * C64 * 1024), 0, NCB * C64 * 1024, RSRC_FLAGS);
    const __amdgpu_buffer_rsrc_t rs_pe = __builtin_amdgcn_make_buffer_rsrc((void*)(p.pe + (size_t)cb0 * CQ * 256), 0, NCB * CQ * 256, RSRC_FLAGS);

    struct Chunk { v4i a[NRB], b[NCB]; };
    struct Quad { Chunk c[4]; int sa[NRB], sb[NCB]; };
    auto load_scales = [&](Quad& t, int quad) {  // (quads and chunks past the end are clamped: fetched, not used)
        const int q = quad < CQ ? quad : CQ - 1;
#pragma unroll
        for (int i = 0; i < NRB; ++i) t.sa[i] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs_xe[i], lane4, q * 256, 0);
#pragma unroll
        for (int j = 0; j < NCB; ++j) t.sb[j] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs_pe, lane4, (j * CQ + q) * 256, 0);
    };
    auto load_chunk = [&](Chunk& t, int chunk) {
        const int c = chunk < C64 ? chunk : C64 - 1;
#pragma unroll
        for (int j = 0; j < NCB; ++j) t.b[j] = __builtin_bit_cast(v4i, (u4)__builtin_amdgcn_raw_buffer_load_b128(rs_p, lane16, (j * C64 + c) * 1024, 0));
#pragma unroll
        for (int i = 0; i < NRB; ++i) t.a[i] = __builtin_bit_cast(v4i, (u4)__builtin_amdgcn_raw_buffer_load_b128(rs_x[i], lane16, c * 1024, 0));
    };
    Quad qd[DEPTH];
#pragma unroll
    for (int i = 0; i < DEPTH; ++i) {
        load_scales(qd[i], i);
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) load_chunk(qd[i].c[cc], 4 * i + cc);
    }

    v16f t[NRB][NCB];
#pragma unroll
    for (int i = 0; i < NRB; ++i)
#pragma unroll
        for (int j = 0; j < NCB; ++j) t[i][j] = v16f{0};
    // one chunk; its registers are refilled with the chunk DEPTH quads further on as soon as they have been expanded
    auto chunk = [&](Quad& q, const int (&sa)[NRB], const int (&sb)[NCB], auto cc_tag, int quad) {
        constexpr int CC = decltype(cc_tag)::value;
        v8i ae[NRB], be[NCB];
#pragma unroll
        for (int i = 0; i < NRB; ++i) ae[i] = mxi_expand(q.c[CC].a[i]);
#pragma unroll
        for (int j = 0; j < NCB; ++j) be[j] = mxi_expand(q.c[CC].b[j]);
        load_chunk(q.c[CC], 4 * (quad + DEPTH) + CC);
        if (4 * quad + CC < C64) {
#pragma unroll
            for (int i = 0; i < NRB; ++i)
#pragma unroll
                for (int j = 0; j < NCB; ++j)
                    t[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ae[i], be[j], t[i][j], 2, 2, CC, sa[i], CC, sb[j]);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](Quad& q, int quad) {
        int sa[NRB], sb[NCB];
#pragma unroll
        for (int i = 0; i < NRB; ++i) sa[i] = q.sa[i];
#pragma unroll
        for (int j = 0; j < NCB; ++j) sb[j] = q.sb[j];
        load_scales(q, quad + DEPTH);
        chunk(q, sa, sb, std::integral_constant<int, 0>{}, quad);
        chunk(q, sa, sb, std::integral_constant<int, 1>{}, quad);
        chunk(q, sa, sb, std::integral_constant<int, 2>{}, quad);
        chunk(q, sa, sb, std::integral_constant<int, 3>{}, quad);
    };
    int q0 = 0;
    for (; q0 + DEPTH <= CQ; q0 += DEPTH) {
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) multiply(qd[i], q0 + i);
    }
#pragma unroll
    for (int i = 0; i < DEPTH - 1; ++i)
        if (q0 + i < CQ) multiply(qd[i], q0 + i);

    // ---- rank-r expansion and epilogue as in mxi_fwd_kernel
#pragma unroll
    for (int ch = 0; ch < NK16; ++ch) {
        v4i lf[NCB];
#pragma unroll
        for (int j = 0; j < NCB; ++j) lf[j] = *(const v4i*)(p.lv + ((size_t)((size_t)(cb0 + j) * NK16 + ch) * 64 + lane) * 16);
#pragma unroll
        for (int i = 0; i < NRB; ++i) {
            const v4i tf = *(const v4i*)(p.tv + ((size_t)((size_t)rbc[i] * NK16 + ch) * 64 + lane) * 16);
#pragma unroll
            for (int j = 0; j < NCB; ++j)
                t[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, tf), __builtin_bit_cast(v8bf, lf[j]), t[i][j], 0, 0, 0);
        }
    }
    const bool have_y = !HO || p.Y;
    const int rows_valid = p.M - rb0 * 32 < NRB * 32 ? p.M - rb0 * 32 : NRB * 32;
    const __amdgpu_buffer_rsrc_t rs_y = __builtin_amdgcn_make_buffer_rsrc(
        have_y ? (void*)(p.Y + (size_t)(rb0 * 32) * p.ldy + cb0 * 32) : (void*)p.ho_xq, 0,
        have_y ? (int)((rows_valid - 1) * p.ldy * 2 + NCB * 64) : 0, RSRC_FLAGS);
#pragma unroll
    for (int i = 0; i < NRB; ++i) {
#pragma unroll
        for (int j = 0; j < NCB; ++j) {
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
                const bf16x2 h = __builtin_convertvector(f32x2{t[i][j][e], t[i][j][e + 1]}, bf16x2);
                const uint32_t w = __builtin_bit_cast(uint32_t, h);
                const int o = (8 * (e >> 2) + 4 * half + (e & 3)) * ROW + j * 64 + l32 * 2;
                *(uint16_t*)(stage + o) = (uint16_t)(w & 0xFFFFu);
                *(uint16_t*)(stage + o + ROW) = (uint16_t)(w >> 16);
            }
            if (DBG) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int row = (rb0 + i) * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
                    if (row < p.M && p.dbg_y32) p.dbg_y32[(size_t)row * p.N + (cb0 + j) * 32 + l32] = t[i][j][e];
                }
            }
        }
        // read back row-wise (LDS operations of one wavefront complete in order): 4 NCB lanes per row of 64 NCB bytes
        constexpr int LR = 4 * NCB, RP = 64 / LR;
#pragma unroll
        for (int q = 0; q < 32 / RP; ++q) {
            const int row = q * RP + lane / LR, seg = (lane % LR) * 16;
            const v4i o = *(const v4i*)(stage + row * ROW + seg);
            if constexpr (HO) mxi_handoff_emit(p, o, (rb0 + i) * 32 + row, cb0 * 32 + seg / 2);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, o), rs_y, (i * 32 + row) * (int)p.ldy * 2 + seg, 0, 0);
        }
    }
}

template <int NK16, bool DBG, bool HO>
static void mxi_fwd_small_launch(MxiFwdParams p, int rbt, int cbt, hipStream_t s)
{
    p.tilesN = p.N / 32 / cbt;
    p.tilesM = (p.nrb + rbt - 1) / rbt;
    const dim3 grid((unsigned)(p.tilesM * p.tilesN)), block(64);
    if (rbt == 1) hipLaunchKernelGGL((mxi_fwd_small_kernel<NK16, DBG, HO, 1, 1>), grid, block, 0, s, p);
    else if (cbt == 1) hipLaunchKernelGGL((mxi_fwd_small_kernel<NK16, DBG, HO, 2, 1>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((mxi_fwd_small_kernel<NK16, DBG, HO, 2, 2>), grid, block, 0, s, p);
}

template <int NK16>
static void mxi_fwd_launch(const MxiFwdParams& p, hipStream_t s)
{
    // Small layers, by the number T of 32 x 32 tiles (the device holds 2048 wavefronts of these kernels): one tile to a
    // wavefront, larger ones as the L2 traffic of the operands (2, 1.5 and 1 KB per tile and 64-chunk) begins to count, the
    // 128 x 256 tiles once they occupy enough of the chip.  us, the forward's part of activation step and forward, rank 64, the calls of one
    // captured graph with all buffers in turn over 800 MB (the codes of X freshly written, the weights from memory); 1 x 1 / 2 x 1 / 2 x 2:
    //   T =  108 (   2 x 1152 -> 3456):  4.2 /  5.5 /  7.5            T = 1728 ( 512 x 1152 -> 3456):  9.5 /  8.6 / 10.4
    //   T =  144 ( 128 x 4608 -> 1152): 10.9 / 16.1 / 23.1            T = 3360 ( 512 x 2240 -> 6720): 21.5 / 16.7 / 17.3
    //   T = 1152 (1024 x 4608 -> 1152): 13.6 / 14.8 / 21.2            T = 5076 (1500 x 1152 -> 3456): 19.0 / 15.9 / 12.9
    // 2 x 2 / 128 x 256:
    //   T = 5040 (4476 x  896 -> 1152): 11.1 / 11.8                   T = 5076 (1500 x 1152 -> 3456): 13.2 / 13.3
    //   T = 5696 (11389 x 1024 -> 512): 11.3 / 11.7                   T = 6516 (5762 x  896 -> 1152): 12.6 / 12.4
    //   T = 5400 (4770 x 2240 -> 1152): 17.6 / 17.3                   T = 6192 (5500 x 4608 -> 1152): 29.5 / 27.2
    // 12 chunks of K and fewer: the large tiles' prologue weighs more (T = 6144, 8192 x 512 -> 768: 9.5 / 9.9; T = 6912, 1700 x 768 ->
    // 4096: 12.6 / 12.6).  More large tiles than compute units (the tiles of a layer of 128 channels are half-sized): some units get a
    // second one, and the call takes a generation more (T = 6396, 17052 x 832 -> 384: 12.1 / 11.9; T = 6990, 37274 x 2240 -> 192: 18.0 /
    // 21.9; T = 8010, 42700 x 1152 -> 192: 14.3 / 14.7; T = 5150, 82394 x 1152 -> 64: 13.1 / 19.8).
    // With the hand-off, whose codes they form in registers, the large tiles are ahead earlier (T = 3168, 700 x 1152 -> 4608: 14.8 / 15.3; T = 4104,
    // 1200 x 1152 -> 3456: 16.0 / 15.2; T = 4596, 12238 x 1152 -> 384: 15.6 / 13.3), also past one per compute unit (T = 5800, 18532 x 896 -> 320: 15.8 /
    // 13.9; 18545 x 2240 -> 320: 20.4 / 18.5), later by how many wavefronts their last column leaves without
    // channels (T = 6348, 33847 x 512 -> 192: 13.6 / 13.2; T = 4600, 73590 x 896 -> 64: 13.8 / 14.5, 73577 x 64 -> 64: 11.5 / 9.5).
    // Over 5965 random calls of T between 1500 and 9000 measured in the same way in both forms, 508 are more than 3 % of the forward slower than
    // in the better one, 222 more than 8 %; with the lines at 7000 and 5000 instead of 8000 and 5800 589 and 286.  (With everything from
    // memory the large tiles are ahead earlier, with everything in the caches later.)
    const int64_t T = (int64_t)p.nrb * (p.N / 32);
    const bool over = (p.N == 128 ? (p.tilesM + 1) / 2 : p.tilesM * p.tilesN) > compute_units();
    const int over_ho = (p.N & 255) == 192 ? 1 : p.N < 256 ? 12 : 20;  // with the hand-off: chunks from which a second generation counts
    const int line = p.ho_xq ? (over && p.C64 >= over_ho ? 7000 : 4000) : over ? 8000 : p.C64 <= 12 ? 7000 : p.C64 <= 24 ? 6500 : 5800;
    if (T <= line) {
        const int rbt = T <= 1400 ? 1 : 2, cbt = T <= 3600 ? 1 : 2;
        if (p.ho_xq) mxi_fwd_small_launch<NK16, false, true>(p, rbt, cbt, s);
        else if (p.dbg_y32) mxi_fwd_small_launch<NK16, true, false>(p, rbt, cbt, s);
        else mxi_fwd_small_launch<NK16, false, false>(p, rbt, cbt, s);
        return;
    }
    dim3 grid((unsigned)(p.tilesM * p.tilesN)), block(256);
    if (p.ho_xq)
        hipLaunchKernelGGL((mxi_fwd_kernel<NK16, false, true>), grid, block, 0, s, p);
    else if (p.dbg_y32)
        hipLaunchKernelGGL((mxi_fwd_kernel<NK16, true>), grid, block, 0, s, p);
    else
        hipLaunchKernelGGL((mxi_fwd_kernel<NK16, false>), grid, block, 0, s, p);
}

static hipError_t fwd_mxi_launches(const Dims& d, const uint8_t* packed, const uint8_t* act, int64_t M, uint16_t* Y, int64_t ldy,
                                   const lq_fwd_debug* dbg, const Dims* next, uint8_t* act_next, uint8_t* codes, hipStream_t s);

hipError_t launch_fwd_mxi(const Dims& d, const uint8_t* packed, const uint8_t* act, int64_t M, uint16_t* Y, int64_t ldy,
                          const lq_fwd_debug* dbg, hipStream_t s)
{
    return fwd_mxi_launches(d, packed, act, M, Y, ldy, dbg, nullptr, nullptr, nullptr, s);
}

// Forward with the quantized hand-off: `next` is the consuming layer (K = this layer's N), act_next its activation blob
// (main codes and scales are written here), codes the hand-off buffer of its branch codes.  Y may be null.
hipError_t launch_fwd_handoff_mxi(const Dims& d, const uint8_t* packed, const uint8_t* act, int64_t M, uint16_t* Y, int64_t ldy,
                                  const Dims& next, uint8_t* act_next, uint8_t* codes, hipStream_t s)
{
    return fwd_mxi_launches(d, packed, act, M, Y, ldy, nullptr, &next, act_next, codes, s);
}

size_t handoff_codes_bytes(const Dims& next, int64_t M)
{
    const int64_t Mp = (M + 31) / 32 * 32;
    return align256((size_t)Mp * next.K);
}
size_t handoff_total_bytes(const Dims& next, int64_t M)
{
    const int64_t Mp = (M + 31) / 32 * 32;
    return handoff_codes_bytes(next, M) + align256((size_t)Mp * (next.K / 32));
}

static hipError_t fwd_mxi_launches(const Dims& d, const uint8_t* packed, const uint8_t* act, int64_t M, uint16_t* Y, int64_t ldy,
                                   const lq_fwd_debug* dbg, const Dims* next, uint8_t* act_next, uint8_t* codes, hipStream_t s)
{
    const PackedLayout pl = packed_layout(d);
    const ActLayout al = act_layout(d, M);
    MxiFwdParams p;
    p.ho_xq = p.ho_xe = p.ho_cbe = nullptr;
    p.ho_cb = nullptr;
    p.ho_C64 = p.ho_CQ = 0;
    if (next) {
        const ActLayout an = act_layout(*next, M);
        p.ho_xq = act_next + an.off_xq;
        p.ho_xe = act_next + an.off_sx;
        p.ho_cb = (int8_t*)codes;
        p.ho_cbe = codes + handoff_codes_bytes(*next, M);
        p.ho_C64 = next->C64;
        p.ho_CQ = (next->C64 + 3) / 4;
        p.ho_tag = make_tag(*next, LQ_BLOB_ACT, M);
        p.ho_tag_dst = (uint32_t*)act_next;
    }
    p.xq = act + al.off_xq;
    p.xe = act + al.off_sx;
    p.tv = act + al.off_tq;
    p.pq = packed + pl.off_pq;
    p.pe = packed + pl.off_sw;
    p.lv = packed + pl.off_lq;
    p.Y = Y;
    p.ldy = ldy;
    p.M = (int)M;
    p.N = (int)d.N;
    p.C64 = d.C64;
    p.CQ = (d.C64 + 3) / 4;
    p.nrb = (int)(al.Mp / 32);
    p.tilesM = (p.nrb + 3) / 4;
    p.tilesN = (p.N + 255) / 256;
    p.panel = panel_width(p.tilesN, p.C64);
    p.dbg_y32 = dbg ? dbg->y32 : nullptr;
    switch (d.rp >> 4) {
        case 0: mxi_fwd_launch<0>(p, s); break;
        case 2: mxi_fwd_launch<2>(p, s); break;
        case 4: mxi_fwd_launch<4>(p, s); break;
        case 6: mxi_fwd_launch<6>(p, s); break;
        default: mxi_fwd_launch<8>(p, s); break;
    }
    return hipGetLastError();
}

}  // namespace lq
