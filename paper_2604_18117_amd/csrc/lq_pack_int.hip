// Offline packing for the INT family (paper Fig. 1 caption and Eq. 5):
//   Q2(R), Q2(L) with one scale per row; P = W - deq(Q2 L) deq(Q2 R) accumulated in fp64 and
//   rounded once to fp32; Q1(P) = INT4 with one fp32 scale per group of g values along K
//   (SINT4-style blocks, App. A.3), or the literal SINT4 blocks: 64 values, FP16 scale.  Also the inverse
//   views used by tests.
// Quantiser: s = amax / qmax, code = rne(v * (qmax / amax)), symmetric range, all-zero -> s = 1.
#include <type_traits>

#include "lq_pack.h"

namespace lq {

__device__ __forceinline__ void scale_pair(float amax, float qmax, float* s, float* inv)
{
    if (amax == 0.0f) {
        *s = 1.0f;
        *inv = 1.0f;
    } else {
        *s = amax / qmax;
        *inv = qmax / amax;
    }
}

__device__ __forceinline__ int quant_code(float v, float inv, float qmax)
{
    float r = rintf(v * inv);
    r = fminf(fmaxf(r, -qmax), qmax);
    return (int)r;
}

// byte offset of R code (j,k) in the activation kernel's operand order:
// [chunk = k/64][jb = j/16][lane = j%16 + 16*((k%64)/16)][k%16]
__device__ __forceinline__ size_t rq_offset(int j, int k, int r)
{
    const int c = k >> 6, kq = (k & 63) >> 4;
    return ((size_t)((size_t)c * (r >> 4) + (j >> 4)) * 64 + (j & 15) + 16 * kq) * 16 + (k & 15);
}

// Q2 of a row of L or R
struct PackIntRows {
    float qmax;
    __device__ void scale(float amax, float* s, float* inv) const { scale_pair(amax, qmax, s, inv); }
    template <typename V>
    __device__ uint32_t quad(V v, float inv) const
    {
        uint32_t w = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) w |= (uint32_t)(quant_code(v[i], inv, qmax) & 0xFF) << (8 * i);
        return w;
    }
    __device__ size_t r_offset(int j, int k, int r) const { return rq_offset(j, k, r); }
};

// Residual of a scale group of GC chunks: dequantised (from_q) or given factors; Q1 = INT4, fp32 scale (times 2^6, lq_internal.h)
// or SINT4's FP16 scale (stored as its bits; codes against the stored scale).
template <int GC, bool FROMQ>
struct PackIntResidual {
    using Raw = std::conditional_t<FROMQ, PackCodes4, pack_v4f>;
    const float *L, *R;
    const int8_t* lq;
    const float* sl;
    const int8_t* rq;
    const float* sr;
    uint8_t* pq;
    float* swT;
    int N, K, r, rp, ga;
    __device__ void lhat(int n, int j, int q, float (&v)[4]) const
    {
        if constexpr (FROMQ) {
            const uint4 c = *(const uint4*)(lq + (size_t)n * rp + j);
            const uint32_t d[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = (float)(int8_t)(d[i] >> (8 * q)) * sl[n];
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = L[(size_t)n * r + j + 4 * i + q];
        }
    }
    __device__ Raw rload(int j, int k) const
    {
        if constexpr (FROMQ) return Raw{*(const uint32_t*)(rq + rq_offset(j, k, r)), sr[j]};
        else return *(const Raw*)(R + (size_t)j * K + k);
    }
    static constexpr double UNIT = 1.0;
    static constexpr bool PAD_CHECK = GC == 2 && !FROMQ;
    __device__ void rval(const Raw& x, float (&v)[4]) const
    {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if constexpr (FROMQ) v[t] = (float)(int8_t)(x.c >> (8 * t)) * x.s;
            else v[t] = x[t];
        }
    }
    __device__ void encode(int n, int g, const float (&P)[GC][16], int q) const
    {
        float a = pack_amax(P[0]);
        if constexpr (GC == 2) a = fmaxf(a, pack_amax(P[1]));
        a = fmaxf(a, __shfl_xor(a, 16));
        a = fmaxf(a, __shfl_xor(a, 32));
        float s, inv;
        if (ga) {
            const uint32_t bits = sint4_scale(a, &inv);
            if (q == 0) ((uint32_t*)swT)[(size_t)g * N + n] = bits;
        } else {
            scale_pair(a, 7.0f, &s, &inv);
            if (q == 0) swT[(size_t)g * N + n] = ldexpf(s, 6);
        }
#pragma unroll
        for (int cc = 0; cc < GC; ++cc) {
            // 16 six-bit fields = dwords 3 (q % 2) .. 3 (q % 2) + 2 of the operand of K half q / 2
            uint32_t w[3] = {0u, 0u, 0u};
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const uint64_t v = (uint64_t)f6_field(quant_code(P[cc][e], inv, 7.0f)) << ((6 * e) & 31);
                w[(6 * e) >> 5] |= (uint32_t)v;
                if (((6 * e) & 31) > 26) w[((6 * e) >> 5) + 1] |= (uint32_t)(v >> 32);
            }
            uint8_t* ch = pq + f6_chunk_offset(n, (g * GC + cc) * 64, K >> 6);
            const int slot = (n & 31) + 32 * (q >> 1);
            typedef uint32_t u2 __attribute__((ext_vector_type(2)));
            if (q & 1) {
                *(uint32_t*)(ch + f6_dword_offset(slot, 3)) = w[0];
                *(u2*)(ch + f6_dword_offset(slot, 4)) = u2{w[1], w[2]};
            } else {
                *(u2*)(ch + f6_dword_offset(slot, 0)) = u2{w[0], w[1]};
                *(uint32_t*)(ch + f6_dword_offset(slot, 2)) = w[2];
            }
        }
    }
};

__global__ __launch_bounds__(256) void pack_fill_kernel(PackFill f)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    size_t begin = 0;
    for (int k = 0; k < f.n; ++k) {
        if (i < f.end[k]) {
            f.p[k][i - begin] = f.v[k];
            return;
        }
        begin = f.end[k];
    }
}
hipError_t launch_pack_fill(const PackFill& f, hipStream_t s)
{
    if (f.n == 0) return hipSuccess;
    const size_t n = f.end[f.n - 1];
    hipLaunchKernelGGL(pack_fill_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, f);
    return hipGetLastError();
}

// reciprocals of the smoothing vector
__global__ __launch_bounds__(256) void smooth_recip_kernel(const float* gamma, int Ks, int K, float* rg)
{
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < K) rg[k] = k < Ks ? __fdiv_rn(1.0f, gamma[k]) : 1.0f;  // (k >= Ks: layout padding)
}

hipError_t launch_set_smoothing(const Dims& d, const float* gamma, uint8_t* packed, hipStream_t s)
{
    const PackedLayout pl = packed_layout(d);
    hipLaunchKernelGGL(smooth_recip_kernel, dim3((unsigned)((d.K + 255) / 256)), dim3(256), 0, s, gamma, (int)d.Ks, (int)d.K,
                       (float*)(packed + pl.off_rg));
    return hipGetLastError();
}

hipError_t launch_pack_int(const Dims& d, int from_q, const float* W, const float* L,
                           const float* R, uint8_t* packed, hipStream_t s)
{
    const PackedLayout pl = packed_layout(d);
    int8_t* lq = (int8_t*)(packed + pl.off_lq);
    float* sl = (float*)(packed + pl.off_sl);
    int8_t* rq = (int8_t*)(packed + pl.off_rq);
    float* sr = (float*)(packed + pl.off_sr);
    uint8_t* pq = packed + pl.off_pq;
    float* swT = (float*)(packed + pl.off_sw);
    const int N = (int)d.N, K = (int)d.K;
    PackFill fill;
    fill.n = 0;
    if (d.smooth) fill.add(packed + pl.off_rg, (size_t)K * 4, 0x3F800000u);  // reciprocals of the smoothing vector start at 1
    hipError_t e = launch_pack_fill(fill, s);
    if (e != hipSuccess) return e;
    pack_row_factors(PackIntRows{(float)d.qmax_bw}, L, R, N, K, K, d.r, d.rp, (uint8_t*)lq, sl, (uint8_t*)rq, sr, s);
    e = hipGetLastError();
    const BlobTag tag = make_tag(d, LQ_BLOB_PACKED, 0);
    auto residual = [&](auto gc, auto fq) {
        constexpr int GC = decltype(gc)::value;
        return pack_residual<GC>(e, PackIntResidual<GC, decltype(fq)::value>{L, R, lq, sl, rq, sr, pq, swT, N, K, d.r, d.rp, d.ga ? 1 : 0}, W, N, K, d.r, d.G,
                                 packed, tag, s);
    };
    const std::integral_constant<int, 1> one{};
    const std::integral_constant<int, 2> two{};
    if (from_q && d.r > 0) return d.g == 64 ? residual(one, std::true_type{}) : residual(two, std::true_type{});
    return d.g == 64 ? residual(one, std::false_type{}) : residual(two, std::false_type{});
}

// ---- plain views ----------------------------------------------------------------------------
__global__ __launch_bounds__(256) void unpack_w_kernel(const uint8_t* packed, PackedLayout pl, int N, int K,
                                                       int r, int rp, int g, int ga, lq_weights_view out)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int C64 = K >> 6, G = K / g;
    if (idx < (size_t)N * K) {
        const int n = (int)(idx / K), k = (int)(idx % K);
        if (out.pq) {
            out.pq[idx] = (int8_t)f6_get(packed + pl.off_pq, n, k, C64);
        }
    }
    if (idx < (size_t)N * G && out.sw) {
        const int n = (int)(idx / G), gi = (int)(idx % G);
        out.sw[idx] = ga ? f16_bits_value(((const uint32_t*)(packed + pl.off_sw))[(size_t)gi * N + n])
                         : ldexpf(((const float*)(packed + pl.off_sw))[(size_t)gi * N + n], -6);
    }
    if (idx < (size_t)N * r && out.lq) {
        const int n = (int)(idx / r), j = (int)(idx % r);
        out.lq[idx] = ((const int8_t*)(packed + pl.off_lq))[(size_t)n * rp + j];
    }
    if (idx < (size_t)N && out.sl) out.sl[idx] = ((const float*)(packed + pl.off_sl))[idx];
    if (idx < (size_t)r * K && out.rq) {
        const int j = (int)(idx / K), k = (int)(idx % K);
        out.rq[idx] = ((const int8_t*)(packed + pl.off_rq))[rq_offset(j, k, r)];
    }
    if (idx < (size_t)r && out.sr) out.sr[idx] = ((const float*)(packed + pl.off_sr))[idx];
}

hipError_t launch_unpack_weights_int(const Dims& d, const uint8_t* packed, const lq_weights_view* out,
                                     hipStream_t s)
{
    const PackedLayout pl = packed_layout(d);
    const size_t n = (size_t)(d.N > d.r ? d.N : d.r) * (d.K > d.r ? d.K : d.r);  // covers N x K, r x K and N x r
    hipLaunchKernelGGL(unpack_w_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, packed, pl, (int)d.N,
                       (int)d.K, d.r, d.rp, d.g, d.ga ? 1 : 0, *out);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void unpack_a_kernel(const uint8_t* act, ActLayout al, int M, int K, int r,
                                                       int rp, int ga, lq_act_view out)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int C64 = K >> 6;
    if (idx < (size_t)M * K && out.xq) {
        const int m = (int)(idx / K), k = (int)(idx % K);
        out.xq[idx] = (int8_t)f6_get(act + al.off_xq, m, k, C64);
    }
    if (ga) {
        if (idx < (size_t)M * C64 && out.sx) {
            const int m = (int)(idx / C64), gi = (int)(idx % C64);
            out.sx[idx] = f16_bits_value(((const uint32_t*)(act + al.off_sx))[sxg_index(m, gi, (int)((al.Mp + 127) / 128))]);
        }
    } else if (idx < (size_t)M && out.sx) {
        out.sx[idx] = ((const float*)(act + al.off_sx))[idx];
    }
    if (idx < (size_t)M && out.st) out.st[idx] = ((const float*)(act + al.off_st))[idx];
    if (idx < (size_t)M * r && out.tq) {
        const int m = (int)(idx / r), j = (int)(idx % r);
        out.tq[idx] = ((const int8_t*)(act + al.off_tq))[(size_t)m * rp + j];
    }
}

hipError_t launch_unpack_act_int(const Dims& d, const uint8_t* act, int64_t M, const lq_act_view* out,
                                 hipStream_t s)
{
    const ActLayout al = act_layout(d, M);
    const size_t n = (size_t)M * (d.K > d.r ? d.K : d.r);
    hipLaunchKernelGGL(unpack_a_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, act, al, (int)M,
                       (int)d.K, d.r, d.rp, d.ga ? 1 : 0, *out);
    return hipGetLastError();
}

}  // namespace lq
