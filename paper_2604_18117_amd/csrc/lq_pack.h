// Shared by the packing code of all format families: the residual P = W - deq(Q2 L) deq(Q2 R) (Fig. 1, Eq. 5) of a tile, formed
// on the fp64 matrix instruction and handed to the family's encoder, and the kernel that presets blob sections.
#pragma once

#include "lq_internal.h"

namespace lq {

// Sections a pack call presets to a constant (padding codes and scales, smoothing reciprocals of 1), all in one launch.
// Lengths in dwords.
struct PackFill {
    static constexpr int MAX = 4;
    uint32_t* p[MAX];
    uint32_t v[MAX];
    size_t end[MAX];  // running sums of the lengths
    int n;
    void add(void* dst, size_t bytes, uint32_t value)
    {
        if (bytes == 0) return;
        p[n] = (uint32_t*)dst;
        v[n] = value;
        end[n] = (n ? end[n - 1] : 0) + bytes / 4;
        ++n;
    }
};
hipError_t launch_pack_fill(const PackFill& f, hipStream_t s);

#if defined(__HIPCC__)
// The fp64 chain d = fma(l_j, r_j, d), ascending j, runs on v_mfma_f64_16x16x4_f64, which is, bit for bit, four fused
// multiply-adds in ascending order of its contraction index (checked against fma chains).  Factors as the pack step
// dequantises them are exact in fp32 in every family, their products in fp64.
//
// A workgroup owns 64 rows of W (16 per wavefront) and a run of scale groups (GC chunks of 64 along K).  The product is
// formed transposed, 16 values of K by 16 rows of W per tile: lane (l15, q) ends up with row n = l15 and, the chunk's
// K values being dealt to the tiles' rows accordingly, the 16 consecutive values k = 16 q .. 16 q + 15 of every chunk: the
// block maxima are one or two lane exchanges and the codes leave as whole dwords.  (One wavefront per row and group, a lane
// per K value, r dependent fp64 multiply-adds with two scattered loads each, took 111 us for 4608 x 1152 at rank 32 and
// 0.85-1.0 ms for 11200 x 2240 and 6720 x 2240 at rank 64.)
//
// F: lhat(n, j) and rhat(j, k) dequantised factors (k inside the source row), encode(n, group, P, q) for the lane's values.
// The last launch of a pack call: it writes the blob's header too.
template <int R, int GC, typename F>
__global__ __launch_bounds__(256) void pack_residual_kernel(F f, const float* W, int Ks, int groups, int per, uint32_t* blob, BlobTag tag)
{
    typedef float v4f __attribute__((ext_vector_type(4), aligned(4)));  // (W is aligned to its elements only)
    typedef double v4d __attribute__((ext_vector_type(4)));
    constexpr int S = 80;  // LDS row stride in floats: lane (l15, q) reads row 4 s + q, so q moves by 16 banks
    constexpr int RS = R > 0 ? R : 1, NB = R <= 64 ? 2 : 1;
    __shared__ float Rs[NB][RS * S];
    const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, q = lane >> 4, wave = tid >> 6;
    const int runs = (groups + per - 1) / per;
    const int n = (blockIdx.x / runs) * 64 + 16 * wave + l15;
    const int g0 = (blockIdx.x % runs) * per, g1 = g0 + per < groups ? g0 + per : groups;
    double l[RS / 4 + 1];
#pragma unroll
    for (int s = 0; s < R / 4; ++s) l[s] = (double)f.lhat(n, 4 * s + q);
    int buf = 0;
    for (int g = g0; g < g1; ++g) {
        float P[GC][16];
#pragma unroll
        for (int cc = 0; cc < GC; ++cc) {
            const int k0 = (g * GC + cc) * 64;
            if (k0 >= Ks) {  // a chunk of layout padding (uniform)
#pragma unroll
                for (int e = 0; e < 16; ++e) P[cc][e] = 0.f;
                continue;
            }
            v4f w[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) w[t] = *(const v4f*)(W + (size_t)n * Ks + k0 + 16 * q + 4 * t);
            v4d d[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) d[t] = v4d{0.0, 0.0, 0.0, 0.0};
            if constexpr (R > 0) {
                // K value kk of the chunk: tile (kk / 4) % 4, tile row kk / 16 + 4 * (kk % 4)
                float rv[R / 4];
#pragma unroll
                for (int e = 0; e < R / 4; ++e) rv[e] = f.rhat((tid >> 6) + 4 * e, k0 + lane);
                if constexpr (NB == 1) __syncthreads();
#pragma unroll
                for (int e = 0; e < R / 4; ++e)
                    Rs[buf][((tid >> 6) + 4 * e) * S + 16 * ((lane >> 2) & 3) + (lane >> 4) + 4 * (lane & 3)] = rv[e];
                __syncthreads();
#pragma unroll
                for (int s = 0; s < R / 4; ++s)
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        d[t] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)Rs[buf][(4 * s + q) * S + 16 * t + l15], l[s], d[t], 0, 0, 0);
                buf ^= NB - 1;
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) P[cc][4 * t + i] = (float)((double)w[t][i] - d[t][i]);
        }
        f.encode(n, g, P, q);
    }
    write_tag(blob, tag);  // (ahead of the loop it takes the MXFP8 form at rank 128 from 188 registers to 256, 70 us to 104)
}
template <int R, int GC, typename F>
static void pack_residual_launch(const F& f, const float* W, int N, int Ks, int groups, uint8_t* blob, const BlobTag& tag, hipStream_t s)
{
    // runs as long as 2048 workgroups (8 per CU) allow: a run reads its rows' factors once
    const int rb = N / 64, want = 2048 / rb > 1 ? 2048 / rb : 1;
    const int per = (groups + want - 1) / want;
    hipLaunchKernelGGL((pack_residual_kernel<R, GC, F>), dim3((unsigned)(rb * ((groups + per - 1) / per))), dim3(256), 0, s, f, W, Ks,
                       groups, per, (uint32_t*)blob, tag);
}
// (not launched, and the header not written, if the launches before it failed: `before`)
template <int GC, typename F>
static hipError_t pack_residual(hipError_t before, const F& f, const float* W, int N, int Ks, int r, int groups, uint8_t* blob,
                                const BlobTag& tag, hipStream_t s)
{
    if (before != hipSuccess) return before;
    switch (r) {
        case 0: pack_residual_launch<0, GC>(f, W, N, Ks, groups, blob, tag, s); break;
        case 16: pack_residual_launch<16, GC>(f, W, N, Ks, groups, blob, tag, s); break;
        case 32: pack_residual_launch<32, GC>(f, W, N, Ks, groups, blob, tag, s); break;
        case 64: pack_residual_launch<64, GC>(f, W, N, Ks, groups, blob, tag, s); break;
        case 96: pack_residual_launch<96, GC>(f, W, N, Ks, groups, blob, tag, s); break;
        default: pack_residual_launch<128, GC>(f, W, N, Ks, groups, blob, tag, s); break;
    }
    return hipGetLastError();
}

// Maximum magnitude over the lane's values and those of the lanes that hold the rest of its row's block (q ^ 1) or chunk
template <int NV>
__device__ __forceinline__ float pack_amax(const float (&P)[NV])
{
    float a = 0.f;
#pragma unroll
    for (int e = 0; e < NV; ++e) a = fmaxf(a, fabsf(P[e]));
    return a;
}

// Factors with one scale per row (symmetric integers, FP8 E4M3): rows of R, one per workgroup, then rows of L, a few lanes per
// row.  E: scale(amax, &s, &inv), quad(v, inv) = four codes in a dword, r_offset(j, k, r) = byte of R code (j, k).
template <typename E>
__global__ __launch_bounds__(256) void pack_row_factors_kernel(E enc, const float* L, const float* R, int N, int Ks, int K, int r, int rp,
                                                               uint8_t* lc, float* sl, uint8_t* rc, float* sr)
{
    typedef float v4f __attribute__((ext_vector_type(4), aligned(4)));  // (L and R are aligned to their elements only)
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < r) {
        __shared__ float red[4];
        const int j = blockIdx.x;
        const v4f* src = (const v4f*)(R + (size_t)j * Ks);
        float a = 0.f;
        for (int k = tid; k < Ks / 4; k += 256) {
            const v4f v = src[k];
            a = fmaxf(a, fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3]))));
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) a = fmaxf(a, __shfl_xor(a, o, 64));
        if ((tid & 63) == 0) red[tid >> 6] = a;
        __syncthreads();
        a = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
        float s, inv;
        enc.scale(a, &s, &inv);
        if (tid == 0) sr[j] = s;
        for (int k = tid; k < K / 4; k += 256)
            *(uint32_t*)(rc + enc.r_offset(j, 4 * k, r)) = k < Ks / 4 ? enc.quad(src[k], inv) : 0u;
        return;
    }
    // L: each lane holds quads of consecutive rank indices; 8, 16 or 32 lanes share a row (rp = r rounded up)
    const int lpr = rp <= 32 ? 8 : rp <= 64 ? 16 : 32;
    const int row = ((blockIdx.x - r) * 256 + tid) / lpr, c = tid & (lpr - 1);
    if (row >= N) return;
    v4f v = {0.f, 0.f, 0.f, 0.f};
    if (4 * c < r) v = *(const v4f*)(L + (size_t)row * r + 4 * c);
    float a = fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3])));
    for (int o = 1; o < lpr; o <<= 1) a = fmaxf(a, __shfl_xor(a, o, 64));
    float s, inv;
    enc.scale(a, &s, &inv);
    if (c == 0) sl[row] = s;  // (rank 0: finite values, the forward multiplies 0 by them)
    if (4 * c < rp) *(uint32_t*)(lc + (size_t)row * rp + 4 * c) = enc.quad(v, inv);
}
template <typename E>
static void pack_row_factors(const E& enc, const float* L, const float* R, int N, int Ks, int K, int r, int rp, uint8_t* lc, float* sl,
                             uint8_t* rc, float* sr, hipStream_t s)
{
    const int lpr = rp <= 32 ? 8 : rp <= 64 ? 16 : 32;
    hipLaunchKernelGGL((pack_row_factors_kernel<E>), dim3((unsigned)(r + (N * lpr + 255) / 256)), dim3(256), 0, s, enc, L, R, N, Ks, K, r,
                       rp, lc, sl, rc, sr);
}
#endif

}  // namespace lq
