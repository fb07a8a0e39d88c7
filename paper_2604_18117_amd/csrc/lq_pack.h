// Shared by the packing code of all format families: the residual P = W - deq(Q2 L) deq(Q2 R) (Fig. 1, Eq. 5) of a tile, formed
// on the fp64 matrix instruction and handed to the family's encoder, and the kernel that presets blob sections.
#pragma once

#include <type_traits>

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
// formed transposed, 16 values of K by 16 rows of W per tile (result register i of lane (l15, q): tile row q + 4 i, column l15).
// The chunk's K values are dealt to the tiles so that lane (l15, q) ends up with row n = l15 and the 16 consecutive values
// k = 16 q .. 16 q + 15 of every chunk (the block maxima are one or two lane exchanges, the codes leave as whole dwords), and
// that the first operand of the four tiles at one rank index is four consecutive values of a row of R: one load per lane, codes of
// 8 bits in one dword.  So the wavefronts share nothing: no LDS, no barriers, D rank steps of R in flight across chunks and
// the next chunk of W requested under the products.  What bounds it: at high ranks the fp64 matrix rate (64 cycles a
// product; the pipe is busy 62 % at 11200 x 2240 rank 128, 54 % at 6720 x 2240 rank 64), below that how few wavefronts a SIMD has (34 % at
// 4608 x 1152 rank 32).  Against R staged through the LDS as fp32, a barrier per chunk and its loads waited for in every one
// (us a pack call): 4608 x 1152 rank 32, groups of 128, 24.5 -> 17.0, 6720 x 2240 rank 64, groups of 64, 80.4 -> 51.1, 11200 x 2240 rank 128 292 -> 139,
// MXINT4 4608 x 1152 rank 128 105 -> 50, MXFP4 6720 x 2240 rank 128 135 -> 84; MXFP6 factors, whose decoding every wavefront now does for
// itself, 6720 x 2240 rank 128 114.7 -> 97.2, rank 96 91.6 -> 78.8, 3456 x 1152 rank 32 18.3 -> 18.3.  Factors as given move 16 bytes of R per lane and
// rank step, which a workgroup then read once and now reads four times: MX layers up to rank 64 that are small or short of rows take up to 6 %
// longer (2240 x 1920 rank 32 17.1 -> 18.1, 1664 x 2688 rank 64 33.7 -> 35.7; 6848 x 9344 at rank 16 76 -> 85), the others are faster (6720 x 2240 rank 128
// 148 -> 88).  (One wavefront per row and group, a lane per K value: 111 us for the first.)
//
// F: lhat(n, j, q, v) dequantised L of row n at j + q, j + q + 4, + 8, + 12 (j a multiple of 16); rload(j, k) row j of R at k .. k + 3 (k inside the
// source row, a multiple of 4) as stored, rval(raw, v) its four dequantised values (UNIT: what lhat and rval together leave out of a product, a
// power of two that L takes in fp64); encode(n, group, P, q) for the lane's values; PAD_CHECK: the layout may have a chunk of padding behind the
// source's last one (MX), or has none but the compiler allocates registers better with the check (without it groups of 128 with factors as
// given spill 12 at rank 32, MXINT takes 4 % longer at ranks 64 and 96).
// The last launch of a pack call: it writes the blob's header too.
typedef float pack_v4f __attribute__((ext_vector_type(4), aligned(4)));  // (W, L and R are aligned to their elements only)
struct PackCodes4 {  // four 8-bit codes and their scale
    uint32_t c;
    float s;
};
template <int R, int GC, typename F>
__global__ __launch_bounds__(256, R < 64 || (R == 64 && sizeof(typename F::Raw) <= 8) ? 3 : 2) void pack_residual_kernel(F f, const float* W, int Ks, int groups, int per, uint32_t* blob, BlobTag tag)
{
    typedef double v4d __attribute__((ext_vector_type(4)));
    constexpr int NS = R / 4, DMAX = (sizeof(typename F::Raw) > 8 && (R > 32 || GC == 2)) || (GC == 2 && R >= 64) ? 4 : 8, D = NS < DMAX ? NS : DMAX;  // (registers)
    static_assert(NS == 0 || NS % D == 0, "whole turns of the ring");
    const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, q = lane >> 4, wave = tid >> 6;
    const int runs = (groups + per - 1) / per;
    const int n = (blockIdx.x / runs) * 64 + 16 * wave + l15;
    const int g0 = (blockIdx.x % runs) * per, g1 = g0 + per < groups ? g0 + per : groups;
    const int kl = 16 * (l15 & 3) + 4 * (l15 >> 2);  // the lane's K values of a chunk as first operand
    pack_v4f w[4];
    auto request = [&](int k0) {
#pragma unroll
        for (int t = 0; t < 4; ++t) w[t] = *(const pack_v4f*)(W + (size_t)n * Ks + k0 + 16 * q + 4 * t);
    };
    const int kfirst = !F::PAD_CHECK || g0 * GC * 64 < Ks ? g0 * GC * 64 : Ks - 64;  // (a run may be layout padding alone)
    double l[NS + 1];
    typename F::Raw rr[D + 1];
#pragma unroll
    for (int s = 0; s < NS; s += 4) {
        float v[4];
        f.lhat(n, 4 * s, q, v);
#pragma unroll
        for (int i = 0; i < 4; ++i) l[s + i] = (double)v[i] * F::UNIT;
    }
#pragma unroll
    for (int s = 0; s < D; ++s) rr[s] = f.rload(4 * s + q, kfirst + kl);
    if constexpr (R > 0) request(kfirst);
    // A chunk's products.  `more`: the run has a source chunk behind it.  Where the ring holds half a chunk or more, a run's last chunk is code of
    // its own that requests nothing past it: refilled from the same chunk, as above that, the ring would fetch up to all of R once more, and many
    // runs are one chunk long (us a pack call, MX: factors as given 2240 x 1920 rank 32 20.9 -> 18.1, 18176 x 5120 rank 32 177 -> 147).
    constexpr bool OWN_LAST = R <= 32 || (R == 64 && GC == 1 && sizeof(typename F::Raw) <= 8);
    constexpr bool PAD_INSIDE = F::PAD_CHECK && R <= 64;  // (padding in the same loop, or in one behind it: as three wavefronts of MXFP8 factors fit a SIMD; 5824 x 14848 rank 96 505 -> 353 us)
    auto products = [&](auto last, bool more, int k0, float (&P)[16]) {
        constexpr bool LAST = OWN_LAST && decltype(last)::value;
        if constexpr (OWN_LAST) more = !LAST;
        const int knext = more ? k0 + 64 : k0;
        if constexpr (R == 0) request(k0);
        pack_v4f wc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) wc[t] = w[t];
        if (R > 0 && more) request(knext);
        v4d d[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) d[t] = v4d{0.0, 0.0, 0.0, 0.0};
        if constexpr (R > 0) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                float a[4];
                f.rval(rr[s % D], a);
                if (!LAST || s + D < NS) rr[s % D] = f.rload(4 * ((s + D) % NS) + q, (s + D < NS ? k0 : knext) + kl);
#pragma unroll
                for (int t = 0; t < 4; ++t) d[t] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[t], l[s], d[t], 0, 0, 0);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t) P[4 * i + t] = (float)((double)wc[i][t] - d[t][i]);
    };
    auto group = [&](auto last, bool more, int g) {
        float P[GC][16];
#pragma unroll
        for (int cc = 0; cc < GC; ++cc) {
            const int k0 = (g * GC + cc) * 64;
            if (PAD_INSIDE && k0 >= Ks) {  // a chunk of layout padding (uniform)
#pragma unroll
                for (int e = 0; e < 16; ++e) P[cc][e] = 0.f;
                continue;
            }
            if (cc + 1 == GC) products(last, more, k0, P[cc]);
            else products(std::false_type{}, true, k0, P[cc]);
        }
        f.encode(n, g, P, q);
    };
    const int gs = F::PAD_CHECK && Ks / (64 * GC) < g1 ? Ks / (64 * GC) : g1;  // (past the run's last source group)
    int g = g0;
    if constexpr (OWN_LAST) {
        for (; g < gs - 1; ++g) group(std::false_type{}, true, g);
        for (; g < g1; ++g) group(std::true_type{}, false, g);
    } else if constexpr (PAD_INSIDE) {
        for (; g < g1; ++g) group(std::false_type{}, g + 1 < gs, g);
    } else {
        for (; g < gs; ++g) group(std::false_type{}, g + 1 < gs, g);
        if constexpr (F::PAD_CHECK) {
            const float P[GC][16] = {};
            for (; g < g1; ++g) f.encode(n, g, P, q);
        }
    }
    write_tag(blob, tag);
}
// Scale groups per run.  A compute unit works through ceil(workgroups / units) of them, each its chunks and about 0.7 of a chunk's
// time until its rows' factors and first operands are there; the matrix unit is busy from about 2.5 workgroups per compute unit on.
// (Runs as long as 2048 workgroups allow, 6720 x 2240 rank 64 takes 59.7 us instead of 54.5, 11200 x 2240 rank 128 169.5 instead of 153.3.)
static inline int pack_residual_run(int rb, int groups, int gc)
{
    const int units = compute_units();
    int best = 1;
    int64_t best_cost = 0;
    for (int per = 1; per <= groups; ++per) {
        const int64_t wgs = (int64_t)rb * ((groups + per - 1) / per), cost = (wgs + units - 1) / units * (10 * per * gc + 7);
        if (per > 1 && 2 * wgs < 5 * units) break;
        if (per == 1 || cost < best_cost) {
            best = per;
            best_cost = cost;
        }
    }
    return best;
}
template <int R, int GC, typename F>
static void pack_residual_launch(const F& f, const float* W, int N, int Ks, int groups, uint8_t* blob, const BlobTag& tag, hipStream_t s)
{
    const int rb = N / 64, want = 2048 / rb > 1 ? 2048 / rb : 1;  // (rank 0 only streams W: 2048 workgroups)
    const int per = R > 0 ? pack_residual_run(rb, groups, GC) : (groups + want - 1) / want;
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
