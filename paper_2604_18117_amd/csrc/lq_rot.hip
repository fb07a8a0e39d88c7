// Rotation search for the low-rank factors (Section 3.3, Eq. 6-7): one step on an orthogonal r x r matrix Omega that
// lowers the error of quantising L Omega and Omega^T R with Q2, the product L R unchanged.
//     loss(Omega) = mean ( Q2(Z1) - Z1 )^2 + mean ( Q2(Z2) - Z2 )^2,   Z1 = L Omega (N x r),  Z2 = Omega^T R (r x K)
// Q2: the branch weight format of the configuration along the rows of Z1 and Z2, as lq_pack_weights applies it to L and R:
// symmetric integers or FP8 E4M3 with one fp32 scale per row, or MXFP8e4 / MXFP6e2 / MXINT blocks of 32 with E8M0 scales.  Z1 and Z2 are fp32 chains z = fma(a_i, b_i, z) over the rank index
// ascending (the codes depend on their rounding); the rounding has zero derivative (App. B.2), so
//     G = -2/(N r) L^T E1 - 2/(r K) R E2^T
// and the update is the Cayley SGD with momentum of the work the paper cites for it (Li et al. 2020, Algorithm 1).
// Four launches per step up to rank 32, five above (one less with block-scaled Q2), no atomics, every sum in a fixed order:
//   rot_z_kernel      128 rows of L (or columns of R) per workgroup turn (64 at ranks 96 and 128): Z1 / Z2 on the fp32
//                     matrix instruction, E1 / E2, their part of G, partial sums of squares.  A row of Z2 runs over all of
//                     K, so with one scale per row a small launch before it, rot_max_kernel, leaves the row maxima of Z2
//   rot_sum_kernel    G from the workgroups' parts (fp64), the loss
//   rot_cayley_kernel one workgroup: momentum, the skew-symmetric W, step length, the fixed-point passes; from rank 64 on
//                     rot_wh_kernel and rot_update_kernel, a workgroup per 16 columns of Omega
//
// v_mfma_f32_16x16x4_f32 is, bit for bit, four fused multiply-adds in ascending order of its contraction index (checked
// against fma chains on random operands over 2^+-12 and on subnormal products), so it evaluates the chains that
// define Z1 and Z2.  One step on 11200 x 64 and 64 x 2240 factors took 202 us with one thread per row or column
// (44 + 9 workgroups, Omega read from LDS for every fourth multiply-add; the update alone 66 us on one CU's vector ALUs).
#include <mutex>

#include <type_traits>

#include "lq_internal.h"

namespace lq {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int ROT_TPB = 256;

// How groups of rows of L and of columns of R are dealt to workgroups.  Every workgroup leaves one r x r part of the
// gradient, so their number is capped: at rank 64 by what LQ_ROT_STATIC_SCRATCH_BYTES holds, at the others by the traffic of
// rot_sum_kernel (128 parts of rank 128 are 8 MB).  Up to rank 64 a group is 128 rows, 8 wavefronts: two wavefronts
// per SIMD hide each other's LDS and barrier waits; Omega and two groups of 128 rows do not fit the LDS at ranks 96 and 128.
struct RotSplit {
    int gL, gR;   // groups
    int wL, wR;   // workgroups that form E1 and E2
    int wM;       // workgroups that leave row maxima of Z2 (row kinds), 64 columns a turn
};
static RotSplit rot_split(const Dims& d)
{
    const int cap = d.r <= 32 ? 256 : d.r == 64 ? 112 : 128, rows = d.r <= 64 ? 128 : 64;
    RotSplit w;
    w.gL = (int)((d.N + rows - 1) / rows);
    w.gR = (int)((d.K + rows - 1) / rows);
    const int per = (w.gL + w.gR + cap - 1) / cap;
    w.wL = (w.gL + per - 1) / per;
    w.wR = w.gR < cap - w.wL ? w.gR : cap - w.wL;
    if (w.wR < 1) w.wR = 1;
    w.wM = (int)(d.K / 64) < 256 ? (int)(d.K / 64) : 256;
    return w;
}

RotLayout rot_layout(const Dims& d)
{
    RotLayout rl;
    const RotSplit w = rot_split(d);
    const size_t rr = (size_t)d.r * d.r * 4;
    size_t o = 0;
    rl.off_X = o;   o = align256(o + rr);
    rl.off_M = o;   o = align256(o + rr);
    rl.off_G = o;   o = align256(o + rr);
    rl.off_E1 = o;  o = align256(o + (size_t)d.N * d.r * 4);
    rl.off_E2 = o;  o = align256(o + (size_t)d.r * d.K * 4);
    rl.off_ax = o;  o = align256(o + (size_t)w.wM * d.r * 4);
    rl.off_lp = o;  o = align256(o + (size_t)(w.wL + w.wR) * 4);
    rl.off_gp = o;  o = align256(o + (size_t)(w.wL + w.wR) * rr);
    rl.total = o;
    // The size callers are told never falls below that of the first layout (row maxima and loss partials per wavefront of 256
    // rows or columns, 64 parts of the gradient, three r x r work matrices): what lq_rot_sizes returned for a layer stays the least it
    // returns, and the library's own array takes no configuration that it refused.
    {
        const size_t nlb = ((size_t)d.N + 255) / 256, nkb = ((size_t)d.K + 255) / 256;
        size_t f = align256(rl.off_ax + nkb * 4 * d.r * 4);
        f = align256(f + (nlb + d.r * nkb) * 4);
        f = align256(f + 64 * rr);
        f = align256(f + 3 * rr);
        if (f > rl.total) rl.total = f;
    }
    return rl;
}

// Q2, the format lq_pack_weights gives L and R (App. A.3).  Row kinds carry one fp32 scale per row: 0 symmetric integers
// of qmax, 1 FP8 E4M3 (largest magnitude 448).  Block kinds carry an E8M0 scale per 32 values along the row: 2 MXFP8e4,
// 3 MXFP6e2, 4 MXINT of `bits`.
struct RotQ {
    int kind;
    float top;  // row kinds: qmax or 448
    int bits;   // MXINT
};

// Row kinds: scale amax / top, codes against top / amax (an all-zero row: scale 1).
__device__ __forceinline__ void rot_scale(float amax, float top, float& s, float& inv)
{
    if (amax == 0.f) {
        s = 1.f;
        inv = 1.f;
    } else {
        s = amax / top;
        inv = top / amax;
    }
}
__device__ __forceinline__ float rot_fp8_value(float u)  // nearest E4M3 number (ties to even), saturating at 448
{
    u = fminf(fmaxf(u, -448.f), 448.f);  // the converter returns NaN above 464
    const int code = __builtin_amdgcn_cvt_pk_fp8_f32(u, u, 0, false) & 0xFF;
    return __builtin_amdgcn_cvt_f32_fp8(code, 0);
}
template <int QK>  // 0: integers of qmax = top; 1: FP8 E4M3
__device__ __forceinline__ float rot_err(float z, float s, float inv, float top)
{
    if constexpr (QK == 0) {
        float c = rintf(z * inv);
        c = fminf(fmaxf(c, -top), top);
        return c * s - z;
    } else {
        return rot_fp8_value(z * inv) * s - z;
    }
}

template <typename F>
__device__ __forceinline__ void for_rows(F f)  // f(0) .. f(3) with the argument as a compile-time constant
{
    f(std::integral_constant<int, 0>{});
    f(std::integral_constant<int, 1>{});
    f(std::integral_constant<int, 2>{});
    f(std::integral_constant<int, 3>{});
}

// Block kinds: the shared exponent floor(log2 amax) - (largest element exponent: 8 for E4M3, 2 for E2M3, 0 for MXINT),
// kept in [-127, 127]; an all-zero block: -127.
__device__ __forceinline__ int rot_block_exp(float amax, const RotQ& q)
{
    if (amax == 0.f) return -127;
    const int e = __builtin_amdgcn_frexp_expf(amax) - 1 - (q.kind == 2 ? 8 : q.kind == 3 ? 2 : 0);
    return e < -127 ? -127 : e > 127 ? 127 : e;
}
__device__ __forceinline__ float rot_err_block(float z, int e, const RotQ& q)
{
    if (q.kind == 2) return __builtin_ldexpf(rot_fp8_value(__builtin_ldexpf(z, -e)), e) - z;
    if (q.kind == 3) {  // E2M3: spacing 1/8 below 2, 1/4 below 4, 1/2 up to the largest magnitude 7.5
        const float m = fminf(fabsf(__builtin_ldexpf(z, -e)), 7.5f);
        const float step = m < 2.f ? 0.125f : m < 4.f ? 0.25f : 0.5f;
        const float v = fminf(rintf(m / step) * step, 7.5f);
        return __builtin_copysignf(__builtin_ldexpf(v, e), z) - z;
    }
    const int frac = q.bits - 2;
    const float qmax = (float)((1 << (q.bits - 1)) - 1);
    float c = rintf(__builtin_ldexpf(z, frac - e));
    c = fminf(fmaxf(c, -qmax), qmax);
    return __builtin_ldexpf(c, e - frac) - z;
}

struct RotZParams {
    const float* L;
    const float* R;
    const float* X;    // Omega
    int N, K;
    RotSplit w;
    RotQ q;
    float *oL, *oR;    // E1, E2 (ROT_OUT: the rotated factors)
    float* ax;         // row maxima of Z2, [wM][r]
    float* lp;         // sums of squares, [wL + wR]
    float* gp;         // parts of the gradient, [wL + wR][r][r]
    float c1, c2;
};

// ROT_OUT: write Z1 and Z2.  ROT_ERR: E1, E2 and their parts of G.
enum { ROT_OUT, ROT_ERR };

// LDS strides in floats, chosen for conflict-free operand reads: lane (l15, q) reads Omega[4 s + q][l15], so q has to move
// by 16 banks; it reads row l15, column 4 s + q of the staged rows of L and, in the second contraction, row 16 s + 4 q + u,
// column l15 of them and of the error: a stride of 4 modulo 16 serves both.  Columns of R are staged as they lie in memory, rows of
// 16 NWV values: column l15 of row 4 s + q and, in the second contraction, 16 bytes (16 s + 4 q ..) of row l15 (transposed on the
// way in, their stores met 8 to a bank: 9340 cycles from a workgroup's start to its first product at rank 64, 2700 for rows of L).
template <int R> constexpr int rot_sx() { return R % 32 ? R : R + 16; }
template <int R> constexpr int rot_sl() { return R + 4; }
template <int NWV> constexpr int rot_sr() { return 16 * NWV + 16; }
template <int R, int NWV> constexpr int rot_stage() { return 16 * NWV * rot_sl<R>() > R * rot_sr<NWV>() ? 16 * NWV * rot_sl<R>() : R * rot_sr<NWV>(); }
template <int R, int NWV> constexpr int rot_z_lds() { return (R * rot_sx<R>() + rot_stage<R, NWV>() + 16 * NWV * rot_sl<R>() + (NWV + 2) * R) * 4; }

// A workgroup turn is a group of 16 * NWV rows of L (columns of R): each wavefront forms 16
// rows of Z (R / 16 tiles of 16 x 16: lane (l15, q) holds rows 4 q + i, column l15), quantises them in registers, and
// leaves the error in LDS, from where each of 4 wavefronts contracts one quadrant of G over their 64 rows; the quadrant
// stays in registers over all turns, and 8 wavefronts add their two halves at the end.
// QK: 0 integer rows, 1 FP8 rows (one scale per row), 2 block kinds.
template <int R, int MODE, int QK, int NWV>
__global__ __launch_bounds__(64 * NWV) void rot_z_kernel(RotZParams p)
{
    constexpr int T = R / 16, H = T > 1 ? T / 2 : 1, SX = rot_sx<R>(), SL = rot_sl<R>(), SR = rot_sr<NWV>();
    constexpr int NTHR = 64 * NWV, ROWS = 16 * NWV;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    float* Xs = lds;                 // Omega
    float* Ls = Xs + R * SX;         // the group's rows of L / columns of R
    float* Es = Ls + rot_stage<R, NWV>();  // their errors
    float* red = Es + ROWS * SL;     // [NWV][R] column maxima per wavefront
    float* sc = red + NWV * R;       // scale[R], 1 / scale[R] of the rows of Z2
    const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nL = p.w.wL;
    const bool left = (int)blockIdx.x < nL;
    const int wg = left ? blockIdx.x : blockIdx.x - nL;
    const int nwg = left ? nL : (int)gridDim.x - nL;
    const int nrows = left ? p.N : p.K;
    const int K = p.K;

    // the group's rows of L or columns of R: requested a turn ahead, the first with everything else a workgroup needs at its start
    constexpr int NX = R * R / 4 / NTHR > 0 ? R * R / 4 / NTHR : 1, NG = ROWS * R / 4 / NTHR;
    v4f xv[NX], lv[NG];
    // (buffer loads: rows and columns past the end are out of range and read as zeros, without a branch the other side would wait at; R is
    // below 2^31 bytes, so offsets and lengths fit)
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    auto load_group = [&](int row0) {
        const int n = nrows - row0 < ROWS ? nrows - row0 : ROWS;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(left ? p.L + (size_t)row0 * R : p.R + row0), 0, (left ? n * R : (R - 1) * K + n) * 4, 0x00020000);
#pragma unroll
        for (int e = 0; e < NG; ++e) {
            const int f = tid + e * NTHR, i = f / (ROWS / 4), c = f & (ROWS / 4 - 1);
            const uint32_t off = left ? 16u * f : 4 * c < n ? 4u * (uint32_t)(i * K + 4 * c) : ~0u;
            lv[e] = __builtin_bit_cast(v4f, (u4)__builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
        }
    };
    if (wg * ROWS < nrows) load_group(wg * ROWS);
    {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)p.X, 0, R * R * 4, 0x00020000);
#pragma unroll
        for (int e = 0; e < NX; ++e)
            xv[e] = __builtin_bit_cast(v4f, (u4)__builtin_amdgcn_raw_buffer_load_b128(rs, 16u * (tid + e * NTHR), 0, 0));
    }
    if (MODE == ROT_ERR && QK != 2 && !left) {  // scales of the rows of Z2, four rows to a thread
        constexpr int SLICES = NTHR / (R / 4), PER = SLICES >= 256 ? 1 : 256 / SLICES < 8 ? 256 / SLICES : 8;
        constexpr bool LANES = (R & (R - 1)) == 0;  // the lanes of a wavefront that hold the same rows are a power of two apart
        constexpr int SETS = LANES ? NWV : SLICES;  // left to reduce through the LDS
        const int sl = tid / (R / 4), j = 4 * (tid - sl * (R / 4));
        v4f m = {0.f, 0.f, 0.f, 0.f};
        for (int i = sl; i < p.w.wM; i += PER * SLICES) {  // (a maximum may see the last set more than once)
            v4f f[PER];
#pragma unroll
            for (int k = 0; k < PER; ++k) f[k] = *(const v4f*)(p.ax + (size_t)(i + k * SLICES < p.w.wM ? i + k * SLICES : p.w.wM - 1) * R + j);
#pragma unroll
            for (int k = 0; k < PER; ++k)
#pragma unroll
                for (int u = 0; u < 4; ++u) m[u] = fmaxf(m[u], f[k][u]);
        }
        // (the errors' buffer is not in use yet; a thread past the last whole slice, at rank 96, has nothing to add)
        if constexpr (LANES) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if constexpr (R <= 16) m[u] = max_dpp<0x124>(m[u]);  // rotations within 16 lanes by 4 and by 8
                if constexpr (R <= 32) m[u] = max_dpp<0x128>(m[u]);
                if constexpr (R <= 64) m[u] = max_xor16(m[u]);
                m[u] = max_xor32(m[u]);
            }
            if (lane < R / 4) *(v4f*)(Es + wave * R + j) = m;
        } else if (sl < SLICES) {
            *(v4f*)(Es + sl * R + j) = m;
        }
        __syncthreads();
        if (tid < R) {
            float a = Es[tid];
#pragma unroll
            for (int i = 1; i < SETS; ++i) a = fmaxf(a, Es[i * R + tid]);
            float s, inv;
            rot_scale(a, p.q.top, s, inv);
            sc[tid] = s;
            sc[R + tid] = inv;
        }
    }
#pragma unroll
    for (int e = 0; e < NX; ++e) {
        const int f = tid + e * NTHR, row = f / (R / 4), c = f - row * (R / 4);
        if (f < R * R / 4) *(v4f*)(Xs + row * SX + 4 * c) = xv[e];
    }
    v4f g[H][H];
#pragma unroll
    for (int a = 0; a < H; ++a)
#pragma unroll
        for (int b = 0; b < H; ++b) g[a][b] = v4f{0.f, 0.f, 0.f, 0.f};
    float sq = 0.f;
    const int ha = (wave >> 1) & 1, hb = wave & 1, hg = wave >> 2;  // quadrant of G, half of the group it is contracted over

    for (int row0 = wg * ROWS; row0 < nrows; row0 += nwg * ROWS) {
        // the last group of 128 may be half (N and K are multiples of 64): the upper wavefronts then work on
        // zeros and store nothing
        const bool live = NWV == 4 || row0 + 64 * hg < nrows;
        __syncthreads();  // the previous turn's contraction has read Ls and Es
        if (left) {
#pragma unroll
            for (int e = 0; e < NG; ++e) {
                const int f = tid + e * NTHR, row = f / (R / 4), c = f - row * (R / 4);
                *(v4f*)(Ls + row * SL + 4 * c) = lv[e];
            }
        } else {
#pragma unroll
            for (int e = 0; e < NG; ++e) {
                const int f = tid + e * NTHR, i = f / (ROWS / 4), c = f & (ROWS / 4 - 1);
                *(v4f*)(Ls + i * SR + 4 * c) = lv[e];
            }
        }
        if (row0 + nwg * ROWS < nrows) load_group(row0 + nwg * ROWS);
        __syncthreads();
        v4f z[T];
#pragma unroll
        for (int t = 0; t < T; ++t) z[t] = v4f{0.f, 0.f, 0.f, 0.f};
        {
            const float* bp = Xs + q * SX + l15;
            auto chain = [&](const float* ap, auto step) {
#pragma unroll 4
                for (int s = 0; s < R / 4; ++s) {
                    const float a = ap[s * decltype(step)::value];
#pragma unroll
                    for (int t = 0; t < T; ++t) z[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, bp[4 * s * SX + 16 * t], z[t], 0, 0, 0);
                }
            };
            if (left) chain(Ls + (16 * wave + l15) * SL + q, std::integral_constant<int, 4>{});
            else chain(Ls + q * SR + 16 * wave + l15, std::integral_constant<int, 4 * SR>{});
        }
        float* dl = p.oL + (size_t)(row0 + 16 * wave + 4 * q) * R + l15;  // row 4 q + i, column 16 t + l15
        float* dr = p.oR + (size_t)l15 * K + row0 + 16 * wave + 4 * q;    // row 16 t + l15, columns 4 q ..
        if constexpr (MODE == ROT_ERR) {
            if (left) {
                // (a row's maximum is in 16 lanes: lane i & 3 divides for row i and hands both factors to the others)
                float sv = 1.f, iv = 1.f;
                if constexpr (QK != 2) {
                    float rm[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        rm[i] = 0.f;
#pragma unroll
                        for (int t = 0; t < T; ++t) rm[i] = fmaxf(rm[i], fabsf(z[t][i]));
                        rm[i] = max_row16(rm[i]);
                    }
                    const float lo = l15 & 1 ? rm[1] : rm[0], hi = l15 & 1 ? rm[3] : rm[2];
                    rot_scale(l15 & 2 ? hi : lo, p.q.top, sv, iv);
                }
                for_rows([&](auto row) {
                    constexpr int i = decltype(row)::value;
                    if constexpr (QK == 2) {
#pragma unroll
                        for (int t = 0; t < T; t += 2) {  // (block kinds have rank >= 32: T is even)
                            const int t1 = t + 1 < T ? t + 1 : t;
                            const int eb = rot_block_exp(max_row16(fmaxf(fabsf(z[t][i]), fabsf(z[t1][i]))), p.q);
                            z[t][i] = rot_err_block(z[t][i], eb, p.q);
                            if (t1 > t) z[t1][i] = rot_err_block(z[t1][i], eb, p.q);
                        }
                    } else {
                        const float s = row16_lane<i>(sv), inv = row16_lane<i>(iv);
#pragma unroll
                        for (int t = 0; t < T; ++t) z[t][i] = rot_err<QK>(z[t][i], s, inv, p.q.top);
                    }
                });
            } else if constexpr (QK == 2) {  // a block is 32 rows of the group: this wavefront's 16 and its neighbour's
                float mx[T];
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    float m = fmaxf(fmaxf(fabsf(z[t][0]), fabsf(z[t][1])), fmaxf(fabsf(z[t][2]), fabsf(z[t][3])));
                    m = fmaxf(m, __shfl_xor(m, 16));
                    m = fmaxf(m, __shfl_xor(m, 32));
                    mx[t] = m;
                    red[wave * R + 16 * t + l15] = m;
                }
                __syncthreads();
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const int eb = rot_block_exp(fmaxf(mx[t], red[(wave ^ 1) * R + 16 * t + l15]), p.q);
#pragma unroll
                    for (int i = 0; i < 4; ++i) z[t][i] = rot_err_block(z[t][i], eb, p.q);
                }
            } else {
#pragma unroll
                for (int t = 0; t < T; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) z[t][i] = rot_err<QK>(z[t][i], sc[16 * t + l15], sc[R + 16 * t + l15], p.q.top);
            }
        }
#pragma unroll
        for (int t = 0; t < T; ++t) {
            if (!live) {
            } else if (left) {
#pragma unroll
                for (int i = 0; i < 4; ++i) dl[i * R + 16 * t] = z[t][i];
            } else {
                *(v4f*)(dr + (size_t)16 * t * K) = z[t];
            }
        }
        if constexpr (MODE == ROT_ERR) {
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    sq = __builtin_fmaf(z[t][i], z[t][i], sq);
                    Es[(16 * wave + 4 * q + i) * SL + 16 * t + l15] = z[t][i];
                }
            __syncthreads();
            if (T > 1 || (wave & 3) == 0) {
                const float* bp = Es + (64 * hg + 4 * q) * SL + 16 * H * hb + l15;
                auto contract = [&](auto left_operand) {  // row 16 s + 4 q + u in step (s, u)
#pragma unroll 2
                    for (int s = 0; s < 4; ++s) {
                        v4f av[H];
#pragma unroll
                        for (int a = 0; a < H; ++a) av[a] = left_operand(s, a);
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            float bv[H];
#pragma unroll
                            for (int b = 0; b < H; ++b) bv[b] = bp[(16 * s + u) * SL + 16 * b];
#pragma unroll
                            for (int a = 0; a < H; ++a)
#pragma unroll
                                for (int b = 0; b < H; ++b) g[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a][u], bv[b], g[a][b], 0, 0, 0);
                        }
                    }
                };
                if (left) {
                    const float* ap = Ls + (64 * hg + 4 * q) * SL + 16 * H * ha + l15;
                    contract([&](int s, int a) {
                        v4f v;
#pragma unroll
                        for (int u = 0; u < 4; ++u) v[u] = ap[(16 * s + u) * SL + 16 * a];
                        return v;
                    });
                } else {
                    const float* ap = Ls + (16 * H * ha + l15) * SR + 64 * hg + 4 * q;
                    contract([&](int s, int a) { return *(const v4f*)(ap + 16 * a * SR + 16 * s); });
                }
            }
        }
    }
    if constexpr (MODE == ROT_ERR) {
        const int part = left ? wg : p.w.wL + wg;
        const float c = left ? p.c1 : p.c2;
        const bool owner = T > 1 || (wave & 3) == 0;
        v4f* other = (v4f*)Xs + (wave & 3) * H * H * 64 + lane;  // (Omega has been read)
        if (NWV == 8 && hg == 1 && owner) {
#pragma unroll
            for (int a = 0; a < H; ++a)
#pragma unroll
                for (int b = 0; b < H; ++b) other[(a * H + b) * 64] = g[a][b];
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sq += __shfl_down(sq, o);
        if (lane == 0) red[wave] = sq;
        __syncthreads();
        if (hg == 0 && owner) {
            float* o = p.gp + (size_t)part * R * R + (16 * H * ha + 4 * q) * R + 16 * H * hb + l15;
#pragma unroll
            for (int a = 0; a < H; ++a)
#pragma unroll
                for (int b = 0; b < H; ++b) {
                    if constexpr (NWV == 8) g[a][b] += other[(a * H + b) * 64];
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[(16 * a + i) * R + 16 * b] = c * g[a][b][i];
                }
        }
        if (tid == 0) {
            float v = 0.f;
            for (int w = 0; w < NWV; ++w) v += red[w];
            p.lp[part] = v;
        }
    }
}

// Row maxima of Z2 (row kinds), ahead of rot_z_kernel: a workgroup per 64 columns of R and 16 rows of Z2, a wavefront per 16 of the columns,
// both operands straight into registers.  Latency bounds it, and in long rows the redundant reads of R through the L1.  The workgroups are
// spread over the rows of Z2 and not over narrower sets of columns because a set of maxima is r floats of the state, whose size must not
// grow, and because every workgroup of rot_z_kernel reads all sets.  us alone, a set per 64 columns through the LDS / per 16 columns / this:
// 11200 x 64 and 64 x 2240 5.2 / 3.4 / 3.3, 128 x 2304 13.3 / 6.1 / 5.2, 64 x 65536 14.2 / 34.5 / 12.0, 128 x 65536 37.8 / 103 / 38.8; a
// whole step 32.3 / 23.7 / 23.8, 98.1 / 48.3 / 47.2, 70.7 / 77.3 / 54.6, 231 / 240 / 173.
template <int R>
__global__ __launch_bounds__(256) void rot_max_kernel(RotZParams p)
{
    __shared__ float red[4][16];
    const int lane = threadIdx.x & 63, l15 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = (int)blockIdx.x / p.w.wM, set = (int)blockIdx.x - t * p.w.wM;
    float a[R / 4], b[R / 4], m = 0.f;
#pragma unroll
    for (int s = 0; s < R / 4; ++s) b[s] = p.X[(4 * s + q) * R + 16 * t + l15];
    for (int c0 = 64 * set + 16 * wave; c0 < p.K; c0 += 64 * p.w.wM) {
#pragma unroll
        for (int s = 0; s < R / 4; ++s) a[s] = p.R[(size_t)(4 * s + q) * p.K + c0 + l15];
        v4f z = {0.f, 0.f, 0.f, 0.f};  // rows: columns c0 + 4 q + i of R, column: row 16 t + l15 of Z2
#pragma unroll
        for (int s = 0; s < R / 4; ++s) z = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[s], z, 0, 0, 0);
        m = fmaxf(m, fmaxf(fmaxf(fabsf(z[0]), fabsf(z[1])), fmaxf(fabsf(z[2]), fabsf(z[3]))));
    }
    m = max_xor32(max_xor16(m));
    if (q == 0) red[wave][l15] = m;
    __syncthreads();
    if (threadIdx.x < 16)
        p.ax[(size_t)set * R + 16 * t + threadIdx.x] = fmaxf(fmaxf(red[0][threadIdx.x], red[1][threadIdx.x]), fmaxf(red[2][threadIdx.x], red[3][threadIdx.x]));
}

struct RotStepParams {
    float* X;          // Omega
    float* M;          // momentum
    float* G;          // gradient of this step
    const float* gp;   // its parts, [parts][r][r]
    float* Wh;         // r x r between the two launches of the update (over the first part, which has been added by then)
    const float* lp;   // partial sums of E1^2 (wL) then of E2^2
    float* loss;       // may be null
    int r, wL, parts;
    float inv1, inv2;  // 1 / (N r), 1 / (r K)
    float lr, beta, eps, q, grad_scale;
    int s;
};

// G = grad_scale * (sum of the parts), 64 entries per workgroup, the parts dealt to its W wavefronts, D loads of a thread in
// flight (16 wavefronts, or 4 where the parts are few); the last workgroup sums the loss.  A launch of its own: read by the
// workgroups of the update, the parts (1.8 MB at rank 64) would pass through each of their compute units.
template <int W, int D>
__global__ __launch_bounds__(64 * W) void rot_sum_kernel(RotStepParams p)
{
    __shared__ double red[W][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, rr = p.r * p.r;
    double v = 0.0;
    const bool of_loss = blockIdx.x == gridDim.x - 1;
    if (of_loss) {
        double a = 0.0, b = 0.0;
        for (int i = tid; i < p.parts; i += 64 * W) (i < p.wL ? a : b) += (double)p.lp[i];
        v = a * (double)p.inv1 + b * (double)p.inv2;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    } else {
        const float* gp = p.gp + blockIdx.x * 64 + lane;
        for (int w = wave; w < p.parts; w += D * W) {  // (a part past the last is the last one again, not added)
            float f[D];
#pragma unroll
            for (int k = 0; k < D; ++k) f[k] = gp[(size_t)(w + W * k < p.parts ? w + W * k : p.parts - 1) * rr];
#pragma unroll
            for (int k = 0; k < D; ++k) v += w + W * k < p.parts ? (double)f[k] : 0.0;
        }
    }
    red[wave][lane] = v;
    __syncthreads();
    if (of_loss) {
        if (tid == 0 && p.loss) {
            for (int w = 1; w < W; ++w) v += red[w][0];
            *p.loss = (float)v;
        }
    } else if (wave == 0) {
#pragma unroll
        for (int w = 1; w < W; ++w) v += red[w][lane];
        p.G[blockIdx.x * 64 + lane] = (float)((double)p.grad_scale * v);
    }
}

// The update.  Every r x r product runs on the fp32 matrix instruction; the contraction index is dealt so that lane
// (l15, q) takes k = 16 s + 4 q + u in step (s, u): an operand read along its rows is one 16-byte read per s.
//
// Up to rank 32: one workgroup, a wavefront per 16 x 16 tile.  Its left operand W (a row of tiles of the skew-symmetric matrix)
// stays in registers over all products that use it; Omega and the right operand sit in LDS, with row strides
// of 4 modulo 16 floats, so that all reads of either operand are free of bank conflicts.
template <int R> constexpr int rot_cayley_threads() { return (R / 16) * (R / 16) * 64; }
template <int N>
__device__ __forceinline__ float rot_step_length(const RotStepParams& p, const double* parts)  // of |W|^2
{
    double nrm2 = 0.0;
    for (int w = 0; w < N; ++w) nrm2 += parts[w];
    const float lim = 2.f * p.q / ((float)sqrt(nrm2) + p.eps);
    return p.lr < lim ? p.lr : lim;
}
template <int R>
__global__ __launch_bounds__(rot_cayley_threads<R>()) void rot_cayley_kernel(RotStepParams p)
{
    constexpr int T = R / 16, S = R + 4, NTHR = rot_cayley_threads<R>(), NWV = NTHR / 64;
    __shared__ __attribute__((aligned(16))) float Xs[R * S], Ts[R * S];
    __shared__ double red[NWV];
    const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rb = wave / T, cb = wave % T;  // row and column of tiles
    typedef v4f Left[T];
    Left va;
#pragma unroll
    for (int s = 0; s < T; ++s) {
        const size_t o = (size_t)(16 * rb + l15) * R + 16 * s + 4 * q;
        const v4f m = *(const v4f*)(p.M + o), g = *(const v4f*)(p.G + o);
#pragma unroll
        for (int u = 0; u < 4; ++u) va[s][u] = p.beta * m[u] - g[u];
    }
    for (int e = tid; e < R * R / 4; e += NTHR) {
        const int row = e / (R / 4), c = e - row * (R / 4);
        *(v4f*)(Xs + row * S + 4 * c) = *(const v4f*)(p.X + 4 * e);
    }
    __syncthreads();
    auto product = [&](auto left, auto right) {
        v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < T; ++s) {
            const v4f a = left(s), b = right(s);
#pragma unroll
            for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u], b[u], acc, 0, 0, 0);
        }
        return acc;
    };
    auto cols = [&](const float* m, int s, int j0) {  // entries (16 s + 4 q + u, j0 + l15)
        v4f v;
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = m[(16 * s + 4 * q + u) * S + j0 + l15];
        return v;
    };
    auto rows = [&](const float* m, int s, int i0) { return *(const v4f*)(m + (i0 + l15) * S + 16 * s + 4 * q); };  // entries (i0 + l15, 16 s + 4 q + u)
    auto put = [&](const v4f& d) {
#pragma unroll
        for (int i = 0; i < 4; ++i) Ts[(16 * rb + 4 * q + i) * S + 16 * cb + l15] = d[i];
    };
    const v4f A = product([&](int s) { return va[s]; }, [&](int s) { return rows(Xs, s, 16 * cb); });             // A = (beta M - G) X^T
    put(A);
    __syncthreads();
    v4f d = product([&](int s) { return cols(Xs, s, 16 * rb); }, [&](int s) { return cols(Ts, s, 16 * cb); });    // B = X^T A
    __syncthreads();
    put(d);
    __syncthreads();
    d = product([&](int s) { return rows(Xs, s, 16 * rb); }, [&](int s) { return cols(Ts, s, 16 * cb); });        // X B
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = A[i] - 0.5f * d[i];                                                       // Wh
    __syncthreads();
    put(d);
    __syncthreads();
    double n2 = 0.0;
#pragma unroll
    for (int s = 0; s < T; ++s) {                                                                           // W = Wh - Wh^T
        const v4f a = rows(Ts, s, 16 * rb), b = cols(Ts, s, 16 * rb);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            va[s][u] = a[u] - b[u];
            n2 += (double)va[s][u] * (double)va[s][u];
        }
    }
    if (cb != 0) n2 = 0.0;  // the T wavefronts of a row of tiles hold the same part of W
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n2 += __shfl_down(n2, o);
    if (lane == 0) red[wave] = n2;
    __syncthreads();
    const float alpha = rot_step_length<NWV>(p, red);
    v4f x, y;
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = Xs[(16 * rb + 4 * q + i) * S + 16 * cb + l15];
    auto store = [&](float* dst, const v4f& v) {
#pragma unroll
        for (int i = 0; i < 4; ++i) dst[(16 * rb + 4 * q + i) * R + 16 * cb + l15] = v[i];
    };
    d = product([&](int s) { return va[s]; }, [&](int s) { return cols(Xs, s, 16 * cb); });                       // M = W X;  Y = X + alpha M
    store(p.M, d);
#pragma unroll
    for (int i = 0; i < 4; ++i) y[i] = __builtin_fmaf(alpha, d[i], x[i]);
    for (int it = 0; it < p.s; ++it) {                                                                      // Y <- X + alpha/2 W (X + Y)
        __syncthreads();
        put(x + y);
        __syncthreads();
        d = product([&](int s) { return va[s]; }, [&](int s) { return cols(Ts, s, 16 * cb); });
#pragma unroll
        for (int i = 0; i < 4; ++i) y[i] = __builtin_fmaf(0.5f * alpha, d[i], x[i]);
    }
    store(p.X, y);
}

// From rank 64 on: one compute unit's matrix rate would bound the update (12 r^3 operations), so every 16 columns of Omega have a
// workgroup, with a wavefront per 16 x 16 tile of them: columns of Wh need no other columns of anything that is computed, nor do
// columns of the fixed-point passes once W is there.  W = Wh - Wh^T and its norm need all of Wh, so there are two launches with Wh in
// memory between them.  A workgroup requests everything it reads at once, straight into operand registers; only its own 16
// columns pass through the LDS between products.  The sums are those of the one workgroup.  us
// per step, one workgroup / this: 11200 x 64 and 64 x 2240 32.9 / 27.9, 3456 x 128 and 128 x 1152 (blocks) 88.4 / 48.0, 2304 x 96 and
// 96 x 1152 (blocks) 47.0 / 32.3; the update alone 12.9 / 8.1 at rank 64, 60.4 / 19.4 at 128, of which the matrix cores take 5.8.  Up to rank
// 32 the one workgroup (4.0) is ahead of two launches.
template <int R>
struct RotCols {  // 16 columns of an r x r matrix in the LDS, between two products: entry (k, column l15)
    static constexpr int S = 20;  // row stride in floats: q moves by 16 banks
    float (&m)[R * S];
    __device__ __forceinline__ v4f get(int s, int l15, int q) const
    {
        v4f v;
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = m[(16 * s + 4 * q + u) * S + l15];
        return v;
    }
    __device__ __forceinline__ void put(const v4f& d, int rb, int l15, int q)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) m[(16 * rb + 4 * q + i) * S + l15] = d[i];
    }
};
template <int R>
struct RotSlab {  // left operands of a wavefront's row of tiles, from a row-major matrix in memory: entries (i0 + l15, 16 s + 4 q + u) or, transposed, their mirror
    v4f v[R / 16];
    __device__ __forceinline__ void rows(const float* m, int i0, int l15, int q)
    {
#pragma unroll
        for (int s = 0; s < R / 16; ++s) v[s] = *(const v4f*)(m + (size_t)(i0 + l15) * R + 16 * s + 4 * q);
    }
    __device__ __forceinline__ void cols(const float* m, int i0, int l15, int q)
    {
#pragma unroll
        for (int s = 0; s < R / 16; ++s)
#pragma unroll
            for (int u = 0; u < 4; ++u) v[s][u] = m[(size_t)(16 * s + 4 * q + u) * R + i0 + l15];
    }
    template <typename F>
    __device__ __forceinline__ v4f times(F right) const
    {
        v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < R / 16; ++s) {
            const v4f b = right(s);
#pragma unroll
            for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v[s][u], b[u], acc, 0, 0, 0);
        }
        return acc;
    }
};

template <int R>
__global__ __launch_bounds__(R * 4) void rot_wh_kernel(RotStepParams p)  // Wh = A - 1/2 X (X^T A), A = (beta M - G) X^T
{
    __shared__ float as[R * RotCols<R>::S], bs[R * RotCols<R>::S];
    const int lane = threadIdx.x & 63, l15 = lane & 15, q = lane >> 4, cb = blockIdx.x;
    const int rb = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    RotSlab<R> m, g, xj, xt, xr;
    m.rows(p.M, 16 * rb, l15, q);
    g.rows(p.G, 16 * rb, l15, q);
    xj.rows(p.X, 16 * cb, l15, q);
    xt.cols(p.X, 16 * rb, l15, q);
    xr.rows(p.X, 16 * rb, l15, q);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < R / 16; ++s)
#pragma unroll
        for (int u = 0; u < 4; ++u) m.v[s][u] = p.beta * m.v[s][u] - g.v[s][u];
    RotCols<R> ac{as}, bc{bs};
    const v4f A = m.times([&](int s) { return xj.v[s]; });
    ac.put(A, rb, l15, q);
    __syncthreads();
    bc.put(xt.times([&](int s) { return ac.get(s, l15, q); }), rb, l15, q);
    __syncthreads();
    const v4f d = xr.times([&](int s) { return bc.get(s, l15, q); });
#pragma unroll
    for (int i = 0; i < 4; ++i) p.Wh[(16 * rb + 4 * q + i) * R + 16 * cb + l15] = A[i] - 0.5f * d[i];
}

template <int R>
__global__ __launch_bounds__(R * 4) void rot_update_kernel(RotStepParams p)
{
    constexpr int T = R / 16;
    __shared__ float ts[2][R * RotCols<R>::S];
    __shared__ double red[T];
    const int lane = threadIdx.x & 63, l15 = lane & 15, q = lane >> 4, cb = blockIdx.x;
    const int rb = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t tile = (size_t)(16 * rb + 4 * q) * R + 16 * cb + l15;
    RotSlab<R> w, wt, xj;
    w.rows(p.Wh, 16 * rb, l15, q);
    wt.cols(p.Wh, 16 * rb, l15, q);
    xj.cols(p.X, 16 * cb, l15, q);
    v4f x, y;
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = p.X[tile + (size_t)i * R];
    __builtin_amdgcn_sched_barrier(0);
    double n2 = 0.0;  // (every workgroup forms the whole norm, in the same order)
#pragma unroll
    for (int s = 0; s < T; ++s)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            w.v[s][u] -= wt.v[s][u];
            n2 += (double)w.v[s][u] * (double)w.v[s][u];
        }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n2 += __shfl_down(n2, o);
    if (lane == 0) red[rb] = n2;
    v4f d = w.times([&](int s) { return xj.v[s]; });  // M = W X;  Y = X + alpha M
    __syncthreads();                                 // (a wavefront's X is in registers by then: the columns stored below are this workgroup's own)
    const float alpha = rot_step_length<T>(p, red);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        p.M[tile + (size_t)i * R] = d[i];
        y[i] = __builtin_fmaf(alpha, d[i], x[i]);
    }
    for (int it = 0; it < p.s; ++it) {               // Y <- X + alpha/2 W (X + Y); two buffers: a pass overwrites what the pass before the last read
        RotCols<R> tc{ts[it & 1]};
        tc.put(x + y, rb, l15, q);
        __syncthreads();
        d = w.times([&](int s) { return tc.get(s, l15, q); });
#pragma unroll
        for (int i = 0; i < 4; ++i) y[i] = __builtin_fmaf(0.5f * alpha, d[i], x[i]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) p.X[tile + (size_t)i * R] = y[i];
}

__global__ __launch_bounds__(ROT_TPB) void rot_init_kernel(float* X, float* M, const float* X0, const float* M0, int r)
{
    const int e = blockIdx.x * ROT_TPB + threadIdx.x;
    if (e >= r * r) return;
    X[e] = X0 ? X0[e] : (e / r == e % r ? 1.f : 0.f);
    M[e] = M0 ? M0[e] : 0.f;
}

hipError_t launch_rot_init(const Dims& d, const float* Omega0, const float* Mom0, uint8_t* state, hipStream_t s)
{
    const RotLayout rl = rot_layout(d);
    hipLaunchKernelGGL(rot_init_kernel, dim3((d.r * d.r + ROT_TPB - 1) / ROT_TPB), dim3(ROT_TPB), 0, s,
                       (float*)(state + rl.off_X), (float*)(state + rl.off_M), Omega0, Mom0, d.r);
    return hipGetLastError();
}

// Q2 of the configuration: the branch weight format.
static RotQ rot_q2(const Dims& d)
{
    RotQ q;
    q.kind = d.mxi ? 4 : d.mxb ? (d.mxb_elem == 8 ? 2 : 3) : d.mx ? 1 : 0;
    q.top = q.kind == 0 ? (float)d.qmax_bw : 448.f;
    q.bits = d.mxi ? d.bw_bits : 0;
    return q;
}

template <int R, int MODE, int QK, int NWV>
static hipError_t rot_launch_z(const RotZParams& p, int grid, hipStream_t s)
{
    constexpr int lds = rot_z_lds<R, NWV>();
    const hipError_t e = allow_lds<rot_z_kernel<R, MODE, QK, NWV>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((rot_z_kernel<R, MODE, QK, NWV>), dim3(grid), dim3(64 * NWV), lds, s, p);
    return hipGetLastError();
}

template <int R>
static hipError_t rot_launch_errors(const RotZParams& p, hipStream_t s)
{
    constexpr int NWV = R <= 64 ? 8 : 4;  // (rot_split's group)
    if (p.q.kind <= 1) {
        hipLaunchKernelGGL((rot_max_kernel<R>), dim3(p.w.wM * (R / 16)), dim3(256), 0, s, p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (p.q.kind == 0) return rot_launch_z<R, ROT_ERR, 0, NWV>(p, p.w.wL + p.w.wR, s);
    if (p.q.kind == 1) return rot_launch_z<R, ROT_ERR, 1, NWV>(p, p.w.wL + p.w.wR, s);
    if constexpr (R >= 32) return rot_launch_z<R, ROT_ERR, 2, NWV>(p, p.w.wL + p.w.wR, s);
    return hipErrorInvalidValue;  // (block kinds have rank >= 32)
}

template <int R>
static hipError_t rot_launch_cayley(const RotStepParams& p, hipStream_t s)
{
    if constexpr (R <= 32) {
        hipLaunchKernelGGL((rot_cayley_kernel<R>), dim3(1), dim3(rot_cayley_threads<R>()), 0, s, p);
    } else {
        hipLaunchKernelGGL((rot_wh_kernel<R>), dim3(R / 16), dim3(R * 4), 0, s, p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((rot_update_kernel<R>), dim3(R / 16), dim3(R * 4), 0, s, p);
    }
    return hipGetLastError();
}

template <typename F>
static hipError_t rot_dispatch(int r, F f)
{
    switch (r) {
        case 16: return f(std::integral_constant<int, 16>{});
        case 32: return f(std::integral_constant<int, 32>{});
        case 64: return f(std::integral_constant<int, 64>{});
        case 96: return f(std::integral_constant<int, 96>{});
        default: return f(std::integral_constant<int, 128>{});
    }
}

// Partial results of a step (row maxima, loss and gradient partials) for callers that
// cannot allocate: one array per device, held until the process ends.  Every element a step reads it has written before
// in that same step, so nothing needs clearing between calls; two steps that overlap on one GPU would race on it.
static __device__ __align__(256) uint8_t scratch[LQ_ROT_STATIC_SCRATCH_BYTES];

// The array's device address on the current device (host code must not use the symbol's name as an address), looked up
// once per device.
static hipError_t rot_scratch_ptr(uint8_t** out)
{
    static std::mutex mu;
    static uint8_t* ptr[64] = {nullptr};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        ptr[dev] = (uint8_t*)p;
    }
    *out = ptr[dev];
    return hipSuccess;
}

size_t rot_static_scratch_needed(const Dims& d)
{
    const RotLayout rl = rot_layout(d);
    return rl.total - rl.off_ax;
}

// part: where the step's partial results live (laid out like the state blob's sections from off_ax on): inside the
// state blob, or the per-device array
static hipError_t rot_step_launches(const Dims& d, const float* L, const float* Rm, uint8_t* state, uint8_t* part,
                                    const lq_cayley* cs, float* loss, hipStream_t s);

hipError_t launch_rot_step(const Dims& d, const float* L, const float* Rm, uint8_t* state, const lq_cayley* cs, float* loss,
                           hipStream_t s)
{
    return rot_step_launches(d, L, Rm, state, state + rot_layout(d).off_ax, cs, loss, s);
}

hipError_t launch_rot_step_static(const Dims& d, const float* L, const float* Rm, uint8_t* state, const lq_cayley* cs,
                                  float* loss, hipStream_t s)
{
    uint8_t* part = nullptr;
    const hipError_t e = rot_scratch_ptr(&part);
    if (e != hipSuccess) return e;
    return rot_step_launches(d, L, Rm, state, part, cs, loss, s);
}

static RotZParams rot_z_params(const Dims& d, const float* L, const float* Rm, const float* X, float* oL, float* oR)
{
    RotZParams p;
    p.L = L;
    p.R = Rm;
    p.X = X;
    p.N = (int)d.N;
    p.K = (int)d.K;
    p.w = rot_split(d);
    p.q = rot_q2(d);
    p.oL = oL;
    p.oR = oR;
    p.ax = p.lp = p.gp = nullptr;
    p.c1 = (float)(-2.0 / ((double)d.N * d.r));
    p.c2 = (float)(-2.0 / ((double)d.r * (double)d.K));
    return p;
}

static hipError_t rot_step_launches(const Dims& d, const float* L, const float* Rm, uint8_t* state, uint8_t* part,
                                    const lq_cayley* cs, float* loss, hipStream_t s)
{
    const RotLayout rl = rot_layout(d);
    RotZParams z = rot_z_params(d, L, Rm, (float*)(state + rl.off_X), (float*)(state + rl.off_E1), (float*)(state + rl.off_E2));
    z.ax = (float*)part;
    z.lp = (float*)(part + (rl.off_lp - rl.off_ax));
    z.gp = (float*)(part + (rl.off_gp - rl.off_ax));
    RotStepParams p;
    p.X = (float*)(state + rl.off_X);
    p.M = (float*)(state + rl.off_M);
    p.G = (float*)(state + rl.off_G);
    p.gp = z.gp;
    p.Wh = z.gp;
    p.lp = z.lp;
    p.loss = loss;
    p.r = d.r;
    p.wL = z.w.wL;
    p.parts = z.w.wL + z.w.wR;
    p.inv1 = (float)(1.0 / ((double)d.N * d.r));
    p.inv2 = (float)(1.0 / ((double)d.r * (double)d.K));
    p.lr = cs->lr;
    p.beta = cs->beta;
    p.eps = cs->eps;
    p.q = cs->q;
    p.grad_scale = cs->grad_scale;
    p.s = cs->s;
    return rot_dispatch(d.r, [&](auto rank) {  // (stops at the first launch that fails: no update from an earlier step's parts)
        constexpr int R = decltype(rank)::value;
        hipError_t e = rot_launch_errors<R>(z, s);
        if (e != hipSuccess) return e;
        if (p.parts > 64) hipLaunchKernelGGL((rot_sum_kernel<16, 8>), dim3(R * R / 64 + 1), dim3(1024), 0, s, p);
        else hipLaunchKernelGGL((rot_sum_kernel<4, 16>), dim3(R * R / 64 + 1), dim3(256), 0, s, p);
        e = hipGetLastError();
        return e != hipSuccess ? e : rot_launch_cayley<R>(p, s);
    });
}

hipError_t launch_rot_apply(const Dims& d, const float* L, const float* Rm, const uint8_t* state, float* Lr, float* Rr,
                            hipStream_t s)
{
    const RotZParams p = rot_z_params(d, L, Rm, (const float*)(state + rot_layout(d).off_X), Lr, Rr);
    // (the rotated factors do not depend on Q2 and leave no parts: every group of 64 has a workgroup of its own)
    return rot_dispatch(d.r, [&](auto rank) {
        RotZParams z = p;
        z.w.gL = z.w.wL = (int)(d.N / 64);
        z.w.gR = (int)(d.K / 64);
        return rot_launch_z<decltype(rank)::value, ROT_OUT, 0, 4>(z, z.w.gL + z.w.gR, s);
    });
}

hipError_t launch_rot_unpack(const Dims& d, const uint8_t* state, const lq_rot_view* out, hipStream_t s)
{
    const RotLayout rl = rot_layout(d);
    const size_t rr = (size_t)d.r * d.r * 4;
    struct { float* dst; size_t off, bytes; } parts[5] = {{out->Omega, rl.off_X, rr}, {out->Mom, rl.off_M, rr}, {out->G, rl.off_G, rr},
                                                         {out->E1, rl.off_E1, (size_t)d.N * d.r * 4},
                                                         {out->E2, rl.off_E2, (size_t)d.r * d.K * 4}};
    for (auto& pt : parts) {
        if (!pt.dst) continue;
        const hipError_t e = hipMemcpyAsync(pt.dst, state + pt.off, pt.bytes, hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lq
