// Data-free calibration of the low-rank factors (Section 3.2, Eq. 4; gradients of App. B.2): one Adam step on
//     loss(L, R) = mean ( Q1(W + L R) - W - L R )^2
// for the main quantiser Q1 of the configuration: INT4 in groups of 64 | 128 along K with fp32 scales, SINT4 blocks with
// FP16 scales, MXFP4 or MXINT4 (blocks of 32, E8M0 scale).  Two launches per step:
//   calib_err_kernel   V = W + L R (fp32 FMA chain over ascending j), E = deq(Q1(V)) - V, partial sums of E^2, and the
//                      strips' parts of grad_L = -2/(N K) E R^T and grad_R = -2/(N K) L^T E while E is on the chip
//   calib_adam_kernel  sums the parts, Adam update of L and R, loss = sum of its partials / (N K)
// No atomics: every sum has a fixed order, so a step is reproducible bit for bit.
#include <utility>

#include "lq_internal.h"

namespace lq {

typedef float v4f __attribute__((ext_vector_type(4)));

// A workgroup owns 128 columns of W and a run of row blocks of 16 rows per wavefront.  It leaves one r x 128 part of grad_R
// for its run and one part of grad_L, 16 rows x r, per wavefront and row block.  The runs are as long as they can be with
// every workgroup slot of the device still taken, so that grad_R has few parts.  Up to rank 64 a workgroup has 8 wavefronts
// (half the parts of grad_R that two workgroups of 4 on the same compute unit leave), or 4 up to rank 32 where that shortens
// the longest chain of strips on a compute unit (at rank 64 it would, 1152 x 1152 19.8 us a step instead of 24.2, but leaves more parts
// than states of earlier sizes hold); from rank 96 on the LDS holds 4.  The split decides the size of the state, which a program asks for
// without a device: it counts the 256 compute units of an MI355X and not those of the current device.
constexpr int CALIB_COLS = 128;
struct CalibSplit {
    int waves;      // wavefronts per workgroup
    int cblocks;    // column blocks = parts of grad_L
    int rblocks;    // row blocks
    int splits;     // runs of row blocks = parts of grad_R
    int per;        // row blocks per run
};
static CalibSplit calib_split(const Dims& d, int waves, int slots)
{
    CalibSplit c;
    const int rows = 16 * waves;
    c.waves = waves;
    c.cblocks = (int)((d.K + CALIB_COLS - 1) / CALIB_COLS);
    c.rblocks = (int)((d.N + rows - 1) / rows);
    const int want = slots > c.cblocks ? slots / c.cblocks : 1;
    c.per = (c.rblocks + want - 1) / want;
    c.splits = (c.rblocks + c.per - 1) / c.per;
    return c;
}
static CalibSplit calib_split(const Dims& d)
{
    if (d.r > 64) return calib_split(d, 4, 256);
    const CalibSplit c8 = calib_split(d, 8, 256);
    if (d.r == 64) return c8;
    const CalibSplit c4 = calib_split(d, 4, 512);  // (two share a compute unit)
    const int chain8 = 8 * c8.per, chain4 = (c4.cblocks * c4.splits > 256 ? 8 : 4) * c4.per;
    return chain4 < chain8 ? c4 : c8;
}

CalibLayout calib_layout(const Dims& d)
{
    CalibLayout cl;
    const size_t nl = (size_t)d.N * d.r * 4, nr = (size_t)d.r * d.K * 4;
    size_t o = 0;
    cl.off_L = o;  o = align256(o + nl);
    cl.off_R = o;  o = align256(o + nr);
    cl.off_mL = o; o = align256(o + nl);
    cl.off_vL = o; o = align256(o + nl);
    cl.off_mR = o; o = align256(o + nr);
    cl.off_vR = o; o = align256(o + nr);
    cl.off_gL = o; o = align256(o + nl);
    cl.off_gR = o; o = align256(o + nr);
    cl.off_E = o;  o = align256(o + (size_t)d.N * d.K * 4);
    const CalibSplit c = calib_split(d);
    cl.n_lp = c.cblocks * c.splits;  // one partial per workgroup of calib_err_kernel
    cl.off_lp = o; o = align256(o + (size_t)cl.n_lp * 4);
    cl.off_gLp = o; o = align256(o + (size_t)c.cblocks * nl);
    cl.off_gRp = o; o = align256(o + (size_t)c.splits * nr);
    cl.total = o;
    // The size callers are told never falls below that of the first layout (a loss partial per wavefront of 16 rows and a group,
    // parts of grad_R over up to 16 row ranges): what lq_calib_sizes returned for a layer stays the least it returns.
    {
        const size_t blocks = (size_t)d.N / 16, groups = (size_t)((d.mx || d.mxi) ? d.C64 : d.G);
        size_t parts = 1;
        for (size_t p = 1; p <= 16; ++p) {
            if (blocks % p) continue;
            parts = p;
            if (p * (d.K / 32) >= 256) break;
        }
        const size_t f = align256(align256(cl.off_lp + blocks * ((groups + 3) / 4) * 4 * 4) + parts * nr);
        if (f > cl.total) cl.total = f;
    }
    return cl;
}

// MX block scales and elements (App. A.3), the arithmetic of the MX pack kernels:
// MXFP4: scale byte floor(log2 amax) - 2 + 127 clamped at 0; E2M1 element by the hardware converter (nearest even, saturating)
__device__ __forceinline__ uint32_t mxfp4_scale_byte(float amax)
{
    const int e = (int)((__float_as_uint(amax) >> 23) & 0xFFu) - 2;
    return (amax == 0.0f || e < 0) ? 0u : (uint32_t)e;
}
__device__ __forceinline__ float e8m0_as_float(uint32_t E) { return E ? __uint_as_float(E << 23) : __uint_as_float(0x00400000u); }
__device__ __forceinline__ float e2m1_value(uint32_t c)  // 1 sign, 2 exponent (bias 1), 1 mantissa bit
{
    const uint32_t m = c & 7u;  // (branch-free: a code from 2 on is the top of a float's bits)
    const uint32_t mag = m < 2u ? (m ? 0x3F000000u : 0u) : (m << 22) + (126u << 23);
    return __uint_as_float(mag | (c & 8u) << 28);
}
// MXINT4: shared exponent = the fp32 exponent field of amax; code = clamp(rne(v 2^(2 - s)), -7, 7), value = code 2^(s - 2)
__device__ __forceinline__ float mxint4_round(float v, uint32_t field)
{
    const int s = (int)field - 127;
    const float q = fminf(fmaxf(rintf(ldexpf(v, 2 - s)), -7.0f), 7.0f);
    return ldexpf(q, s - 2);
}
__device__ __forceinline__ float wave_sum_f(float v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = __fadd_rn(v, __shfl_xor(v, o, 64));
    return v;
}

// f(0), f(1), ... with the argument as a compile-time constant
template <typename F, int... k>
__device__ __forceinline__ void for_constants(F f, std::integer_sequence<int, k...>)
{
    (f(std::integral_constant<int, k>{}), ...);
}

struct CalibParams {
    const float *W, *L, *R;
    float* E;
    float* lp;
    float *gLp, *gRp;
    int N, K;
    CalibSplit c;
};

// LDS images: R as a [r][SC] block shared by the workgroup, L as [16][SL] and E as [16][SC] per wavefront, row strides of 4
// modulo 16 floats: 16-byte reads along a row, 16-byte reads of 16 rows at one column and reads of one column over
// rows 4 q + u each touch every bank once per 16 lanes.
constexpr int CALIB_SC = CALIB_COLS + 4;
// (Behind the loop the same memory takes 32 rank indexes of every wavefront's grad_R.)
constexpr int calib_lds(int r, int waves, bool one)
{
    const int images = r * CALIB_SC + waves * 16 * (r + 4 + CALIB_SC), sums = waves * (r < 32 ? r : 32) * CALIB_SC;
    return (one || images > sums ? images : sums) * 4;
}

// Orders a wavefront's own LDS stores before its lanes' reads of each other's values (the LDS serves a wavefront in order).
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_sched_barrier(0); }

// The maximum over the 8 lanes of each half row.
__device__ __forceinline__ float max_row8(float v)
{
    v = max_dpp<0xB1>(v);        // quad_perm [1,0,3,2]
    v = max_dpp<0x4E>(v);        // quad_perm [2,3,0,1]
    return max_dpp<0x141>(v);    // row_half_mirror
}

// All three products on v_mfma_f32_16x16x4_f32 (lane (l15, q) holds rows 4 q + i, column l15 of a 16 x 16 result tile).
// The instruction is, bit for bit, four fused multiply-adds in ascending order of its contraction index, so V = W + L R with
// W as the initial accumulator is exactly the chain that defines V.  A wavefront works alone on strips of 16 rows x 128
// columns: tile (h, u) of the eight holds columns 64 h + 4 l15 + u, so W, E and the rows of R move 16 bytes per lane.
// ONE (runs of one row block): E and L of all strips lie in the LDS, and behind a barrier every wavefront sums grad_R for its
// own 128 / NWV columns.  Otherwise V's registers are, as they lie, the second operand of grad_R (contraction over the strip's
// rows, row 4 q + u in step u), which a wavefront sums over its run in registers; grad_L (contraction over columns) takes E through
// the wavefront's own part of the LDS; there is no barrier inside the run, so wavefronts drift apart and one's loads
// and stores lie beside another's products, and the next strip is requested as soon as the strip's registers are free.  The sum
// over the wavefronts behind the run moves 16 r x 128 floats through the LDS: a run of one block is shorter without it.
// What bounds it: all wavefronts of a short run load, multiply and store at the same time (3456 x 1152 at rank 32: 40 MB, 8 us at 5 TB/s,
// then 5.7 us of the matrix unit, busy 38 % of the launch); long runs the matrix unit (11200 x 2240 at rank 64: 63 %).  Against one kernel form with barriers between all phases,
// dword loads and stores and E read back for grad_R (us a step): 3456 x 1152 rank 16 16.3 -> 14.5, rank 32 22.1 -> 19.8, rank 64
// 30.5 -> 29.9, 4608 x 1152 MXFP4 rank 32 34.0 -> 28.6, 11200 x 2240 rank 16 54.3 -> 46.3, rank 32 75.0 -> 69.2, rank 64 134.4 -> 118.2,
// rank 128 254.5 -> 214.4.  A run of one strip in the other form: 3456 x 1152 rank 32 20.1, rank 64 31.4.
// GT: 16-column tiles per scale group (4: 64 values, 8: 128, 2: MX block of 32).
// Q: 0 INT4 groups (fp32 scale), 1 SINT4 blocks, 2 MXFP4, 3 MXINT4.
template <int R, int Q, int GT, int NWV, bool ONE>
__global__ __launch_bounds__(64 * NWV, R > 64 ? 1 : 2) void calib_err_kernel(CalibParams p)
{
    constexpr int NTHR = 64 * NWV, T = R / 16, SL = R + 4, SC = CALIB_SC;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float* Rs = lds;                                   // [R][SC]      the column block of R
    float* Es = Rs + R * SC + wave * 16 * SC;          // [16][SC]     the wavefront's strip of E
    float* Ls = Rs + R * SC + NWV * 16 * SC + wave * 16 * SL;  // [16][SL] its rows of L
    const int cb = blockIdx.x % p.c.cblocks, split = blockIdx.x / p.c.cblocks;
    const int N = p.N, K = p.K, col0 = cb * CALIB_COLS;
    const bool full = K - col0 >= CALIB_COLS;          // else the last block, of 64 columns
    const int ncol = full ? CALIB_COLS : 64;

    // (an out-of-range column of the last block is loaded from the block's first columns and replaced by zero)
    constexpr int NR = R * CALIB_COLS / 4 / NTHR;
    v4f rv[NR];
#pragma unroll
    for (int e = 0; e < NR; ++e) {
        const int f = tid + e * NTHR, row = f / (CALIB_COLS / 4), c = 4 * (f % (CALIB_COLS / 4));
        rv[e] = *(const v4f*)(p.R + (size_t)row * K + col0 + (c < ncol ? c : c - 64));
    }
    v4f w[2][4], lv[T];
    // (wave-uniform bases with one 32-bit offset per lane: 64-bit lane addresses of every row would not fit beside grad_R)
    const uint32_t wo = 4u * ((uint32_t)(4 * q) * (uint32_t)K + (uint32_t)(4 * l15));
    auto request = [&](int wrow) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float* wp = p.W + (size_t)(wrow + i) * K + col0 + (full ? 64 * h : 0);
                w[h][i] = *(const v4f*)((const char*)wp + wo);
            }
    };
    auto request_l = [&](int wrow) {
#pragma unroll
        for (int e = 0; e < T; ++e) lv[e] = *(const v4f*)((const char*)(p.L + (size_t)wrow * R + 256 * e) + (uint32_t)(16 * lane));
    };
    auto store_l = [&] {
#pragma unroll
        for (int e = 0; e < T; ++e) {
            const int f = lane + e * 64, row = f / (R / 4), c = f - row * (R / 4);
            *(v4f*)(Ls + row * SL + 4 * c) = lv[e];
        }
    };
    constexpr int ROWS = 16 * NWV;
    int wrow = split * p.c.per * ROWS + 16 * wave;
    const int run_end = (split + 1) * p.c.per * ROWS, row_end = run_end < N ? run_end : N;
    const bool any = wrow < row_end;
    if (any) {
        request(wrow);
        request_l(wrow);
    }
#pragma unroll
    for (int e = 0; e < NR; ++e) {
        const int f = tid + e * NTHR, row = f / (CALIB_COLS / 4), c = 4 * (f % (CALIB_COLS / 4));
        *(v4f*)(Rs + row * SC + c) = c < ncol ? rv[e] : v4f{0.f, 0.f, 0.f, 0.f};
    }
    constexpr int CT = ONE ? 8 / NWV : 8;  // 16-column tiles of grad_R a wavefront sums
    v4f gr[T][CT];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) gr[t][c] = v4f{0.f, 0.f, 0.f, 0.f};
    float lsum = 0.f;
    if (any) {
        store_l();
    } else if constexpr (ONE) {  // a strip past N is zeros in grad_R
#pragma unroll
        for (int e = 0; e < T; ++e) lv[e] = v4f{0.f, 0.f, 0.f, 0.f};
        store_l();
#pragma unroll
        for (int i = 0; i < 8; ++i) *(v4f*)(Es + (2 * i + (lane >> 5)) * SC + 4 * (lane & 31)) = v4f{0.f, 0.f, 0.f, 0.f};
    }
    __syncthreads();
    for (; wrow < row_end; wrow = ONE ? row_end : wrow + ROWS) {
        v4f v[8];
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) v[t][i] = t < 4 || full ? w[t >> 2][i][t & 3] : 0.f;
        wave_lds_fence();
        {
            const float* ap = Ls + l15 * SL + q;
            const float* bp = Rs + q * SC + 4 * l15;
#pragma unroll 4
            for (int s = 0; s < R / 4; ++s) {
                const float a = ap[4 * s];
                const v4f b0 = *(const v4f*)(bp + 4 * s * SC), b1 = *(const v4f*)(bp + 4 * s * SC + 64);
#pragma unroll
                for (int t = 0; t < 8; ++t) v[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, t < 4 ? b0[t & 3] : b1[t & 3], v[t], 0, 0, 0);
            }
        }
        constexpr int NG = GT == 8 ? 1 : 2, NT = 8 / NG;  // scale groups a lane has values of (4 rows of each), its tiles in each
        float am[NG][4];
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float a = 0.f;
#pragma unroll
                for (int t = g * NT; t < (g + 1) * NT; ++t) a = fmaxf(a, fabsf(v[t][i]));
                am[g][i] = GT == 2 ? max_row8(a) : max_row16(a);
            }
        // INT / SINT4 scales need correctly rounded divisions: the 16 lanes that share a row's maxima share the work, lane
        // 4 g + i dividing for (g, i) and handing the result to the others (two divisions per lane instead of 2 * 4 * NG)
        float sv = 1.0f, iv = 1.0f;
        if constexpr (Q <= 1) {
            float a = am[0][0];
#pragma unroll
            for (int k = 1; k < 4 * NG; ++k) a = (l15 & (4 * NG - 1)) == k ? am[k >> 2][k & 3] : a;
            if constexpr (Q == 1) {
                sv = f16_bits_value(sint4_scale(a, &iv));
            } else {  // branch-free: an all-zero group takes scale 1
                const float sd = __fdiv_rn(a, 7.0f), id = __fdiv_rn(7.0f, a);
                sv = a == 0.0f ? 1.0f : sd;
                iv = a == 0.0f ? 1.0f : id;
            }
        }
        auto finish = [&](auto k_) {  // scale group k >> 2, row k & 3
            constexpr int k = decltype(k_)::value, g = k >> 2, i = k & 3;
            const float a = am[g][i];
            float s = 1.0f, inv = 1.0f;
            uint32_t eb = 0u;
            if constexpr (Q <= 1) {
                s = row16_lane<k>(sv);
                inv = row16_lane<k>(iv);
            } else if constexpr (Q == 2) {
                eb = mxfp4_scale_byte(a);
                s = e8m0_as_float(eb);
            } else {
                eb = (__float_as_uint(a) >> 23) & 0xFFu;
            }
#pragma unroll
            for (int t = g * NT; t < (g + 1) * NT; ++t) {
                float deq;
                if constexpr (Q <= 1) {
                    float c = rintf(__fmul_rn(v[t][i], inv));
                    c = fminf(fmaxf(c, -7.0f), 7.0f);
                    deq = __fmul_rn(c, s);
                } else if constexpr (Q == 2) {
                    const uint32_t code = a != 0.0f ? (__builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, v[t][i], 0.0f, s, 0) & 0xFu) : 0u;
                    deq = __fmul_rn(e2m1_value(code), s);
                } else {
                    deq = mxint4_round(v[t][i], eb);
                }
                const float e = __fsub_rn(deq, v[t][i]);
                v[t][i] = e;
                lsum = __builtin_fmaf(e, e, lsum);
            }
            if constexpr (Q == 2) __builtin_amdgcn_sched_barrier(0);  // (interleaved, the element decodings take 50 registers more)
        };
        for_constants(finish, std::make_integer_sequence<int, 4 * NG>{});
        // E is not read again in a step: non-temporal, it leaves W and the gradient parts in the caches (us per step, steps back
        // to back, cached / non-temporal: 3456 x 1152 rank 32 23.8 / 22.3, rank 64 31.5 / 31.1, 4608 x 1152 rank 128 72.6 / 71.3, 11200 x 2240 rank 32
        // 77.6 / 75.6, rank 64 138.9 / 134.6)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const v4f e = {v[4 * h][i], v[4 * h + 1][i], v[4 * h + 2][i], v[4 * h + 3][i]};
                *(v4f*)(Es + (4 * q + i) * SC + 64 * h + 4 * l15) = e;
                if (h == 0 || full) __builtin_nontemporal_store(e, (v4f*)((char*)(p.E + (size_t)(wrow + i) * K + col0 + 64 * h) + wo));
            }
        __builtin_amdgcn_sched_barrier(0);
        // grad_R: contraction over the strip's rows, row 4 q + u in step u
        if constexpr (!ONE) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const float a = Ls[(4 * q + u) * SL + 16 * t + l15];
#pragma unroll
                    for (int c = 0; c < 8; ++c) gr[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, v[c][u], gr[t][c], 0, 0, 0);
                }
        }
        const bool more = !ONE && wrow + ROWS < row_end;
        constexpr bool LATE = R == 64;  // (no registers left for the rows of L under grad_L; they come from the L2)
        if (more) {
            request(wrow + ROWS);
            if (!LATE) request_l(wrow + ROWS);
        }
        wave_lds_fence();
        // grad_L of the strip's rows: contraction over the block's columns, column 16 s + 4 q + u in step (s, u); R first, so that
        // a lane ends with four consecutive rank indexes of its row
        {
            v4f gl[T];
#pragma unroll
            for (int t = 0; t < T; ++t) gl[t] = v4f{0.f, 0.f, 0.f, 0.f};
            const float* ap = Es + l15 * SC + 4 * q;
            const float* bp = Rs + l15 * SC + 4 * q;
#pragma unroll R == 64 && !ONE ? 1 : 2
            for (int s = 0; s < CALIB_COLS / 16; ++s) {
                const v4f a = *(const v4f*)(ap + 16 * s);
                v4f b[T];
#pragma unroll
                for (int t = 0; t < T; ++t) b[t] = *(const v4f*)(bp + 16 * t * SC + 16 * s);
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int t = 0; t < T; ++t) gl[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[t][u], a[u], gl[t], 0, 0, 0);
            }
#pragma unroll
            for (int t = 0; t < T; ++t) *(v4f*)((char*)(p.gLp + ((size_t)cb * N + wrow) * R + 16 * t) + 4u * (uint32_t)(l15 * R + 4 * q)) = gl[t];
        }
        if (more && LATE) request_l(wrow + ROWS);
        if (more) store_l();  // (grad_R has read the strip's rows of L)
        wave_lds_fence();     // the strip's reads of Es come before the next one's stores
    }
    if constexpr (ONE) {
        // one strip per wavefront: grad_R of the wavefront's columns over all the block's rows, row 16 s + 4 q + u in step (s, u);
        // E first, so that a lane ends with four consecutive columns of one rank index
        __syncthreads();
        const float* ap = Rs + R * SC + 4 * q * SC + 16 * CT * wave + l15;
        const float* bp = Rs + R * SC + NWV * 16 * SC + 4 * q * SL + l15;
#pragma unroll 2
        for (int s = 0; s < NWV; ++s)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float a[CT], b[T];
#pragma unroll
                for (int c = 0; c < CT; ++c) a[c] = ap[(16 * s + u) * SC + 16 * c];
#pragma unroll
                for (int t = 0; t < T; ++t) b[t] = bp[(16 * s + u) * SL + 16 * t];
#pragma unroll
                for (int t = 0; t < T; ++t)
#pragma unroll
                    for (int c = 0; c < CT; ++c) gr[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c], b[t], gr[t][c], 0, 0, 0);
            }
        if (16 * CT * wave < ncol) {
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    *(v4f*)(p.gRp + ((size_t)split * R + 16 * t + l15) * K + col0 + 16 * (CT * wave + c) + 4 * q) = gr[t][c];
        }
    } else {
        // the wavefronts' parts of grad_R, added in order, 32 rank indexes at a time (the whole LDS is free by now)
        constexpr int TR = T < 2 ? T : 2;
        static_assert(T % TR == 0, "whole turns");
        float* Gs = lds + wave * 16 * TR * SC;
        __syncthreads();
#pragma unroll
        for (int t0 = 0; t0 < T; t0 += TR) {
            if (t0) __syncthreads();
#pragma unroll
            for (int t = 0; t < TR; ++t)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        *(v4f*)(Gs + (16 * t + 4 * q + i) * SC + 64 * h + 4 * l15) =
                            v4f{gr[t0 + t][4 * h][i], gr[t0 + t][4 * h + 1][i], gr[t0 + t][4 * h + 2][i], gr[t0 + t][4 * h + 3][i]};
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 16 * TR * CALIB_COLS / 4 / NTHR; ++e) {
                const int f = tid + e * NTHR, row = f / (CALIB_COLS / 4), c = 4 * (f % (CALIB_COLS / 4));
                v4f sum = *(const v4f*)(lds + row * SC + c);
#pragma unroll
                for (int k = 1; k < NWV; ++k) {
                    const v4f x = *(const v4f*)(lds + (k * 16 * TR + row) * SC + c);
#pragma unroll
                    for (int i = 0; i < 4; ++i) sum[i] = __fadd_rn(sum[i], x[i]);
                }
                if (c < ncol) *(v4f*)(p.gRp + ((size_t)split * R + 16 * t0 + row) * K + col0 + c) = sum;
            }
        }
    }
    __syncthreads();
    lsum = wave_sum_f(lsum);
    if (lane == 0) lds[wave] = lsum;
    __syncthreads();
    if (tid == 0) {
        float v = lds[0];
#pragma unroll
        for (int k = 1; k < NWV; ++k) v = __fadd_rn(v, lds[k]);
        p.lp[blockIdx.x] = v;
    }
}

struct AdamParams {
    float lr, b1, b2, eps, ic1, ic2;  // ic = 1 / (1 - beta^t)
};

// One thread per parameter: the N x r values of L, then the r x K values of R; the parts of its gradient are added in order
// and scaled.  Block 0 also sums the loss partials (thread-strided, a fixed shuffle tree per wavefront, then the four
// wavefronts in order).
struct AdamArrays {
    float *p, *m, *v, *g;
    const float* part;
    int parts;
    size_t n;
};
__global__ __launch_bounds__(256) void calib_adam_kernel(AdamArrays aL, AdamArrays aR, float gscale, AdamParams a, const float* lp,
                                                         int n_lp, float inv_count, float* loss)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx < aL.n + aR.n) {
        const bool isL = idx < aL.n;
        const AdamArrays& x = isL ? aL : aR;
        const size_t i = isL ? idx : idx - aL.n;
        const float m0 = x.m[i], v0 = x.v[i], p0 = x.p[i];
        float sum = 0.f;
        for (int sp = 0; sp < x.parts; sp += 16) {  // 16 loads in flight; a part past the last is the last one again, not added
            float f[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) f[k] = x.part[(size_t)(sp + k < x.parts ? sp + k : x.parts - 1) * x.n + i];
#pragma unroll
            for (int k = 0; k < 16; ++k) sum = __fadd_rn(sum, sp + k < x.parts ? f[k] : 0.f);
        }
        const float g = __fmul_rn(gscale, sum);
        x.g[i] = g;
        const float mm = __fadd_rn(__fmul_rn(a.b1, m0), __fmul_rn(1.0f - a.b1, g));
        const float vv = __fadd_rn(__fmul_rn(a.b2, v0), __fmul_rn(1.0f - a.b2, __fmul_rn(g, g)));
        x.m[i] = mm;
        x.v[i] = vv;
        const float den = __fadd_rn(__fsqrt_rn(__fmul_rn(vv, a.ic2)), a.eps);
        x.p[i] = __fsub_rn(p0, __fdiv_rn(__fmul_rn(a.lr, __fmul_rn(mm, a.ic1)), den));
    }
    if (loss && blockIdx.x == 0) {  // block-uniform
        __shared__ float s_part[4];
        float s = 0.f;
#pragma unroll 8
        for (int i = threadIdx.x; i < n_lp; i += 256) s = __fadd_rn(s, lp[i]);
        s = wave_sum_f(s);
        if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0)
            *loss = __fmul_rn(__fadd_rn(__fadd_rn(s_part[0], s_part[1]), __fadd_rn(s_part[2], s_part[3])), inv_count);
    }
}

// Copies (or zero fills) of whole sections, all in one launch; every length is a multiple of 4 floats and every section
// starts 16-byte aligned.
constexpr int CALIB_MAX_PARTS = 9;
struct CalibCopy {
    v4f* dst[CALIB_MAX_PARTS];
    const v4f* src[CALIB_MAX_PARTS];  // null: zeros
    size_t end[CALIB_MAX_PARTS];      // running sums of the lengths, in v4f
    int n;
};
__global__ __launch_bounds__(256) void calib_copy_kernel(CalibCopy c)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < c.end[c.n - 1]; i += (size_t)gridDim.x * 256) {
        size_t begin = 0;
        int k = 0;
        for (; i >= c.end[k]; ++k) begin = c.end[k];
        c.dst[k][i - begin] = c.src[k] ? c.src[k][i - begin] : v4f{0.f, 0.f, 0.f, 0.f};
    }
}
static void calib_copy_add(CalibCopy& c, void* dst, const void* src, size_t bytes)
{
    c.dst[c.n] = (v4f*)dst;
    c.src[c.n] = (const v4f*)src;
    c.end[c.n] = (c.n ? c.end[c.n - 1] : 0) + bytes / 16;
    ++c.n;
}
static hipError_t calib_copy_run(const CalibCopy& c, hipStream_t s)
{
    if (c.n == 0) return hipSuccess;
    // (a launch has fewer than 2^32 threads: an error matrix of 64 GB takes more than one turn)
    const size_t blocks = (c.end[c.n - 1] + 255) / 256, cap = (size_t)1 << 22;
    hipLaunchKernelGGL(calib_copy_kernel, dim3((unsigned)(blocks < cap ? blocks : cap)), dim3(256), 0, s, c);
    return hipGetLastError();
}

hipError_t launch_calib_init(const Dims& d, const float* L, const float* R, uint8_t* state, hipStream_t s)
{
    const CalibLayout cl = calib_layout(d);
    CalibCopy c;
    c.n = 0;
    calib_copy_add(c, state + cl.off_L, L, (size_t)d.N * d.r * 4);
    calib_copy_add(c, state + cl.off_R, R, (size_t)d.r * d.K * 4);
    calib_copy_add(c, state + cl.off_mL, nullptr, cl.off_gL - cl.off_mL);  // moments start at zero (one contiguous range: mL, vL, mR, vR)
    return calib_copy_run(c, s);
}

template <auto KERNEL>
static hipError_t calib_launch_err(const CalibParams& p, int lds, hipStream_t s)
{
    const hipError_t e = allow_lds<KERNEL>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(KERNEL, dim3((unsigned)(p.c.cblocks * p.c.splits)), dim3(64 * p.c.waves), lds, s, p);
    return hipGetLastError();
}

template <int R, int NWV, bool ONE>
static hipError_t calib_err_form(const Dims& d, const CalibParams& p, hipStream_t s)
{
    constexpr int lds = calib_lds(R, NWV, ONE);
    if (d.mxi) return calib_launch_err<calib_err_kernel<R, 3, 2, NWV, ONE>>(p, lds, s);
    if (d.mx) return calib_launch_err<calib_err_kernel<R, 2, 2, NWV, ONE>>(p, lds, s);
    if (d.ga) return calib_launch_err<calib_err_kernel<R, 1, 4, NWV, ONE>>(p, lds, s);
    if (d.g == 64) return calib_launch_err<calib_err_kernel<R, 0, 4, NWV, ONE>>(p, lds, s);
    return calib_launch_err<calib_err_kernel<R, 0, 8, NWV, ONE>>(p, lds, s);
}
template <int R, int NWV>
static hipError_t calib_err(const Dims& d, const CalibParams& p, hipStream_t s)
{
    return p.c.per == 1 ? calib_err_form<R, NWV, true>(d, p, s) : calib_err_form<R, NWV, false>(d, p, s);
}

hipError_t launch_calib_step(const Dims& d, const float* W, uint8_t* state, int step, const lq_adam* ad, float* loss,
                             hipStream_t s)
{
    const CalibLayout cl = calib_layout(d);
    CalibParams p;
    p.W = W;
    p.L = (float*)(state + cl.off_L);
    p.R = (float*)(state + cl.off_R);
    p.E = (float*)(state + cl.off_E);
    p.lp = (float*)(state + cl.off_lp);
    p.gLp = (float*)(state + cl.off_gLp);
    p.gRp = (float*)(state + cl.off_gRp);
    p.N = (int)d.N;
    p.K = (int)d.K;
    p.c = calib_split(d);
    hipError_t e;
    switch (d.r) {
        case 16: e = p.c.waves == 8 ? calib_err<16, 8>(d, p, s) : calib_err<16, 4>(d, p, s); break;
        case 32: e = p.c.waves == 8 ? calib_err<32, 8>(d, p, s) : calib_err<32, 4>(d, p, s); break;
        case 64: e = calib_err<64, 8>(d, p, s); break;
        case 96: e = calib_err<96, 4>(d, p, s); break;
        default: e = calib_err<128, 4>(d, p, s); break;
    }
    if (e != hipSuccess) return e;  // (the parts in the state are an earlier step's: no update from them)
    AdamParams a;
    a.lr = ad->lr;
    a.b1 = ad->beta1;
    a.b2 = ad->beta2;
    a.eps = ad->eps;
    a.ic1 = (float)(1.0 / (1.0 - pow((double)ad->beta1, (double)step)));
    a.ic2 = (float)(1.0 / (1.0 - pow((double)ad->beta2, (double)step)));
    const size_t nL = (size_t)d.N * d.r, nR = (size_t)d.r * d.K;
    const AdamArrays aL = {(float*)(state + cl.off_L), (float*)(state + cl.off_mL), (float*)(state + cl.off_vL),
                           (float*)(state + cl.off_gL), p.gLp, p.c.cblocks, nL};
    const AdamArrays aR = {(float*)(state + cl.off_R), (float*)(state + cl.off_mR), (float*)(state + cl.off_vR),
                           (float*)(state + cl.off_gR), p.gRp, p.c.splits, nR};
    hipLaunchKernelGGL(calib_adam_kernel, dim3((unsigned)((nL + nR + 255) / 256)), dim3(256), 0, s, aL, aR,
                       (float)(-2.0 / ((double)d.N * (double)d.K)), a, p.lp, cl.n_lp, (float)(1.0 / ((double)d.N * (double)d.K)), loss);
    return hipGetLastError();
}

hipError_t launch_calib_unpack(const Dims& d, const uint8_t* state, const lq_calib_view* out, hipStream_t s)
{
    const CalibLayout cl = calib_layout(d);
    const size_t nl = (size_t)d.N * d.r * 4, nr = (size_t)d.r * d.K * 4;
    const struct { float* dst; size_t off, bytes; } parts[CALIB_MAX_PARTS] = {
        {out->L, cl.off_L, nl},   {out->R, cl.off_R, nr},   {out->mL, cl.off_mL, nl}, {out->vL, cl.off_vL, nl},
        {out->mR, cl.off_mR, nr}, {out->vR, cl.off_vR, nr}, {out->gL, cl.off_gL, nl}, {out->gR, cl.off_gR, nr},
        {out->E, cl.off_E, (size_t)d.N * d.K * 4}};
    CalibCopy c;
    c.n = 0;
    for (auto& p : parts) {
        if (!p.dst) continue;
        if ((uintptr_t)p.dst % 16) {  // (the views' alignment is the caller's)
            const hipError_t e = hipMemcpyAsync(p.dst, state + p.off, p.bytes, hipMemcpyDeviceToDevice, s);
            if (e != hipSuccess) return e;
        } else {
            calib_copy_add(c, p.dst, state + p.off, p.bytes);
        }
    }
    return calib_copy_run(c, s);
}

}  // namespace lq
