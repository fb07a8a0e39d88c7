// Per-call activation kernel, INT family (Section 3.4 and the low-rank branch of Fig. 1).
// One pass over X does, per token row:
//   sx = amax/7,      xq = rne(x * 7/amax)          4-bit main codes (stored as 6-bit fields s00mmm)
//   sxb = amax/qa,    xb = rne(x * qa/amax)         branch codes, kept in registers only
//   accT = xb . rq^T  (int8 MFMA, int32)            skinny contraction with Q2(R)
//   T = (float(accT) * sxb) * sr ;  st = max|T|/qa ;  tq = rne(T * qa/max|T|)
// SINT4 blocks (App. A.3; template flag GA): the main codes take one FP16 scale per 64-chunk of K instead
// of one scale per token, sx[m,g] = fp16(amax_g / 7), codes clamp(rne(x * fl(1 / sx))); the branch is unchanged.
//
// Decomposition: a workgroup of NW = 4 or 8 wavefronts owns 16 token rows; lane l of every wavefront
// works on row l%16 and on the 16-value quarter l/16 of each 64-deep K chunk, which is
// exactly the A-operand layout of v_mfma_i32_16x16x64_i8.  In small batches a workgroup owns 16 / CS rows and the 16 rows of
// the operand are CS chunks of each: a product per chunk, the other chunks' rows zeroed, leaves a row's sum spread over CS rows
// of the result, which are added at the end (whole numbers: the same sum).  The 64-chunks of K are dealt
// round-robin to the wavefronts, so a whole row block lives in registers between the
// amax pass and the quantisation pass: X is read from HBM once.  Rows too long for that (MAXC = 0) are
// streamed twice through a two-chunk ring instead: once for the amax, once for the codes (the second read
// comes from the caches: a workgroup's 16 rows are at most a few hundred KB).
#include "lq_internal.h"

namespace lq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned short us2 __attribute__((ext_vector_type(2)));

struct ActParams {
    const void* X;
    int64_t ldx;
    int M, K, C64, r, rp;
    float qa;  // qmax of the branch activation format
    const float* rg;  // reciprocals of the smoothing vector (smoothing variant only)
    const int8_t* rq;
    const float* sr;
    uint8_t* xq;
    float* sx;
    uint32_t* sxg;  // SINT4 blocks: FP16 bits of the block scales (sxg_index), tiles128 = 128-row tiles
    int tiles128, Mp;
    int8_t* tq;
    float* st;
    int8_t* dbg_xb;
    float* dbg_sxb;
    int32_t* dbg_accT;
    float* dbg_T;
    BlobTag tag;        // header of the activation blob (written by the first workgroup)
    uint32_t* tag_dst;
};

template <bool BF16>
struct XChunk;

template <>
struct XChunk<true> {  // 16 bf16 values = 8 dwords
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
struct XChunk<false> {  // 16 fp32 values
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

// Smoothing variant: 16 values of X (bf16 or fp32 source) times the reciprocals of the smoothing vector,
// held as fp32 (the products are no longer bf16 numbers).
template <bool BF16IN>
__device__ __forceinline__ void load_smoothed(XChunk<false>& xc, const void* X, size_t elem, const float* rg, bool ok)
{
    float raw[16];
    if constexpr (BF16IN) {
        XChunk<true> t;
        t.load(X, elem, ok);
#pragma unroll
        for (int i = 0; i < 16; ++i) raw[i] = t.get(i);
    } else {
        XChunk<false> t;
        t.load(X, elem, ok);
#pragma unroll
        for (int i = 0; i < 16; ++i) raw[i] = t.get(i);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v4i g = {0, 0, 0, 0};
        if (ok) g = ((const v4i*)rg)[q];
#pragma unroll
        for (int i = 0; i < 4; ++i) xc.v[4 * q + i] = __fmul_rn(raw[4 * q + i], __int_as_float(g[i]));
    }
}

__device__ __forceinline__ void scales(float amax, float qmax, float* s, float* inv)
{
    if (amax == 0.0f) {
        *s = 1.0f;
        *inv = 1.0f;
    } else {
        *s = amax / qmax;
        *inv = qmax / amax;
    }
}

// round-to-nearest-even of a value with |u| < 2^22, returned in the low bits (two's complement)
__device__ __forceinline__ uint32_t rne_bits(float u) { return __float_as_uint(__fadd_rn(u, 12582912.0f)); }

// 16 values in [-7, 7] (already scaled, fp32) -> their nearest integers as 6-bit sign-magnitude fields, code i at bits
// 6i .. 6i+5 of three dwords.  The field s00mmm is the E2M3 pattern of +-m/8, so this is the hardware FP6 converter
// applied to v/8 (round to nearest even; the scale operand divides).  The two-source converter interleaves its
// sources (result position 2j holds a[j], 2j+1 holds b[j]); only the lower halves of the sources are defined, the
// codes of the upper halves (result dwords 3..5) are not used.
__device__ __forceinline__ void f6_codes16(const float (&v)[16], uint32_t (&out)[3])
{
    typedef float v8f __attribute__((ext_vector_type(8)));
    typedef float v16f __attribute__((ext_vector_type(16)));
    typedef unsigned int v6u __attribute__((ext_vector_type(6)));
    const v8f ev = {v[0], v[2], v[4], v[6], v[8], v[10], v[12], v[14]};
    const v8f od = {v[1], v[3], v[5], v[7], v[9], v[11], v[13], v[15]};
    const v16f a = __builtin_shufflevector(ev, ev, 0, 1, 2, 3, 4, 5, 6, 7, -1, -1, -1, -1, -1, -1, -1, -1);
    const v16f b = __builtin_shufflevector(od, od, 0, 1, 2, 3, 4, 5, 6, 7, -1, -1, -1, -1, -1, -1, -1, -1);
    const float sc = 8.0f;
    v6u c = __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(a, b, sc);
    // The converter writes its result registers over several passes while still reading its sources, and the
    // register allocator is not told: the sources are kept live past it so that the result cannot land on them.  (The
    // result passes through the statement: one that only reads the sources may be moved ahead of the conversion.)
    asm volatile("" : "+v"(c) : "v"(a), "v"(b), "v"(sc));
    out[0] = c[0];
    out[1] = c[1];
    out[2] = c[2];
}

// Chunks of R a wavefront of eight holds or has requested: what its registers leave, at most four (us, two / this: 2 x 1152 rank 16 3.9 / 3.5, 300 x
// 1152 rank 32 5.3 / 4.9, 64 x 2240 rank 64 7.4 / 7.1, 71 x 4544 rank 128 13.7 / 13.3, with 16 rows to a workgroup).  With four wavefronts the workgroups of a
// compute unit cover for each other and registers are better spent on them.  Two as well from rank 96 on for rows of at most three chunks per wavefront, 16 of
// which share a workgroup: most wavefronts have one or two, and R past them, requested and not used, held the others up (SINT4, four / two: 2 x
// 1024 rank 128 6.9 / 6.3, 400 x 768 rank 128 6.9 / 6.2, 1024 x 256 rank 96 5.6 / 5.1, 400 x 640 rank 128 6.1 / 5.6).
constexpr int act_int_ring(bool bf16in, int maxc, int njb, bool sm, bool ga, int nw, int cs)
{
    if (cs == 1 && maxc == 3 && njb >= 6) return 2;
    const int rows = maxc * (bf16in && !sm && !ga ? 8 : 16), left = njb > 0 ? (208 - rows - 4 * njb) / (4 * njb) : 0;
    return maxc == 0 || nw == 4 || (sm && !bf16in && maxc == 9) || left < 2 ? 2 : left < 4 ? left : 4;
}

// BF16IN: element type of X; SM: smoothing variant (X times stored reciprocals, row held as fp32).
template <bool BF16IN, int MAXC, int NJB, bool SM, bool GA, int NW, int CS>
__global__ __launch_bounds__(NW * 64) void act_int_kernel(ActParams p)
{
    write_tag(p.tag_dst, p.tag);
    constexpr bool BF16 = BF16IN && !SM;  // representation of the row in registers
    __shared__ float s_amax[NW][16];
    __shared__ float s_sxb[16];
    __shared__ int s_acc[NW][NJB > 0 ? NJB : 1][64][4];  // [wave][j block][lane][4]
    __shared__ float s_tmax[NW][16];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // scalar: with smoothing, whose row is fp32 in registers, 8192 x 2240 took 29.6 us with it in a vector register and takes 18.0
    const int r16 = lane & 15, kq = lane >> 4;
    constexpr int RW = 16 / CS;                      // rows per workgroup; a wavefront's turn is CS chunks of them
    const int cs = r16 / RW, row = blockIdx.x * RW + (r16 & (RW - 1));
    const bool row_ok = row < p.M;
    const int C64 = p.C64;
    constexpr int njb = NJB;  // rank / 16

    constexpr bool STREAM = MAXC == 0;
    constexpr int NS = STREAM ? 2 : MAXC;            // chunk slots in registers
    const int nmy = (C64 - wave + NW - 1) / NW;      // (STREAM) chunks of this wavefront: c = wave + NW * ci, ci < nmy
    static_assert(!STREAM || CS == 1, "the streamed form takes one chunk at a time");
    XChunk<BF16> xc[NS];
    auto load_x = [&](XChunk<BF16>& ch, int ci) {
        const int c = CS * (wave + NW * ci) + cs;
        const size_t koff = (size_t)c * 64 + kq * 16;
        if constexpr (SM)
            load_smoothed<BF16IN>(ch, p.X, (size_t)row * p.ldx + koff, p.rg + (c < C64 ? koff : 0), row_ok && c < C64);
        else
            ch.load(p.X, (size_t)row * p.ldx + koff, row_ok && c < C64);
    };
#pragma unroll
    for (int ci = 0; ci < NS; ++ci) load_x(xc[ci], ci);

    // Operands that do not depend on X are requested now, so that their latency overlaps the
    // load of X: the Q2(R) fragments of this wavefront's first chunks (later ones are fetched RD - 1
    // chunks ahead inside the loop) and the row scales of R.
    constexpr int NJA = NJB > 0 ? NJB : 1;
    constexpr int RD = act_int_ring(BF16IN, MAXC, NJB, SM, GA, NW, CS);
    v4i bv[RD][NJA];
    auto load_rq = [&](v4i (&dst)[NJA], int t) {
        int c = CS * (wave + NW * (t / CS)) + t % CS;
        c = c < C64 ? c : C64 - 1;  // clamped: a fragment past the end is fetched but not used
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) dst[jb] = *(const v4i*)(p.rq + ((size_t)((size_t)c * NJB + jb) * 64 + lane) * 16);
    };
#pragma unroll
    for (int k = 0; k < RD - 1; ++k)
        if (k < CS * NS) load_rq(bv[k], k);
    constexpr int PW = NJB <= 2 ? 1 : NW;        // wavefronts that re-quantise the intermediate
    constexpr int NT = (NJA + PW - 1) / PW;      // column blocks each of them takes
    float srj[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) srj[t] = p.sr[(wave + PW * t < NJB ? wave + PW * t : 0) * 16 + r16];

    // ---- per-row amax -------------------------------------------------------------------
    float a = 0.f;
    us2 m2 = {0, 0};  // |bf16| is monotonic in its low 15 bits: packed unsigned 16-bit max, two values per op
    auto amax_chunk = [&](const XChunk<BF16>& ch) {
        if constexpr (BF16) {
#pragma unroll
            for (int d = 0; d < 8; ++d) m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(us2, ch.w[d] & 0x7FFF7FFFu));
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) a = fmaxf(a, fabsf(ch.get(i)));
        }
    };
    if constexpr (STREAM) {
        for (int ci0 = 0; ci0 < nmy; ci0 += 2) {
#pragma unroll
            for (int sl = 0; sl < 2; ++sl) {
                amax_chunk(xc[sl]);               // (a slot past the end holds zeros)
                load_x(xc[sl], ci0 + sl + 2);
            }
        }
        // second pass: the ring starts over
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) load_x(xc[sl], sl);
    } else {
#pragma unroll
        for (int ci = 0; ci < NS; ++ci) amax_chunk(xc[ci]);
    }
    if constexpr (BF16) {
        const uint32_t mm = m2[0] > m2[1] ? m2[0] : m2[1];
        a = __uint_as_float(mm << 16);
    }
    a = max_xor16(a);
    a = max_xor32(a);
    if constexpr (CS > 1) a = max_dpp<0x128>(a);  // the row's other chunks: rotations within 16 lanes by 8 and by 4
    if constexpr (CS > 2) a = max_dpp<0x124>(a);
    if (kq == 0) s_amax[wave][r16] = a;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) a = fmaxf(a, s_amax[w][r16]);

    float inv4 = a == 0.0f ? 1.0f : 7.0f / a, invb = a == 0.0f ? 1.0f : p.qa / a;
    if (wave == NW - 1 && kq == 0) {  // (the scales themselves: by the wavefront with the fewest chunks)
        const float s4 = a == 0.0f ? 1.0f : a / 7.0f, sb = a == 0.0f ? 1.0f : a / p.qa;
        if constexpr (!GA) p.sx[row] = s4;
        s_sxb[r16] = sb;
        if (p.dbg_sxb && row_ok) p.dbg_sxb[row] = sb;
        if (p.r == 0) p.st[row] = 1.0f;
    }

    v4i acc[NJB > 0 ? NJB : 1];
#pragma unroll
    for (int jb = 0; jb < NJB; ++jb) acc[jb] = v4i{0, 0, 0, 0};

    const int rb = row >> 5;
    // one 64-chunk: main codes (and the block scale with SINT4 blocks), branch codes, skinny contraction
    auto code_chunk = [&](const XChunk<BF16>& ch, const int ci, const int bslot) {
        const int c = CS * (wave + NW * ci) + cs;
        const bool have = CS == 1 || c < C64;
        uint32_t pk[3];
        uint32_t xb4[4] = {0u, 0u, 0u, 0u};
        if constexpr (GA) {
            // block scale of this 64-chunk: amax over the lane's 16 values, then over the row's 4 lanes
            float ac = 0.f;
            if constexpr (BF16) {
                us2 m2 = {0, 0};
#pragma unroll
                for (int d = 0; d < 8; ++d)
                    m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(us2, ch.w[d] & 0x7FFF7FFFu));
                const uint32_t mm = m2[0] > m2[1] ? m2[0] : m2[1];
                ac = __uint_as_float(mm << 16);
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) ac = fmaxf(ac, fabsf(ch.get(i)));
            }
            ac = max_xor16(ac);
            ac = max_xor32(ac);
            const uint32_t bits = sint4_scale(ac, &inv4);
            if (kq == 0 && have) {
                p.sxg[sxg_index(row, c, p.tiles128)] = bits;
                // row blocks of the last 128-row tile that do not exist: finite scales (the forward multiplies
                // them by zero)
                if (row + 32 >= p.Mp)
                    for (int rr = row + 32; (rr >> 7) == (row >> 7); rr += 32) p.sxg[sxg_index(rr, c, p.tiles128)] = 0u;
            }
        }
        {
            // Main codes: x * inv rounded to the nearest integer by the FP6 converter (f6_codes16).  Branch codes:
            // low bytes of x*invb + 1.5*2^23, gathered with byte permutes.
            float um[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                um[i] = __fmul_rn(ch.get(i), inv4);
                if constexpr (GA) um[i] = __builtin_amdgcn_fmed3f(um[i], -7.0f, 7.0f);  // the stored scale may be smaller than amax / 7
            }
            f6_codes16(um, pk);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t tb[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) tb[e] = rne_bits(__fmul_rn(ch.get(8 * h + e), invb));
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint32_t p01 = __builtin_amdgcn_perm(tb[4 * q + 1], tb[4 * q], 0x0c0c0400u);
                const uint32_t p23 = __builtin_amdgcn_perm(tb[4 * q + 3], tb[4 * q + 2], 0x0c0c0400u);
                xb4[2 * h + q] = __builtin_amdgcn_perm(p23, p01, 0x05040100u);
            }
        }
        // the lane's 16 codes are dwords 3*(kq&1) .. +2 of the forward lane (row % 32, K half kq/2): an aligned
        // 8-byte and a 4-byte store
        if (have) {
            uint8_t* chunk = p.xq + ((size_t)rb * C64 + c) * F6_CHUNK;
            const int fl = (row & 31) + 32 * (kq >> 1);
            const bool odd = kq & 1;
            uint8_t* d8 = chunk + (odd ? 1024 + fl * 8 : fl * 16);
            uint8_t* d4 = chunk + fl * 16 + (odd ? 12 : 8);
            *(uint2*)d8 = odd ? make_uint2(pk[1], pk[2]) : make_uint2(pk[0], pk[1]);
            *(uint32_t*)d4 = odd ? pk[0] : pk[2];
        }
        if (p.dbg_xb && row_ok && have)
            *(v4i*)(p.dbg_xb + (size_t)row * p.K + c * 64 + kq * 16) = v4i{(int)xb4[0], (int)xb4[1], (int)xb4[2], (int)xb4[3]};
        if (njb > 0) {
            const v4i av = {(int)xb4[0], (int)xb4[1], (int)xb4[2], (int)xb4[3]};
            if constexpr (CS == 1) {
#pragma unroll
                for (int jb = 0; jb < NJB; ++jb)
                    acc[jb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av, bv[bslot][jb], acc[jb], 0, 0, 0);
            } else {
                // a product per chunk, with zeros in the other chunks' rows
#pragma unroll
                for (int k = 0; k < CS; ++k) {
                    const int t = CS * ci + k, m = cs == k ? ~0 : 0;
                    if (t + RD - 1 < CS * NS) load_rq(bv[(t + RD - 1) % RD], t + RD - 1);
                    const v4i am = {av[0] & m, av[1] & m, av[2] & m, av[3] & m};
#pragma unroll
                    for (int jb = 0; jb < NJB; ++jb)
                        acc[jb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(am, bv[t % RD][jb], acc[jb], 0, 0, 0);
                }
            }
        }
    };
    if constexpr (STREAM) {
        for (int ci0 = 0; ci0 < nmy; ci0 += 2) {
#pragma unroll
            for (int sl = 0; sl < 2; ++sl) {
                const int ci = ci0 + sl, c = wave + NW * ci;
                load_rq(bv[(sl + 1) & 1], ci + 1);
                if (c < C64) code_chunk(xc[sl], ci, sl);  // wave-uniform
                load_x(xc[sl], ci + 2);
            }
        }
    } else {
#pragma unroll
        for (int ci = 0; ci < NS; ++ci) {
            if (CS == 1 && ci + RD - 1 < NS) load_rq(bv[(ci + RD - 1) % RD], ci + RD - 1);
            if (CS * (wave + NW * ci) < C64) code_chunk(xc[ci], ci, ci % RD);  // wave-uniform
        }
    }
    if (njb == 0) return;

    // ---- combine the wavefronts' partial accumulators, dequantise, re-quantise.  Up to two column blocks: the first wavefront;
    // more: wavefront w takes the column blocks w, w + NW, and the row maxima meet in LDS
#pragma unroll
    for (int jb = 0; jb < NJB; ++jb) *(v4i*)&s_acc[wave][jb][lane][0] = acc[jb];
    __syncthreads();
    if (wave >= PW) return;

    // lane holds column j = jb*16 + lane%16 and token rows 4*(lane/16) + i; with several chunks to a turn, after their sum, rows 4 * (kq & TG - 1) + i,
    // the same in 64 / (16 TG) lanes
    constexpr int TG = 4 / CS;
    const int tok0 = 4 * (kq & (TG - 1));
    float T[NT][4];
    float tmax[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int jb = wave + PW * t;
        if (jb >= NJB) break;  // wave-uniform
        v4i s = *(const v4i*)&s_acc[0][jb][lane][0];
#pragma unroll
        for (int w = 1; w < NW; ++w) s += *(const v4i*)&s_acc[w][jb][lane][0];
        if constexpr (CS > 1) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (CS > 2) s[i] += __shfl_xor(s[i], 16);
                s[i] += __shfl_xor(s[i], 32);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int tok = tok0 + i;
            const float tv = __fmul_rn(__fmul_rn((float)s[i], s_sxb[tok]), srj[t]);
            T[t][i] = tv;
            tmax[i] = fmaxf(tmax[i], fabsf(tv));
            const int grow = blockIdx.x * RW + tok;
            if (grow < p.M) {
                if (p.dbg_accT) p.dbg_accT[(size_t)grow * p.r + jb * 16 + r16] = s[i];
                if (p.dbg_T) p.dbg_T[(size_t)grow * p.r + jb * 16 + r16] = tv;
            }
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
    scales(r16 & 2 ? (r16 & 1 ? tmax[3] : tmax[2]) : (r16 & 1 ? tmax[1] : tmax[0]), p.qa, &sv, &iv);
    const float st4[4] = {row16_lane<0>(sv), row16_lane<1>(sv), row16_lane<2>(sv), row16_lane<3>(sv)};
    const float inv4t[4] = {row16_lane<0>(iv), row16_lane<1>(iv), row16_lane<2>(iv), row16_lane<3>(iv)};
    if (kq >= TG) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int grow = blockIdx.x * RW + tok0 + i;
        const float stv = st4[i], invt = inv4t[i];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int jb = wave + PW * t;
            if (jb >= NJB) break;
            p.tq[(size_t)grow * p.rp + jb * 16 + r16] = (int8_t)(rne_bits(__fmul_rn(T[t][i], invt)) & 0xFFu);
        }
        if (wave == 0) {
            if (r16 == 0) p.st[grow] = stv;
            if (p.rp > p.r && r16 < (p.rp - p.r)) p.tq[(size_t)grow * p.rp + p.r + r16] = 0;
        }
    }
}

template <bool BF16, int MAXC, int NJB, bool SM, bool GA, int NW, int CS>
static hipError_t launch_one(const ActParams& p, int64_t Mp, hipStream_t s)
{
    hipLaunchKernelGGL((act_int_kernel<BF16, MAXC, NJB, SM, GA, NW, CS>), dim3((unsigned)(Mp / 16 * CS)), dim3(NW * 64), 0, s, p);
    return hipGetLastError();
}

template <bool BF16, int MAXC, bool SM, bool GA, int NW, int CS>
static hipError_t launch_rank2(const ActParams& p, int64_t Mp, hipStream_t s)
{
    switch (p.r) {
        case 0: return launch_one<BF16, MAXC, 0, SM, GA, NW, CS>(p, Mp, s);
        case 16: return launch_one<BF16, MAXC, 1, SM, GA, NW, CS>(p, Mp, s);
        case 32: return launch_one<BF16, MAXC, 2, SM, GA, NW, CS>(p, Mp, s);
        case 64: return launch_one<BF16, MAXC, 4, SM, GA, NW, CS>(p, Mp, s);
        case 96: return launch_one<BF16, MAXC, 6, SM, GA, NW, CS>(p, Mp, s);
        default: return launch_one<BF16, MAXC, 8, SM, GA, NW, CS>(p, Mp, s);
    }
}

template <bool BF16, int MAXC, bool SM, int NW, int CS = 1>
static hipError_t launch_rank(const ActParams& p, int64_t Mp, hipStream_t s)
{
    return p.sxg ? launch_rank2<BF16, MAXC, SM, true, NW, CS>(p, Mp, s) : launch_rank2<BF16, MAXC, SM, false, NW, CS>(p, Mp, s);
}

template <bool BF16, bool SM>
static hipError_t launch_len(const ActParams& p, int64_t Mp, hipStream_t s)
{
    // Four or eight rows to a workgroup while that leaves every workgroup a compute unit of its own: coding 16 rows, 136 instructions per chunk and
    // wavefront, was the time of a small batch (us, 16 rows / this: 2 x 1152 rank 16 3.8 / 3.4, 300 x 1152 rank 32 4.9 / 4.3, 64 x 4608 rank 32 10.4 /
    // 6.1, 71 x 4544 rank 128 13.2 / 9.8, SINT4 64 x 2240 rank 64 8.7 / 6.1, fp32 500 x 2240 rank 64 8.9 / 6.4; eight rows 2000 x 1152 rank 32 5.2 / 4.8,
    // 2000 x 4608 rank 32 11.7 / 9.0, 2048 x 3072 rank 96 10.8 / 8.7).  Not for rows of at most a chunk per wavefront (700 x 320 rank 32 3.8 / 4.0, 1500 x 320 rank
    // 128 5.2 / 5.6, 12 x 512 3.7 / 3.8), from rank 96 on two, where the few wavefronts with chunks wait for R (12 x 640 rank 128 5.1 / 5.5, 1500 x 768 5.9 / 6.0, 1500 x
    // 1024 6.3 / 6.3, but 300 x 1152 6.3 / 5.9).
    const bool few_rows = p.C64 > (p.r >= 96 ? 16 : 8);
    if (few_rows && Mp <= 4 * compute_units()) {
        if (p.C64 <= 32) return launch_rank<BF16, 1, SM, 8, 4>(p, Mp, s);
        if (p.C64 <= 96) return launch_rank<BF16, 3, SM, 8, 4>(p, Mp, s);
    }
    if (few_rows && Mp <= 8 * compute_units()) {
        if (p.C64 <= 48) return launch_rank<BF16, 3, SM, 8, 2>(p, Mp, s);
        if (p.C64 <= 80) return launch_rank<BF16, 5, SM, 8, 2>(p, Mp, s);
    }
    // Eight wavefronts to a workgroup while there is at most one workgroup per compute unit: the time is then one
    // workgroup's chain (64 x 4608: 12.8 -> 10.8 us, SINT4 64 x 2240: 11.1 -> 9.1, 4096 x 4608: 18.7 -> 16.6); with more
    // workgroups four are as fast or faster (8192 x 4608: 27.3 against 29.6, 16384 x 1152: 15.7 against 17.3).
    // Smoothed fp32 rows spill 80 to 95 registers in the nine-chunk form (two multiplicands per value until the row is formed), which
    // costs more than a second pass over a row of six chunks per wavefront (4096 x 2624 rank 128: streamed 23.7 us, in
    // registers 28.0; 2 x 2624 rank 16: 10.5, 13.6) and less than one over nine (1024 x 4608 rank 32: 27.3, 24.4).  The other types spill at
    // rank 128 alone, at most 29 registers, and are within 3 % of the streamed form or faster.
    // So they are where four would stream the row, but for smoothed fp32 rows (smoothed 8192 x 4608 rank 64 34.5 us, four 41.6, 12000 x 2560 rank 64 31.0,
    // 36.9, fp32 6001 x 4480 44.8, 54.0).  Sixteen are slower at every size (64 x 1536 rank 64 7.0 us, eight 5.9, 2 x 1152 4.1, 3.7, 12 x 4480 9.1, 9.2).
    if (Mp <= 16 * compute_units() || (p.C64 > 36 && p.C64 <= 72 && BF16 == SM)) {
        const int mc = (p.C64 + 7) / 8;
        if (mc <= 3) return launch_rank<BF16, 3, SM, 8>(p, Mp, s);
        if (mc <= 5) return launch_rank<BF16, 5, SM, 8>(p, Mp, s);
        if (mc <= 9 && (BF16 || !SM || mc > 6)) return launch_rank<BF16, 9, SM, 8>(p, Mp, s);
        return launch_rank<BF16, 0, SM, 8>(p, Mp, s);
    }
    // MAXC = 0: the streamed kernel, for rows that do not fit in registers (K > 4608; smoothed fp32 rows beyond K = 2304)
    const int mc = (p.C64 + 3) / 4;
    if (mc <= 5) return launch_rank<BF16, 5, SM, 4>(p, Mp, s);
    if (mc <= 9) return launch_rank<BF16, 9, SM, 4>(p, Mp, s);
    if constexpr (BF16 && !SM) {
        if (mc <= 18) return launch_rank<BF16, 18, SM, 4>(p, Mp, s);
    }
    return launch_rank<BF16, 0, SM, 4>(p, Mp, s);
}

hipError_t launch_quantize_act_int(const Dims& d, int x_dtype, const uint8_t* packed, const void* X,
                                   int64_t M, int64_t ldx, uint8_t* act, const lq_act_debug* dbg,
                                   hipStream_t s)
{
    const PackedLayout pl = packed_layout(d);
    const ActLayout al = act_layout(d, M);
    ActParams p;
    p.tag = make_tag(d, LQ_BLOB_ACT, M);
    p.tag_dst = (uint32_t*)act;
    p.X = X;
    p.ldx = ldx;
    p.M = (int)M;
    p.K = (int)d.K;
    p.C64 = d.C64;
    p.r = d.r;
    p.rp = d.rp;
    p.qa = (float)d.qmax_ba;
    p.rq = (const int8_t*)(packed + pl.off_rq);
    p.sr = (const float*)(packed + pl.off_sr);
    p.xq = act + al.off_xq;
    p.sx = (float*)(act + al.off_sx);
    p.sxg = d.ga ? (uint32_t*)(act + al.off_sx) : nullptr;
    p.tiles128 = (int)((al.Mp + 127) / 128);
    p.Mp = (int)al.Mp;
    p.tq = (int8_t*)(act + al.off_tq);
    p.st = (float*)(act + al.off_st);
    p.dbg_xb = dbg ? dbg->xb : nullptr;
    p.dbg_sxb = dbg ? dbg->sxb : nullptr;
    p.dbg_accT = dbg ? dbg->accT : nullptr;
    p.dbg_T = dbg ? dbg->T : nullptr;
    p.rg = (const float*)(packed + pl.off_rg);
    if (d.smooth) return x_dtype == LQ_BF16 ? launch_len<true, true>(p, al.Mp, s) : launch_len<false, true>(p, al.Mp, s);
    return x_dtype == LQ_BF16 ? launch_len<true, false>(p, al.Mp, s) : launch_len<false, false>(p, al.Mp, s);
}

}  // namespace lq
