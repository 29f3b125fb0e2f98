// Attention of group-wise parallel training (see include/ps_train.h; Section 4.1).
//
// Two kernels per call: the rotary table (cos, sin of position * base^(-2j/d) in double precision) with the
// rotation of k (to the storage type, rounded as the inference path caches keys), and the attention itself,
// which rotates its query rows (in float32) while it brings them in.
//
// The attention kernels walk (a) the real tokens of groups up to the queries' own and (b) the rows of the queries'
// own groups, whose [MASK] tokens they see: no key tile that the mask hides entirely is touched.  Online softmax over
// the key tiles; scores are MFMA tiles (the keys' rows are the row operand, the query rows the column operand).  bf16
// values: ga_attn_wide_kernel (and, for the smallest calls, ga_attn_bf16_kernel); float32 values: ga_attn_f32_kernel (and, for
// short calls, ga_attn_f32_short_kernel).
// Each describes its own scheme.
#include <algorithm>

#include "ps_device.h"
#include "ps_train.h"
#include "ps_draft_debug.h"

namespace {

constexpr int GA_THREADS = 256, GA_WAVES = GA_THREADS / 64;
constexpr float GA_LAZY = 8.f;
// A launch may have 2^32 - 1 work items in x at most: workgroups beyond GA_GRID_X go on in y (blockIdx.y is 0 but in huge calls)
constexpr unsigned GA_GRID_X = 1u << 22;
constexpr long long GA_MAX_WG = 0x7FFFFFFF;                // the kernels number their workgroups in 31 bits (the float32 ones in 32)

// Wide accesses to the caller's q, k, v and out, which are only promised to be aligned to 4 bytes: the types say so, and the
// compiler emits the same 16-byte instructions (global memory takes them at any multiple of 4).
typedef unsigned u32x4_q __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned u32x2_q __attribute__((ext_vector_type(2), aligned(4)));
typedef float f32x4_q __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ uint4 ld16_q(const void* p) { return __builtin_bit_cast(uint4, (u32x4)*reinterpret_cast<const u32x4_q*>(p)); }
__device__ __forceinline__ uint4 ldg_stream16_q(const void* p) {
    return __builtin_bit_cast(uint4, (u32x4)__builtin_nontemporal_load(reinterpret_cast<const u32x4_q*>(p)));
}
template <typename WT> __device__ __forceinline__ f32x4 load4_q(const void* p) {
    if constexpr (Traits<WT>::BF) {
        const u32x2 v = *reinterpret_cast<const u32x2_q*>(p);
        return f32x4{bf16_to_f32(v[0] & 0xFFFFu), bf16_to_f32(v[0] >> 16), bf16_to_f32(v[1] & 0xFFFFu), bf16_to_f32(v[1] >> 16)};
    } else {
        return *reinterpret_cast<const f32x4_q*>(p);
    }
}
__device__ __forceinline__ void stg_stream16_q(float* p, f32x4 v) { __builtin_nontemporal_store((f32x4_q)v, reinterpret_cast<f32x4_q*>(p)); }

// Division of numbers below 2^31 by one that the host knows: n / d = (n * mul) >> shift
struct GaDiv {
    unsigned mul, shift;
    __device__ __forceinline__ unsigned operator()(unsigned n) const { return (unsigned)((u64)n * mul >> shift); }
};
GaDiv ga_div(unsigned d) {
    unsigned s = 0;
    while ((1ull << s) < d) ++s;
    return GaDiv{(unsigned)(((1ull << (31 + s)) + d - 1) / d), 31 + s};   // (mul * d exceeds 2^(31 + s) by less than d <= 2^s)
}
struct GaParams {
    int seqs, T, k, nq, nkv, rows, gpt, ntiles;   // gpt: groups per query tile
    unsigned k1_magic;    // ceil(2^32 / (k + 1)): a row's group is the upper half of the product (rows < 2^28; k > 0)
    float inv_sqrt_d;
    GaDiv by_heads, by_slots, by_nkv;   // nq * seqs, nkv * seqs, nkv
    int group;            // query heads per kv head
    const void *q, *k_, *v;
    float* out;
    float2* table;      // [T + k][d / 2]
    void* k_rot;        // rotated keys, storage type: [seqs][rows][nkv][d], or real tokens only as [seqs][nkv][T][d]
    double log2_base;
};

// 2^x: Taylor's series of e^(f ln 2), |f| <= 1/2, to the 13th power (the next is 4e-18)
__device__ __forceinline__ double ga_exp2(double x) {
    const double n = rint(x), y = (x - n) * 0.69314718055994530942;
    double p = 1.0 / 6227020800.0;
    constexpr double c[13] = {1.0, 1.0, 1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720, 1.0 / 5040, 1.0 / 40320, 1.0 / 362880,
                              1.0 / 3628800, 1.0 / 39916800, 1.0 / 479001600};
#pragma unroll
    for (int i = 12; i >= 0; --i) p = fma(p, y, c[i]);
    return ldexp(p, (int)n);
}
// cosine and sine of a >= 0: the multiple of pi / 2 taken off in two parts (Cody and Waite's reduction; the first product is exact inside its fma, the second
// part is below 1e-9), Taylor's series on [-pi / 4, pi / 4] to r^16 and r^17 (what follows is below 2e-18).  Angles beyond
// 2^22 (a base below 1) are the library's business
__device__ __forceinline__ float2 ga_cos_sin(double a) {
    if (!(a <= 4194304.0)) return make_float2((float)cos(a), (float)sin(a));
    const double n = rint(a * 0.63661977236758134308);
    const double r = fma(-n, 6.123233995736766036e-17, fma(-n, 1.5707963267948965580, a)), z = r * r;
    constexpr double cc[9] = {1.0, -1.0 / 2, 1.0 / 24, -1.0 / 720, 1.0 / 40320, -1.0 / 3628800, 1.0 / 479001600, -1.0 / 87178291200.0, 1.0 / 20922789888000.0};
    constexpr double sc[9] = {1.0, -1.0 / 6, 1.0 / 120, -1.0 / 5040, 1.0 / 362880, -1.0 / 39916800, 1.0 / 6227020800.0, -1.0 / 1307674368000.0, 1.0 / 355687428096000.0};
    double c = cc[8], s = sc[8];
#pragma unroll
    for (int i = 7; i >= 0; --i) {
        c = fma(c, z, cc[i]);
        s = fma(s, z, sc[i]);
    }
    const float fc = (float)c, fs = (float)(s * r);
    const int q = (int)n;                                   // quarter turns
    const float x = q & 1 ? fs : fc, y = q & 1 ? fc : fs;
    return make_float2((q + 1) & 2 ? -x : x, q & 2 ? -y : y);
}

// Rotary table and keys in one launch.  A workgroup takes one position, works out its cosines and sines (double precision,
// once for all heads, sequences and slots) and rotates the key rows that stand there, rounded as the inference path caches
// keys; gridDim.y workgroups share a position's rows.  ALL: the rows of every slot, to k_rot in the layout of k (a row (group,
// slot) stands at group + slot).  Otherwise the real tokens' rows only, to k_rot as [seq][kv head][token][D]: a [MASK] key is
// seen by its own group only, and ga_attn_wide_kernel rotates those while it stages them.  (A table kernel and a kernel over
// all rows that reads the table back: about 30 us at T 2048, k 4, 32 heads x 128; the real tokens only, as here: 9.8 us.)
// What bounds it where positions are few is the chain of one workgroup: its first key rows are requested before the table is
// worked out, and the table takes some 45 double operations per pair, where the library's exp, cos and sin took most of the
// kernel's time (whole calls, us: 2 x T 300, k 3, 8 heads x 64, float32 22.9 -> 22.4, 3 x T 120, k 2 16.9 -> 16.5, 2 x T 200, k 5,
// 16 / 4 heads x 64, bf16 15.5 -> 15.3).  As exact: of 4.75 million entries (bases 2 .. 10^6, positions up to 2^20) 1068 are not
// the nearest floats, 1268 with the library's; none is further off than that by more than 1e-10, with either.
template <typename WT, int D, bool ALL>
__global__ void __launch_bounds__(256) ga_rope_kernel(const GaParams P) {
    constexpr int ESZ = Traits<WT>::ESZ, Q4 = D / 8;       // groups of 4 pairs per head
    __shared__ float2 cs[D / 2];
    const int pos = blockIdx.x, tid = threadIdx.x;
    const int s0 = max(0, pos - P.T + 1), slots = ALL ? min(pos, P.k) - s0 + 1 : pos < P.T;   // slots s0 .. at this position
    const long long n = (long long)slots * P.seqs * P.nkv * Q4;
    const int g4 = tid % Q4;                                // (256 and the grid's stride are multiples of Q4)
    size_t to = 0;
    f32x4 a, b;
    auto request = [&](long long x) __attribute__((always_inline)) {
        const unsigned y = (unsigned)(x / Q4), z = y / P.nkv, head = y - z * P.nkv;   // y = (slot * seqs + seq) * nkv + head
        const unsigned slot = z / P.seqs, seq = z - slot * P.seqs;
        const int sl = ALL ? s0 + (int)slot : 0;
        const size_t row = (size_t)seq * P.rows + (size_t)(pos - sl) * (P.k + 1) + sl;
        const size_t from = ((row * P.nkv + head) * D + 4 * g4) * ESZ;
        to = ALL ? from : ((((size_t)seq * P.nkv + head) * P.T + pos) * D + 4 * g4) * ESZ;
        a = load4_q<WT>((const char*)P.k_ + from);
        b = load4_q<WT>((const char*)P.k_ + from + D / 2 * ESZ);
    };
    long long x = (long long)blockIdx.y * 256 + tid;
    if (x < n) request(x);                                  // (on its way while the table is worked out)
    if (tid < D / 2) {
        const float2 t = ga_cos_sin((double)pos * ga_exp2(-2.0 * tid / D * P.log2_base));
        cs[tid] = t;
        if (blockIdx.y == 0) P.table[(size_t)pos * (D / 2) + tid] = t;
    }
    __syncthreads();
    while (x < n) {
        f32x4 ra, rb;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float2 t = cs[4 * g4 + e];
            ra[e] = a[e] * t.x - b[e] * t.y;
            rb[e] = b[e] * t.x + a[e] * t.y;
        }
        store4<WT>((char*)P.k_rot + to, ra);
        store4<WT>((char*)P.k_rot + to + D / 2 * ESZ, rb);
        x += (long long)gridDim.y * 256;
        if (x < n) request(x);
    }
}

// the largest of z, |a|, |b|, or NaN if there is one
__device__ __forceinline__ float abs_max3(float z, float a, float b) {
    return __builtin_elementwise_maximum(__builtin_elementwise_maximum(z, __builtin_fabsf(a)), __builtin_fabsf(b));
}

// One output row by itself, from the keys and values that it sees and no others.  The kernels below multiply whole tiles: a
// key that the mask hides has probability 0, and 0 times a value row that holds Inf or NaN would reach rows that may not see
// it.  Nothing finite comes of a non-finite sum, so a row whose sum of exponentials is a number but whose output is not
// finite is looked at here by its wavefront: if a column that is not finite has no visible value to blame, the row is worked
// out again.  No call with finite values gets here: what it costs them is the look at the output registers.
template <typename WT, int D>
__device__ __forceinline__ void ga_row_alone(const GaParams& P, int seq, int h, int row, int lane) {
    constexpr int ESZ = Traits<WT>::ESZ, CPL = D / 64;
    const int K1 = P.k + 1, g = row / K1, n = g + 1 + (row - g * K1), hk = h / (P.nq / P.nkv);   // n visible keys, key i at position i
    const size_t rs = (size_t)P.nkv * D * ESZ, head = ((size_t)seq * P.rows * P.nkv + hk) * D * ESZ;
    const char* q = (const char*)P.q + (((size_t)seq * P.rows + row) * P.nq + h) * D * ESZ;
    const float2* tq = P.table + (size_t)(row - g * P.k) * (D / 2);
    auto key_off = [&](int i) __attribute__((always_inline)) { return (size_t)(unsigned)(i <= g ? i * K1 : g * K1 + i - g) * rs + head; };
    auto value = [&](int i, int e) __attribute__((always_inline)) {   // column lane + 64 e of key i's value
        const char* vp = (const char*)P.v + key_off(i) + (size_t)(lane + 64 * e) * ESZ;
        if constexpr (Traits<WT>::BF) return bf16_to_f32(*(const uint16_t*)vp);
        else return *(const float*)vp;
    };
    float* out = P.out + (((size_t)seq * P.rows + row) * P.nq + h) * D + lane;
    bool open = false, bad[CPL];                            // columns of this lane that no visible value explains so far
#pragma unroll
    for (int e = 0; e < CPL; ++e) {
        bad[e] = !(fabsf(__hip_atomic_load(out + 64 * e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < INFINITY);
        open |= bad[e];
    }
    for (int i0 = 0; i0 < n && __any(open); i0 += 8) {
        open = false;
#pragma unroll
        for (int e = 0; e < CPL; ++e) {
            float z = 0.f;
#pragma unroll
            for (int x = 0; x < 8; x += 2) z = abs_max3(z, value(min(i0 + x, n - 1), e), value(min(i0 + x + 1, n - 1), e));
            bad[e] = bad[e] && z < INFINITY;
            open |= bad[e];
        }
    }
    if (!__any(open)) return;
    float m = -INFINITY, l = 0.f, o[CPL];
#pragma unroll
    for (int e = 0; e < CPL; ++e) o[e] = 0.f;
    for (int i0 = 0; i0 < n; i0 += 64) {
        const int i = min(i0 + lane, n - 1);
        const char* kp = (const char*)P.k_ + key_off(i);
        const float2* tk = P.table + (size_t)i * (D / 2);
        float sc = 0.f;
#pragma unroll 1
        for (int j = 0; j < D / 2; j += 4) {
            const f32x4 qa = load4_q<WT>(q + j * ESZ), qb = load4_q<WT>(q + (D / 2 + j) * ESZ);
            const f32x4 ka = load4_q<WT>(kp + j * ESZ), kb = load4_q<WT>(kp + (D / 2 + j) * ESZ);
            f32x4 ra, rb;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ra[e] = ka[e] * tk[j + e].x - kb[e] * tk[j + e].y;
                rb[e] = kb[e] * tk[j + e].x + ka[e] * tk[j + e].y;
            }
            ra = store4<WT>(nullptr, ra, false);            // (rounded as cached keys are)
            rb = store4<WT>(nullptr, rb, false);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float c = tq[j + e].x, s = tq[j + e].y;
                sc += (qa[e] * c - qb[e] * s) * ra[e] + (qb[e] * c + qa[e] * s) * rb[e];
            }
        }
        sc = i0 + lane < n ? sc * (P.inv_sqrt_d * 1.4426950408889634f) : -INFINITY;
        const float m_new = fmaxf(m, wave_max(sc)), ref = m_new > -INFINITY ? m_new : 0.f;
        const float alpha = __builtin_amdgcn_exp2f(m - ref), p = __builtin_amdgcn_exp2f(sc - ref);
        l = l * alpha + wave_sum(p);
        m = m_new;
#pragma unroll
        for (int e = 0; e < CPL; ++e) o[e] *= alpha;
        for (int x = 0; x < min(64, n - i0); ++x) {
            const float px = __shfl(p, x, 64);
#pragma unroll
            for (int e = 0; e < CPL; ++e) o[e] += px * value(i0 + x, e);
        }
    }
#pragma unroll
    for (int e = 0; e < CPL; ++e) out[64 * e] = o[e] / l;
}
// Rows r0 + (the bits of rows), which the wavefront has just stored as they came out.  A call, not inlined, that reads the
// kernel's arguments again: what it needs would otherwise be kept in registers from the start (wide kernel at head_dim 128:
// 16 spilled instead of none, whole calls 2 .. 14 % slower).  With finite scores and every value NaN a call takes two to four times
// as long.
typedef const __attribute__((address_space(4))) GaParams* ga_args_t;
__device__ __forceinline__ ga_args_t ga_args() { return (ga_args_t)__builtin_amdgcn_kernarg_segment_ptr(); }
template <typename WT, int D>
__device__ __attribute__((noinline)) void ga_rows_alone(ga_args_t args, int seq, int h, int r0, unsigned rows, int lane) {
    const u64 a = (u64)args;
    const ga_args_t ua = (ga_args_t)((u64)(unsigned)__builtin_amdgcn_readfirstlane((unsigned)(a >> 32)) << 32 | (unsigned)__builtin_amdgcn_readfirstlane((unsigned)a));
    GaParams P;
    __builtin_memcpy(&P, (const void*)ua, sizeof(P));
    seq = __builtin_amdgcn_readfirstlane(seq);
    h = __builtin_amdgcn_readfirstlane(h);
    r0 = __builtin_amdgcn_readfirstlane(r0);
    rows = __builtin_amdgcn_readfirstlane(rows);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");      // (those stores have arrived before other lanes write the same rows)
    for (; rows; rows &= rows - 1) ga_row_alone<WT, D>(P, seq, h, r0 + __builtin_ctz(rows), lane);
}

// ------------------------------------------------------------------------------------------
// float32 values.  A workgroup takes 16 QT consecutive layout rows, 16 per wavefront, with KH wavefronts to every 16 rows
// that share their keys; it walks the real tokens' keys 16 KH at a time, then the rows R0 - 16 .. R0 + 16 QT - 1, among which the
// queries see their own groups' [MASK] rows, and of every stage's keys a wavefront takes 16.
//
// All products are v_mfma_f32_16x16x4_f32 with the queries along the lanes (lane = query c + 16 kb): scores as S^T, a lane
// holding keys 4 kb .. 4 kb + 3 of its query, register i of which is the column operand of O^T = V^T P^T for the four keys
// 4 kb + i; the row operand, column 4 m + e of those keys' values (m = the lane's c, e = 0 .. 3), are the four elements of one 16-byte
// LDS read.  Maximum, sum and output stay with the four lanes of a query; the wavefronts of 16 rows meet in LDS at the
// end.  K and V rows are staged for all wavefronts, into two buffers that take turns.
//
// Large calls are bound by the float32 matrix rate (32 MFMAs of 32 cycles per 16 x 16 tile at head_dim 64): 4 x T 512, k 10, 16 / 4 heads
// x 64 takes 294 us, 185 at that rate.  A small one is bound by the chain of its longest rows' stages and by compute units that have
// nothing left to do: 2 x T 300, k 3, 8 heads x 64 had 304 workgroups of 64 rows, the longest with 13 stages of 1.4 us.  So
// - large calls, head_dim 64: 32 rows, two wavefronts each (QT, KH = 2, 2; with 4, 2 311 us), whose LDS four workgroups share a
//   compute unit; head_dim 128: 64 rows (T 1024, k 4, 32 heads: 442 us, with 2, 2 515: two workgroups of half the size in the same LDS);
// - small ones: 32 rows, four wavefronts each (2, 4): half the stages, where the places suffice.  us, 4, 2 / 2, 2 / 2, 4: 2 x T 300, k 3,
//   8 heads x 64 27.9 / 26.2 / 23.1; T 100, k 3 (two) 14.8 / 11.7 / 11.2; T 300, k 3, 8 heads x 128 36.7 / 31.2 / 25.5; from 704 workgroups of 32
//   rows on (8 heads x 64: T 700, k 3 48.0 / 40.6 / 37.5, T 512, k 5 41.6 / 34.3 / 35.3), x 128 from 400 on (2 x T 300 46.2 / 42.0 / 46.8), not.
// Before 16x16x4 tiles, P.V was FMA work against probabilities broadcast from LDS: 724 and 40.5 us for the first two.
// ------------------------------------------------------------------------------------------
constexpr int GF_ROWS = 64;

template <int D, int QT, int KH>
__device__ __forceinline__ void ga_attn_f32(const GaParams& P) {
    constexpr int THREADS = 64 * QT * KH, ROWS = 16 * QT, KEYS = 16 * KH, TPR = THREADS / KEYS;   // keys of a stage, threads that stage a row
    constexpr int STEPS = D / 16, NV = D / 64, NS = D / 4 / TPR;   // 64-byte steps of a row; its 16-byte pieces per lane of 16, per thread that stages it
    constexpr int KSTR = 4 * D + 16, VSTR = 4 * D, KBUF = KEYS * KSTR, BUF = KBUF + KEYS * VSTR;
    constexpr int QAREA = 16 * D * 4;                       // 16 query rows as MFMA operands; later one wavefront's output on its way to the other
    constexpr int OFF_ML = QT * (KH - 1) * QAREA;           // [KH - 1][QT][64 lanes] (maximum, sum)
    static_assert(QT * QAREA <= 2 * BUF && OFF_ML + QT * (KH - 1) * 64 * 8 <= 2 * BUF, "query and merge areas fit the buffers");
    __shared__ __attribute__((aligned(16))) char smem[2 * BUF];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, kb = lane >> 4, qt = wave % QT, kh = wave / QT;   // query tile, half of the keys
    const int K1 = P.k + 1;
    auto group_of = [&](int row) __attribute__((always_inline)) { return P.k > 0 ? (int)__umulhi((unsigned)row, P.k1_magic) : row; };
    const unsigned wg = blockIdx.y * GA_GRID_X + blockIdx.x;
    const int blk = (P.rows + ROWS - 1) / ROWS - 1 - (int)(wg / (unsigned)P.nq);   // the rows with the most keys start first
    if (blk < 0) return;                                    // (beyond the last, in a launch of several rows of workgroups)
    const int h = wg % (unsigned)P.nq, seq = blockIdx.z, hk = h / (P.nq / P.nkv);
    const int R0 = ROWS * blk, r0 = R0 + 16 * qt;
    const bool active = r0 < P.rows;
    const int r_last = min(R0 + ROWS, P.rows) - 1, g_last_wg = group_of(r_last);
    const int n_real = g_last_wg / KEYS + 1, n_stages = n_real + (P.k > 0 ? (r_last - R0 + 16) / KEYS + 1 : 0);
    const int wg0 = group_of(min(r0, r_last)), wg1 = group_of(min(r0 + 15, r_last));   // the tile's first and last group
    const int qrow = min(r0 + c, r_last), qg = group_of(qrow);   // this lane's query (beyond the end: the last, repeated)

    // ---- staging
    const int skey = tid / TPR, sp = tid % TPR;
    const size_t rs = (size_t)P.nkv * D * 4, head_off = (((size_t)seq * P.rows) * P.nkv + hk) * D * 4 + sp * 16;
    const char* kbase = (const char*)P.k_rot + head_off;
    const char* vbase = (const char*)P.v + head_off;
    struct Stage { uint4 k[NS], v[NS]; };
    auto stage_load = [&](int t, Stage& x) __attribute__((always_inline)) {
        const int row = t < n_real ? min(KEYS * t + skey, g_last_wg) * K1 : min(max(R0 - 16 + KEYS * (t - n_real) + skey, 0), r_last);
        const size_t off = (size_t)(unsigned)row * rs;
#pragma unroll
        for (int i = 0; i < NS; ++i) { x.k[i] = ld16(kbase + off + 16 * TPR * i); x.v[i] = ld16_q(vbase + off + 16 * TPR * i); }
    };
    auto stage_store = [&](int t, const Stage& x) __attribute__((always_inline)) {
        char* b = smem + (t & 1) * BUF;
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            *reinterpret_cast<uint4*>(b + skey * KSTR + sp * 16 + 16 * TPR * i) = x.k[i];
            *reinterpret_cast<uint4*>(b + KBUF + skey * VSTR + sp * 16 + 16 * TPR * i) = x.v[i];
        }
    };
    Stage st, st1;
    stage_load(0, st);
    stage_load(min(1, n_stages - 1), st1);

    // ---- the query rows, rotated, into LDS as MFMA operands, and from there into both of their wavefronts' registers
    {
        const char* qsrc = (const char*)P.q + ((size_t)seq * P.rows * P.nq + h) * D * 4;
#pragma unroll
        for (int i = 0; i < (ROWS * (D / 8) + THREADS - 1) / THREADS; ++i) {
            const int x = tid + THREADS * i, r = x / (D / 8), g4 = x % (D / 8);
            if (ROWS * (D / 8) % THREADS != 0 && x >= ROWS * (D / 8)) break;
            const int row = min(R0 + r, r_last), pos = row - group_of(row) * P.k;                // group + slot
            const char* qr = qsrc + (size_t)row * P.nq * D * 4 + 16 * g4;
            const f32x4 a = load4_q<float>(qr), b = load4_q<float>(qr + 2 * D);
            const float4* tab = reinterpret_cast<const float4*>(P.table + (size_t)pos * (D / 2) + 4 * g4);
            const float4 t0 = tab[0], t1 = tab[1];
            const float cs[4] = {t0.x, t0.z, t1.x, t1.z}, sn[4] = {t0.y, t0.w, t1.y, t1.w};
            u32x4 ra, rb;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ra[e] = __float_as_uint(a[e] * cs[e] - b[e] * sn[e]);
                rb[e] = __float_as_uint(b[e] * cs[e] + a[e] * sn[e]);
            }
            const int ts = (r & 15) * (D / 4) + g4;                                             // (row, group of 4 elements) as attn_store_q counts
            attn_store_q<float, D>(smem + (r >> 4) * QAREA, ts, ra);
            attn_store_q<float, D>(smem + (r >> 4) * QAREA, ts + D / 8, rb);
        }
    }
    __syncthreads();
    BRegs<float, 1> bq[STEPS];
#pragma unroll
    for (int t = 0; t < STEPS; ++t) bq[t].h[0] = ld16(smem + qt * QAREA + (t * 64 + lane) * 16);
    __syncthreads();

    const float scale = P.inv_sqrt_d * 1.4426950408889634f;   // scores in units of ln 2
    float m_run = -INFINITY, l_run = 0.f;                   // of this lane's query: the reference (the same in its four lanes), the lane's own sum
    f32x4 o[D / 16];                                        // O^T: o[4 v + e][i] is column 64 v + 16 kb + 4 i + e of this lane's query
#pragma unroll
    for (int j = 0; j < D / 16; ++j) o[j] = f32x4{0.f, 0.f, 0.f, 0.f};

    stage_store(0, st);
    st = st1;
    __syncthreads();
    for (int t = 0; t < n_stages; ++t) {
        if (t + 1 < n_stages) stage_store(t + 1, st);
        if (t + 2 < n_stages) stage_load(t + 2, st);
        // this wavefront's 16 keys: first token / layout row; of the own rows the 16 of the tile itself and, where its first
        // row is not the first of its group, the 16 before
        const bool real = t < n_real;
        const int unit = KH * (real ? t : t - n_real) + kh, first = 16 * unit + (real ? 0 : R0 - 16);
        const bool busy = active & (real ? first <= wg1 : (unit == qt + 1) | ((unit == qt) & (wg0 * K1 != r0)));
        if (busy) {
            const char* kt = smem + (t & 1) * BUF + 16 * kh * KSTR + c * KSTR + kb * 16;
            const char* vt = smem + (t & 1) * BUF + KBUF + (16 * kh + 4 * kb) * VSTR + c * 16;
            f32x4 acc[2][1] = {{f32x4{0.f, 0.f, 0.f, 0.f}}, {f32x4{0.f, 0.f, 0.f, 0.f}}};   // (two shorter sums: less rounding, no MFMA waits for the one before)
#pragma unroll
            for (int s = 0; s < STEPS; s += 2) {
                mma_step<float, 1>(ld16(kt + 64 * s), bq[s], acc[0]);
                mma_step<float, 1>(ld16(kt + 64 * s + 64), bq[s + 1], acc[1]);
            }
            f32x4 sc = (acc[0][0] + acc[1][0]) * scale;
            if (!real | (first + 15 > wg0)) {
                const int lo = real ? 0 : qg * K1 + 1 - first - 4 * kb, hi = (real ? qg : qrow) - first - 4 * kb;
#pragma unroll
                for (int e = 0; e < 4; ++e) sc[e] = (e >= lo && e <= hi) ? sc[e] : -INFINITY;
            }
            const float mt = quad_rows_max(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])));
            const bool moved = mt > m_run + GA_LAZY;        // (the reference follows the maximum in steps of at least GA_LAZY)
            if (__any(moved)) {
                const float m_new = moved ? mt : m_run;
                const float alpha = moved ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.f;
                l_run *= alpha;
                m_run = m_new;
#pragma unroll
                for (int j = 0; j < D / 16; ++j) o[j] *= alpha;
            }
            const float m_use = m_run > -INFINITY ? m_run : 0.f;   // (no visible key yet: every exponent is -inf)
            f32x4 pr;
#pragma unroll
            for (int e = 0; e < 4; ++e) pr[e] = __builtin_amdgcn_exp2f(sc[e] - m_use);
            l_run += (pr[0] + pr[1]) + (pr[2] + pr[3]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const f32x4 vv = *reinterpret_cast<const f32x4*>(vt + i * VSTR + 256 * v);
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[4 * v + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[e], pr[i], o[4 * v + e], 0, 0, 0);
                }
        }
        __syncthreads();
    }

    // ---- the wavefronts of a tile meet; the first writes the rows
    l_run = quad_rows_sum(l_run);
    if (kh > 0) {
        const int area = (kh - 1) * QT + qt;
        *reinterpret_cast<float2*>(smem + OFF_ML + (area * 64 + lane) * 8) = make_float2(m_run, l_run);
#pragma unroll
        for (int j = 0; j < D / 16; ++j) *reinterpret_cast<f32x4*>(smem + area * QAREA + (j * 64 + lane) * 16) = o[j];
    }
    __syncthreads();
    if (kh == 0 && active) {
        float2 ml[KH - 1];
        float M = m_run;                                    // (-inf only if no visible score is finite)
#pragma unroll
        for (int i = 0; i < KH - 1; ++i) {
            ml[i] = *reinterpret_cast<const float2*>(smem + OFF_ML + ((i * QT + qt) * 64 + lane) * 8);
            M = fmaxf(M, ml[i].x);
        }
        const float f0 = __builtin_amdgcn_exp2f(m_run - M);
        float den = l_run * f0;
#pragma unroll
        for (int j = 0; j < D / 16; ++j) o[j] *= f0;
#pragma unroll
        for (int i = 0; i < KH - 1; ++i) {
            const float f = __builtin_amdgcn_exp2f(ml[i].x - M);
            den += ml[i].y * f;
#pragma unroll
            for (int j = 0; j < D / 16; ++j) o[j] += *reinterpret_cast<const f32x4*>(smem + (i * QT + qt) * QAREA + (j * 64 + lane) * 16) * f;
        }
#pragma unroll
        for (int j = 0; j < D / 16; ++j) o[j] = o[j] / den;
        float z = 0.f;
#pragma unroll
        for (int j = 0; j < D / 16; ++j) z = abs_max3(abs_max3(z, o[j][0], o[j][1]), o[j][2], o[j][3]);
        const u64 b = __ballot(den == den && !(z < INFINITY) && r0 + c < P.rows);
        if (r0 + c < P.rows) {
            float* orow = P.out + (((size_t)seq * P.rows + r0 + c) * P.nq + h) * D + 16 * kb;
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int i = 0; i < 4; ++i) stg_stream16_q(orow + 64 * v + 4 * i, f32x4{o[4 * v][i], o[4 * v + 1][i], o[4 * v + 2][i], o[4 * v + 3][i]});
        }
        const unsigned alone = (unsigned)(b | b >> 16 | b >> 32 | b >> 48) & 0xFFFFu;
        if (alone) ga_rows_alone<float, D>(ga_args(), seq, h, r0, alone, lane);
    }
}

constexpr int GF_QT(int head_dim) { return head_dim == 64 ? 2 : 4; }
template <int D>
__global__ void __launch_bounds__(128 * GF_QT(D), 4) ga_attn_f32_kernel(const GaParams P) {   // four wavefronts per SIMD
    ga_attn_f32<D, GF_QT(D), 2>(P);
}
template <int D>
__global__ void __launch_bounds__(512, D == 64 ? 4 : 2) ga_attn_f32_short_kernel(const GaParams P) {
    ga_attn_f32<D, 2, 4>(P);
}

// ------------------------------------------------------------------------------------------
// bf16 values, 16-row tiles (the smallest calls).  A query tile is a whole number of parallel groups (as many as fit into
// 16 rows), so the [MASK] tokens of its groups all lie inside its own rows.  A workgroup takes four adjacent query tiles, one per wavefront, and walks the key tiles of real
// tokens two at a time; the pair's K and V rows are brought in once for all four wavefronts.
//
// Loads are laid out for the texture unit, which handles a load in units of four lanes: four adjacent lanes read
// adjacent bytes of one row (a lane that fetched its own MFMA operand directly would make every lane of such a unit
// touch another row).  K: wavefront w brings in half of tile w / 2's rows; lane (key = lane / 4, j = lane % 4) reads
// bytes [64 t + 16 j, +16) of its key and puts them into LDS at (t ^ key % 4, j ^ key / 4 % 4) of the key's row,
// where lane (c, kb) of every wavefront picks up bytes [64 t + 16 kb, +16) of key c, its operand of MFMA step t (the
// placement keeps writers and readers off each other's banks).  V: wavefront w brings in keys 4 w .. 4 w + 3 of both
// tiles; a lane reads 4 bytes (two columns) of each and stores, per column, the dwords (key 4 w, 4 w + 1) and
// (4 w + 2, 4 w + 3) of the first tile and of the second side by side: lane (c, kb) then reads, per 16 output columns,
// one 16-byte piece = its 8 keys of the 32-key contraction (index 8 kb + e = key 4 kb + e of the first tile,
// 4 kb + e - 4 of the second); 4 dwords are left out every 8 columns and 4 more per block of 4 keys (banks again).
// Two such buffers take turns: while a pair is worked on, the next one is written (from registers that were
// requested an iteration earlier) and the one after it is requested; one barrier per pair.
//
// The tile of a query tile's own [MASK] rows comes last: the four wavefronts' own tiles are staged like two more
// pairs, and a wavefront works on the one that holds its tile with the other tile masked.
//
// Per wavefront: the 16 query rows, rotated in float32, scaled by log2(e) / sqrt(d) (scores in units of ln 2: the
// exponentials are single v_exp_f32) and split into bf16 high and low parts, stay in registers as the 16-column
// operand; online softmax per pair of tiles (the maxima and sums of the four lanes that share a query row are
// exchanged with row swaps; the running output is rescaled only when a maximum moved); P, split into high and low
// parts, is the 16-row operand of P.V straight from the score registers.  A wavefront owns its rows: no merge.
// ------------------------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(GA_THREADS, 4) ga_attn_bf16_kernel(const GaParams P) {
    typedef bf16_t WT;
    constexpr int STEPS = D / 32, NCH = D / 8;
    constexpr int KT = 16 * D * 2;                          // bytes of a staged K tile
    constexpr int RSTR = (D / 8) * 36 + 4;                  // dwords per block of 4 keys of the staged V pair
    constexpr int BUF = 2 * KT + 4 * RSTR * 4;              // bytes of a buffer: two K tiles, the V pair
    constexpr int OFF_A = 2 * BUF;                          // [waves][16] rescale factors, later the rows' sums
    constexpr int QAREA = 16 * D * 4;                       // a wavefront's query rows on their way into registers, later its output
    static_assert(GA_WAVES * QAREA <= 2 * BUF, "the wavefronts' query and output areas fit the buffers");
    __shared__ __attribute__((aligned(16))) char smem[OFF_A + GA_WAVES * 16 * 4];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, kb = lane >> 4;
    const int K1 = P.k + 1;
    const int nblk = (P.ntiles + GA_WAVES - 1) / GA_WAVES;
    const int blk = nblk - 1 - (int)blockIdx.x;             // the tiles with the most keys start first
    const int h = blockIdx.y, seq = blockIdx.z, hk = h / (P.nq / P.nkv);
    // this wavefront's query tile (a wavefront beyond the last tile keeps the last one's numbers and only helps to stage)
    const int qt = GA_WAVES * blk + wave;
    const bool active = qt < P.ntiles;
    const int g0 = min(qt, P.ntiles - 1) * P.gpt, ng = min(P.gpt, P.T - g0), nrows = ng * K1, r0 = g0 * K1, g_last = g0 + ng - 1;
    // the workgroup's key tiles of real tokens, in pairs, then two pairs with the four own-[MASK] tiles
    const int g_last_wg = min((min(GA_WAVES * blk + GA_WAVES - 1, P.ntiles - 1) + 1) * P.gpt, P.T) - 1;
    const int real_pairs = ((g_last_wg >> 4) + 2) >> 1;
    const int n_pairs = real_pairs + (P.k > 0 ? 2 : 0);

    float* sA = reinterpret_cast<float*>(smem + OFF_A) + wave * 16;
    char* const sQ = smem + wave * QAREA;
    const unsigned rs32 = (unsigned)(P.nkv * D * 2);       // bytes between layout rows
    const unsigned K1rs = (unsigned)K1 * rs32;              // ... between real tokens
    const char* kbase = (const char*)P.k_rot + ((size_t)seq * P.rows * P.nkv + hk) * D * 2;
    const char* vbase = (const char*)P.v + ((size_t)seq * P.rows * P.nkv + hk) * D * 2;

    // ---- staging: this lane's share of a pair
    // K: tile kg of the pair, requests t = kt0 .. kt0 + STEPS / 2 - 1 of (key kkey, piece kj)
    constexpr int KL = STEPS / 2;                           // K requests per lane
    constexpr int TM = STEPS - 1, TL = STEPS == 4 ? 2 : 1;  // the row's 64-byte segments: mask and log2
    const int kg = wave >> 1, kt0 = (wave & 1) * KL, kkey = lane >> 2, kj = lane & 3;
    auto k_lds = [&](int key, int j) __attribute__((always_inline)) {
        return key * (2 * D) + ((key & TM) << 6) + ((j ^ ((key >> TL) & 3)) << 4);
    };
    const int kw_rel = kg * KT + k_lds(kkey, kj), kr_rel = k_lds(c, kb);
    // V: keys 4 wave .. 4 wave + 3 of both tiles, columns 2 vc, 2 vc + 1 (lanes beyond D / 2 columns repeat the last and store nothing)
    const int vc = min(lane, D / 2 - 1);
    const bool vlane = lane < D / 2;
    const int vw_rel = 2 * KT + (wave * RSTR + (vc >> 2) * 36 + (vc & 3) * 8) * 4;
    const int vr_rel = 2 * KT + (kb * RSTR + (c >> 3) * 36 + (c & 7) * 4) * 4;
    struct Stage { uint4 k[KL]; unsigned v[2][4]; };
    // layout row of key j of tile g of pair p: real tokens up to the workgroup's last group, then the own rows of query
    // tile 4 blk + 2 (p - real_pairs) + g (clamped to rows that exist)
    auto stage_load = [&](int p, Stage& s) __attribute__((always_inline)) {
        size_t voff[2][4];                                  // bytes from vbase to the V rows (wavefront-uniform)
        unsigned krow, kmul;                                // the lane's K row: index and bytes per index
        if (p < real_pairs) {
            krow = (unsigned)min(16 * (2 * p + kg) + kkey, g_last_wg);
            kmul = K1rs;
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i) voff[g][i] = (size_t)(unsigned)min(16 * (2 * p + g) + 4 * wave + i, g_last_wg) * K1rs;
        } else {
            const int o = p - real_pairs;
            int first[2], last[2];                          // the own rows of the pair's two query tiles
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const int go = min(GA_WAVES * blk + 2 * o + g, P.ntiles - 1) * P.gpt;
                first[g] = go * K1;
                last[g] = min(P.gpt, P.T - go) * K1 - 1;
            }
            krow = (unsigned)(first[kg] + min(kkey, last[kg]));
            kmul = rs32;
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i) voff[g][i] = (size_t)(unsigned)(first[g] + min(4 * wave + i, last[g])) * rs32;
        }
        const char* kp = kbase + (size_t)krow * kmul + kj * 16;
#pragma unroll
        for (int u = 0; u < KL; ++u) s.k[u] = ld16(kp + (kt0 + u) * 64);
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i)                      // (descriptor at the pair's first row, scalar offset per row: no vector address arithmetic)
                s.v[g][i] = __builtin_amdgcn_raw_buffer_load_b32(make_rsrc(vbase + voff[0][0]), (unsigned)(vc * 4), (unsigned)(voff[g][i] - voff[0][0]), 0);
    };
    auto stage_store = [&](char* buf, const Stage& s) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < KL; ++u) *reinterpret_cast<uint4*>(buf + (kw_rel ^ ((kt0 + u) << 6))) = s.k[u];
        if (vlane) {
            unsigned lo[4], hi[4];
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                lo[2 * g] = __builtin_amdgcn_perm(s.v[g][1], s.v[g][0], 0x05040100u); lo[2 * g + 1] = __builtin_amdgcn_perm(s.v[g][3], s.v[g][2], 0x05040100u);
                hi[2 * g] = __builtin_amdgcn_perm(s.v[g][1], s.v[g][0], 0x07060302u); hi[2 * g + 1] = __builtin_amdgcn_perm(s.v[g][3], s.v[g][2], 0x07060302u);
            }
            *reinterpret_cast<uint4*>(buf + vw_rel) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            *reinterpret_cast<uint4*>(buf + vw_rel + 16) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
        }
    };

    Stage st;
    stage_load(0, st);                                      // (on its way while the query rows are brought in)

    // ---- the query rows into registers, by way of LDS
    {
        const char* qsrc = (const char*)P.q + ((size_t)seq * P.rows * P.nq + h) * D * 2;
        const float qscale = P.inv_sqrt_d * 1.4426950408889634f;
        for (int t2 = lane; t2 < 16 * (D / 8); t2 += 64) {
            const int r = min(t2 / (D / 8), nrows - 1), g4 = t2 % (D / 8);
            const int row = r0 + r, pos = row / K1 + row % K1;                  // group + slot
            const char* qrow = qsrc + (size_t)row * P.nq * D * 2;
            const f32x4 a = load4_q<WT>(qrow + 4 * g4 * 2), b = load4_q<WT>(qrow + (D / 2 + 4 * g4) * 2);
            u32x4 ra, rb;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float2 t = P.table[(size_t)pos * (D / 2) + 4 * g4 + e];
                ra[e] = __float_as_uint((a[e] * t.x - b[e] * t.y) * qscale);
                rb[e] = __float_as_uint((b[e] * t.x + a[e] * t.y) * qscale);
            }
            const int ts = (t2 / (D / 8)) * (D / 4) + g4;                       // (row, group of 4 elements) as attn_store_q counts
            attn_store_q<WT, D>(sQ, ts, ra);
            attn_store_q<WT, D>(sQ, ts + D / 8, rb);
        }
    }
    lds_sync_wave();
    __builtin_amdgcn_wave_barrier();
    BRegs<WT, 1> bq[STEPS];
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
        bq[t].h[0] = ld16(sQ + (2 * t * 64 + lane) * 16);
        bq[t].l[0] = ld16(sQ + ((2 * t + 1) * 64 + lane) * 16);
    }
    __syncthreads();                                        // the buffers take K and V rows from here on

    // ---- this lane's query (column c of the score tile): group, slot, and which keys 4 kb + e of a tile it sees
    const int qr = min(c, nrows - 1), qg = g0 + qr / K1, qs = qr % K1;
    const bool qlive = active && c < nrows;
    const int real_hi0 = qlive ? qg - 4 * kb : -(1 << 20);   // real tokens of tile t: e <= real_hi0 - 16 t
    const int own_lo = qr - qs + 1 - 4 * kb, own_hi = qlive ? qr - 4 * kb : -(1 << 20);   // own [MASK] rows: those of the query's group, up to its slot
    float m_run = -INFINITY, l_run = 0.f;                   // of query c (the same in the four lanes that share it)
    f32x4 oacc[D / 16];                                     // MFMA tiles, lane (c, kb): column 16 j + c of rows 4 kb .. 4 kb + 3
#pragma unroll
    for (int j = 0; j < D / 16; ++j) oacc[j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // one pair of tiles: lo[g] <= e <= hi[g] are the keys 4 kb + e of tile g the lane's query sees (unmasked: all of them)
    auto work = [&](const char* buf, bool unmasked, int lo0, int hi0, int lo1, int hi1) __attribute__((always_inline)) {
        f32x4 acc[2][1];
#pragma unroll
        for (int g = 0; g < 2; ++g) acc[g][0] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < STEPS; ++t)
#pragma unroll
            for (int g = 0; g < 2; ++g) mma_step<WT, 1>(ld16(buf + g * KT + (kr_rel ^ (t << 6))), bq[t], acc[g]);
        float sc[2][4], mt = -INFINITY;
        if (unmasked) {
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sc[g][e] = acc[g][0][e];
                    mt = fmaxf(mt, sc[g][e]);
                }
        } else {
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const int lo = g ? lo1 : lo0, hi = g ? hi1 : hi0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sc[g][e] = (e >= lo && e <= hi) ? acc[g][0][e] : -INFINITY;
                    mt = fmaxf(mt, sc[g][e]);
                }
            }
        }
        mt = quad_rows_max(mt);
        // The reference m_run the exponentials are taken against follows the row's maximum only when that has moved
        // up by more than GA_LAZY (in units of ln 2): sums and outputs are relative to the same reference, so the
        // quotient is the same, the probabilities stay below 2^GA_LAZY, and most pairs need no rescaling
        const bool moved = mt > m_run + GA_LAZY;            // (also the first keys a row sees: m_run = -inf)
        const float m_new = moved ? mt : m_run;
        const float alpha = moved ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.f;   // exp2(-inf) = 0 when nothing was seen before
        const float m_use = m_new > -INFINITY ? m_new : 0.f;
        f32x4 pr[2];
        float ls = 0.f;
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                pr[g][e] = __builtin_amdgcn_exp2f(sc[g][e] - m_use);
                ls += pr[g][e];
            }
        ls = quad_rows_sum(ls);
        l_run = l_run * alpha + ls;
        m_run = m_new;
        if (__any(moved)) {                                 // rows 4 kb .. 4 kb + 3 of the running output: their factors by way of LDS
            if (kb == 0) sA[c] = alpha;
            lds_sync_wave();
            __builtin_amdgcn_wave_barrier();
            const f32x4 al = *reinterpret_cast<const f32x4*>(sA + 4 * kb);
#pragma unroll
            for (int j = 0; j < D / 16; ++j) oacc[j] *= al;
            lds_sync_wave();
            __builtin_amdgcn_wave_barrier();
        }
        unsigned ph2[2][2], pl2[2][2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            ph2[g][0] = pack_bf16x2(pr[g][0], pr[g][1]); ph2[g][1] = pack_bf16x2(pr[g][2], pr[g][3]);
            pl2[g][0] = pack_bf16x2(pr[g][0] - __uint_as_float(ph2[g][0] << 16), pr[g][1] - __uint_as_float(ph2[g][0] & 0xFFFF0000u));
            pl2[g][1] = pack_bf16x2(pr[g][2] - __uint_as_float(ph2[g][1] << 16), pr[g][3] - __uint_as_float(ph2[g][1] & 0xFFFF0000u));
        }
        const bf16x8 pa = __builtin_bit_cast(bf16x8, make_uint4(ph2[0][0], ph2[0][1], ph2[1][0], ph2[1][1]));
        const bf16x8 pb = __builtin_bit_cast(bf16x8, make_uint4(pl2[0][0], pl2[0][1], pl2[1][0], pl2[1][1]));
        // four blocks of 16 output columns at a time: the MFMAs with P's high parts, then those with its low parts
        // (an MFMA that follows the one it depends on directly would wait for it)
#pragma unroll
        for (int j0 = 0; j0 < D / 16; j0 += 4) {
            bf16x8 vv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) vv[u] = __builtin_bit_cast(bf16x8, ld16(buf + vr_rel + 72 * 4 * (j0 + u)));
#pragma unroll
            for (int u = 0; u < 4; ++u) oacc[j0 + u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa, vv[u], oacc[j0 + u], 0, 0, 0);
#pragma unroll
            for (int u = 0; u < 4; ++u) oacc[j0 + u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pb, vv[u], oacc[j0 + u], 0, 0, 0);
        }
    };

    // ---- the pairs
    stage_store(smem, st);
    if (n_pairs > 1) stage_load(1, st);
    __syncthreads();
    for (int p = 0; p < n_pairs; ++p) {
        const char* buf = smem + (p & 1) * BUF;
        if (p + 1 < n_pairs) stage_store(smem + ((p + 1) & 1) * BUF, st);
        if (p + 2 < n_pairs) stage_load(p + 2, st);
        // what this wavefront's queries see of the pair.  Real tokens: nothing if every key of the pair lies after the
        // tile's last group, everything if every key lies before its first.  The own-[MASK] pairs: the pair
        // p - real_pairs = wave / 2 holds this wavefront's tile, as its tile wave % 2; the other tile is masked
        const bool real = p < real_pairs, mine = (wave >> 1) == p - real_pairs, first = (wave & 1) == 0;
        const bool busy = active && (real ? 32 * p <= g_last : mine);
        const bool unmasked = real && 32 * p + 31 <= g0;
        const int lo = real ? 0 : own_lo;
        const int hi0 = real ? real_hi0 - 32 * p : (first ? own_hi : -(1 << 20));
        const int hi1 = real ? real_hi0 - 32 * p - 16 : (first ? -(1 << 20) : own_hi);
        if (busy) work(buf, unmasked, lo, hi0, lo, hi1);
        __syncthreads();
    }

    // ---- output: rows by way of the wavefront's LDS area (the buffers are free now), divided by their sums
    if (kb == 0) sA[c] = l_run;
    float* sO = reinterpret_cast<float*>(sQ);
#pragma unroll
    for (int j = 0; j < D / 16; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) sO[(4 * kb + r) * D + 16 * j + c] = oacc[j][r];
    unsigned alone = 0;                                     // rows whose output is not finite
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float z = 0.f;
#pragma unroll
        for (int j = 0; j < D / 16; j += 2) z = abs_max3(z, oacc[j][r], oacc[j + 1][r]);
        const u64 b = __ballot(!(z < INFINITY));
#pragma unroll
        for (int i = 0; i < 4; ++i) alone |= (b >> (16 * i) & 0xFFFFu) ? 1u << (4 * i + r) : 0u;
    }
    alone &= (unsigned)__ballot(l_run == l_run) & ((1u << nrows) - 1u);
    lds_sync_wave();
    __builtin_amdgcn_wave_barrier();
    if (active) {
        float* obase = P.out + ((size_t)seq * P.rows * P.nq + h) * D;
        for (int x = lane; x < nrows * D; x += 64) {
            const int rr = x / D, dd = x - rr * D;
            obase[(size_t)(r0 + rr) * P.nq * D + dd] = sO[x] / sA[rr];   // (every row sees at least its own real token: the sum is > 0)
        }
        if (alone) ga_rows_alone<WT, D>(ga_args(), seq, h, r0, alone, lane);
    }
}

// ------------------------------------------------------------------------------------------
// bf16 values, the wide kernel.  A workgroup takes 128 consecutive layout rows, 32 per wavefront, whatever groups they
// belong to (every row of every MFMA tile is a query: with 9 rows per group a tile of whole groups fills 9 of 16).  It
// works on the rows of its own groups, whose [MASK] tokens its queries see, then on the real tokens' keys, 32 at a time.
//
// All products are v_mfma_f32_32x32x16_bf16 with the queries along the lanes (lane = query c + 32 * half): the scores
// leave the matrix core as S^T, a lane holding 16 of 32 keys of its query, which is - the contraction may take the
// keys in any order as long as both operands do - the operand layout of O^T = V^T P^T.  So a query's maximum, sum
// and output belong to the lane pair (c, c + 32) from start to end: one exchange per 32 keys for the maximum, none for
// the sum (each half adds up its own keys; the halves meet at the end), and rescaling is one multiplication per register.
// Queries and probabilities are split into bf16 high and low parts (two MFMAs per product).
//
// K and V rows are staged once per workgroup, row by row, into two LDS buffers that take turns (registers requested a
// tile ahead); V is transposed by the LDS unit on the way out (ds_read_b64_tr_b16: 16 lanes get 4 keys of one column each).
// The scores of tile t + 1 are worked out beside the exponentials of tile t, and its maxima, the stages' stores and the next
// requests beside P.V of tile t, so every wavefront has matrix and vector work to offer at any time; the last tile works out no
// further scores, and tiles that every query sees entirely have a loop without masks.  (With maxima and stores in front of the
// tile's first MFMA, one loop for all tiles and scores one tile too far: 1.3 .. 3.5 % slower, T 60 15.3 -> 14.8, T 500 (two) 56.4
// -> 54.8, T 1300, k 0 50.0 -> 48.4 us.)  Two workgroups per compute unit (256 registers) are what the query and output registers allow.
// Everything that a workgroup reads for the first time (table, query rows, own rows, first tiles) is requested at once.  Its start
// took 17 .. 20 thousand clocks of a workgroup's 25 (T 60), 40 (T 203), 74 (T 700) thousand: so query rows pass through LDS once, as
// they are, and are rotated and split as operands (three passes before: high parts, low parts), the own rows' two tiles share their maximum
// and the second multiplies the 16 keys that count, and no index is divided for.  Whole calls, us: T 60, k 4, 32 heads 14.8 -> 13.7; T 203 24.6 ->
// 23.3; T 700, k 2, 40 heads 58.3 -> 57.2; 4 x T 1024, k 8 725 -> 702.  The output rows in one pass through LDS instead of two: 0 (head_dim 64: slower).  The query
// rows are read and the output rows are written once, past the caches (non-temporal): the L2 is left to the heads' keys and
// values (3.7 % of a T 2048, k 4 call, 4.5 % of 4 x T 1024, k 8, 9 % of T 203; the own rows read that way, too: 1 % slower, the next
// workgroup reads 16 of them again).
//
// A tile is 32 MFMAs of 32 cycles per wavefront and about as much vector work: at T 2048, k 4 the matrix cores are busy 53 % of the
// kernel's time and the vector ALU 47 %, at 1.9 GHz or less: large calls are bound by power (the same instructions on zeros: 259 us where random
// values take 360 on that card, 545 for 735 at 4 x T 1024, k 8).  A workgroup's start (its rows come from memory) and its own rows have few
// MFMAs to show.  At T 203 that is most of the time (matrix cores 11 %).  All 256 registers are in use and none is spilled: eight spilled ones cost 1 .. 4 %.
// Whole calls among others of their kind, against the 16-row kernel and its three launches: T 2048, k 4, 32 heads x 128: 503 -> 339 us
// (507 TFLOP/s of visible pairs, every product twice); 4 x T 1024, k 8, 32 / 8 heads: 1501 -> 700 us; T 203, k 5, 40 heads: 40.9 -> 23.3 us.
// Tried: no scores ahead (other wavefront alone fills the gaps): 5 % slower; own rows as further tiles of the loop, rotated
// between the barriers: 4 % (T 2048) and 12 % (4 x 1024, k 8) slower; raised wavefront priority in the matrix part, two
// accumulators for the scores, four K operands requested ahead: no change; the low parts by v_dot2c_f32_bf16 (no shift or mask per
// value) 0.6 .. 5.5 % slower; MFMAs and vector instructions in a given alternation (sched_group_barrier) 2 .. 12 % slower.
// ------------------------------------------------------------------------------------------
constexpr int GW_ROWS = 32 * GA_WAVES;                     // query rows of a workgroup
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

__device__ __forceinline__ bf16x8 split_hi(const float (&v)[8], unsigned (&hi)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) hi[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
    return __builtin_bit_cast(bf16x8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
}
__device__ __forceinline__ bf16x8 split_lo(const float (&v)[8], const unsigned (&hi)[4]) {
    unsigned lo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        lo[i] = pack_bf16x2(v[2 * i] - __uint_as_float(hi[i] << 16), v[2 * i + 1] - __uint_as_float(hi[i] & 0xFFFF0000u));
    return __builtin_bit_cast(bf16x8, make_uint4(lo[0], lo[1], lo[2], lo[3]));
}

template <int D>
__global__ void __launch_bounds__(GA_THREADS, 2) ga_attn_wide_kernel(const GaParams P) {   // two workgroups per compute unit
    constexpr int STEPS = D / 16;                           // MFMA steps of a score tile
    constexpr int NJ = D / 32;                              // blocks of 32 output columns
    constexpr int PAIRS = D / 16;                           // pairs (j, j + PAIRS) of 16-byte pieces of a row that are rotary partners
    // the stages: two tiles of 32 K rows, two of V rows (paddings: no two of the lanes that are served together meet in a bank)
    constexpr int NP = D / 64;                              // pieces of a row per thread, 8 threads per row
    constexpr int KSTR = 2 * D + 16, VSTR = 2 * D + 64, KBUF = 32 * KSTR, VBUF = 32 * VSTR, OFF_V = 2 * KBUF;
    // before them: the query rows on their way into registers (from 0), the rows' part of the rotary table
    constexpr int OFF_T = GA_WAVES * 32 * KSTR, TROW = D / 2 * 8 + 16, TROWS = 66;   // positions of GW_ROWS rows: at most (GW_ROWS - 2) / K1 + 1 + K1, K1 = 2 .. 16
    // ... then the own rows: layout rows R0 - 16 .. R0 + 127, K and V
    constexpr int OROWS = GW_ROWS + 16, OFF_OV = OROWS * 2 * D;
    constexpr int OCOLS = D == 128 ? 64 : 32;               // output columns that pass through LDS at a time
    constexpr int SMEM = 2 * OFF_OV > OFF_T + TROWS * TROW ? 2 * OFF_OV : OFF_T + TROWS * TROW;
    constexpr int TAREA = SMEM / GA_WAVES & ~15;            // k = 0: the wavefront's part of the table
    static_assert(32 * TROW <= TAREA && OFF_V + 2 * VBUF <= SMEM && GA_WAVES * 32 * OCOLS * 4 <= SMEM && 2 * SMEM <= 160 * 1024, "");
    __shared__ __attribute__((aligned(16))) char smem[SMEM];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, half = lane >> 5;
    const int K1 = P.k + 1;
    // Workgroups with the most keys start first; neighbours in the launch order, which go to different XCDs, take different
    // heads, so that (kv heads x sequences a multiple of 8) a kv head's rows are read through one L2
    const unsigned slots = (unsigned)P.nkv * P.seqs, heads = (unsigned)P.nq * P.seqs;
    const unsigned wg = blockIdx.y * GA_GRID_X + blockIdx.x;
    const unsigned wb = P.by_heads(wg), hs = wg - wb * heads, hb = P.by_slots(hs), sl = hs - hb * slots;
    const int blk = (P.rows + GW_ROWS - 1) / GW_ROWS - 1 - (int)wb;
    if (blk < 0) return;                                    // (beyond the last, in a launch of several rows of workgroups)
    const int seq = P.by_nkv(sl), hk = sl - seq * P.nkv, h = hk * P.group + hb;
    const int R0 = GW_ROWS * blk, r0 = R0 + 32 * wave;
    const bool active = r0 < P.rows;
    auto group_of = [&](int row) __attribute__((always_inline)) { return P.k > 0 ? (int)__umulhi((unsigned)row, P.k1_magic) : row; };
    const int r_last = min(R0 + GW_ROWS, P.rows) - 1;       // of the workgroup
    const int g_last_wg = group_of(r_last), gB0 = group_of(R0);   // its last and first group
    const int n_real = g_last_wg / 32 + 1;                  // tiles of 32 real tokens
    const int w_first = min(r0, r_last), wg0 = group_of(w_first), wg1 = group_of(min(r0 + 31, r_last));   // this wavefront's first and last group
    const int qrow = min(r0 + c, r_last), qg = group_of(qrow);   // this lane's query row (beyond the end: the last, repeated) and group
    const size_t rs = (size_t)P.nkv * D * 2;                // bytes between layout rows
    const char* kraw = (const char*)P.k_ + ((size_t)seq * P.rows * P.nkv + hk) * D * 2;
    const char* vraw = (const char*)P.v + ((size_t)seq * P.rows * P.nkv + hk) * D * 2;

    // ---- requests: the rows' part of the rotary table, the query rows, the own rows, the first tiles
    constexpr int TPC = D / 4, TU = (TROWS * TPC + GA_THREADS - 1) / GA_THREADS, TU1 = 4;   // 16-byte units per thread; the first 4 do for K1 >= 5
    u32x4 tv[TU1];
    const u32x4* const tab_src = reinterpret_cast<const u32x4*>(P.table + (size_t)gB0 * (D / 2));
    const int tab_n = (g_last_wg - gB0 + K1) * TPC;   // positions of the rows of groups gB0 .. g_last_wg
    if (P.k > 0) {
#pragma unroll
        for (int i = 0; i < TU1; ++i) tv[i] = tab_src[min(tid + GA_THREADS * i, tab_n - 1)];
    }
    constexpr int QPI = 64 / PAIRS, QI = 32 / QPI;          // query rows per request of a wavefront, requests
    constexpr int OPI = GA_THREADS / PAIRS, OI = (OROWS + OPI - 1) / OPI;   // own rows per request of the workgroup, requests
    const int pj = tid % PAIRS;                             // this thread's pair of pieces
    uint4 qa[QI], qb[QI], ok[OI][2], ov[OI][2];
    {
        const char* src = (const char*)P.q + ((size_t)seq * P.rows * P.nq + h) * D * 2 + pj * 16;
#pragma unroll
        for (int i = 0; i < QI; ++i) {
            const char* a = src + (size_t)min(r0 + QPI * i + lane / PAIRS, r_last) * P.nq * D * 2;
            qa[i] = ldg_stream16_q(a);
            qb[i] = ldg_stream16_q(a + D);
        }
    }
    auto own_row = [&](int i) __attribute__((always_inline)) { return min(max(R0 - 16 + OPI * i + tid / PAIRS, 0), r_last); };
    if (P.k > 0) {
#pragma unroll
        for (int i = 0; i < OI; ++i) {
            const size_t off = (size_t)own_row(i) * rs + pj * 16;
            ok[i][0] = ld16_q(kraw + off);
            ok[i][1] = ld16_q(kraw + off + D);
            ov[i][0] = ld16_q(vraw + off);
            ov[i][1] = ld16_q(vraw + off + D);
        }
    }
    // staging of the real tokens' tiles: 8 threads per key
    const int skey = tid / 8, sj = tid % 8;
    const char* krot = (const char*)P.k_rot + (size_t)(seq * (size_t)P.nkv + hk) * P.T * D * 2;
    auto load_k = [&](int t, uint4 (&x)[NP]) __attribute__((always_inline)) {
        const char* kp = krot + (size_t)(unsigned)min(32 * t + skey, g_last_wg) * (2 * D) + sj * 16;
#pragma unroll
        for (int i = 0; i < NP; ++i) x[i] = ld16(kp + i * 128);
    };
    const unsigned K1rs = (unsigned)K1 * (unsigned)rs;
    auto load_v = [&](int t, uint4 (&x)[NP]) __attribute__((always_inline)) {
        const char* vp = vraw + (size_t)(unsigned)min(32 * t + skey, g_last_wg) * K1rs + sj * 16;
#pragma unroll
        for (int i = 0; i < NP; ++i) x[i] = ld16_q(vp + i * 128);
    };
    auto store_k = [&](int t, const uint4 (&x)[NP]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NP; ++i) *reinterpret_cast<uint4*>(smem + (t & 1) * KBUF + skey * KSTR + sj * 16 + i * 128) = x[i];
    };
    auto store_v = [&](int t, const uint4 (&x)[NP]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NP; ++i) *reinterpret_cast<uint4*>(smem + OFF_V + (t & 1) * VBUF + skey * VSTR + sj * 16 + i * 128) = x[i];
    };
    auto table_unit = [&](int u) __attribute__((always_inline)) { return reinterpret_cast<u32x4*>(smem + OFF_T + u / TPC * TROW + u % TPC * 16); };
    uint4 k0[NP], k1[NP], v0[NP], kst[NP], vst[NP];
    load_k(0, k0);
    load_k(1, k1);
    load_k(2, kst);
    load_v(0, v0);
    load_v(1, vst);
    if (P.k > 0) {
#pragma unroll
        for (int i = 0; i < TU1; ++i) *table_unit(min(tid + GA_THREADS * i, tab_n - 1)) = tv[i];
        if (tab_n > TU1 * GA_THREADS) {                     // (two or three rows per group: more positions)
            u32x4 tw[TU - TU1];
#pragma unroll
            for (int i = TU1; i < TU; ++i) tw[i - TU1] = tab_src[min(tid + GA_THREADS * i, tab_n - 1)];
#pragma unroll
            for (int i = TU1; i < TU; ++i) *table_unit(min(tid + GA_THREADS * i, tab_n - 1)) = tw[i - TU1];
        }
        __syncthreads();
    }

    // (a row R0 - 16 .. R0 - 1 of an earlier group is seen by nobody here and takes any entry of the table)
    // a pair of pieces of a row, rotated: cosines and sines of pairs 8 pj .. 8 pj + 7 at the row's position
    auto rotate = [&](uint4 xa, uint4 xb, const float4* tab, float scale, float (&ra)[8], float (&rb)[8]) __attribute__((always_inline)) {
        float a[8], b[8];
        unpack_group<bf16_t>(xa, a);
        unpack_group<bf16_t>(xb, b);
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const float4 cs = tab[e / 2];
            ra[e] = (a[e] * cs.x - b[e] * cs.y) * scale;
            rb[e] = (b[e] * cs.x + a[e] * cs.y) * scale;
            ra[e + 1] = (a[e + 1] * cs.z - b[e + 1] * cs.w) * scale;
            rb[e + 1] = (b[e + 1] * cs.z + a[e + 1] * cs.w) * scale;
        }
    };
    auto position = [&](int row) __attribute__((always_inline)) { return row - group_of(row) * P.k; };   // group + slot
    auto table_lds = [&](int pos) __attribute__((always_inline)) {
        return reinterpret_cast<const float4*>(smem + OFF_T + max(pos - gB0, 0) * TROW) + pj * 4;
    };

    // ---- the query rows by way of LDS into registers, as operands (lane (c, half): bytes [32 t + 16 half, +16) of row c at step
    // t, so both pieces of a pair), rotated in float32, scaled by log2(e) / sqrt(d), split into high and low parts
    bf16x8 qh[STEPS], ql[STEPS];
    {
        char* const sQ = smem + wave * (32 * KSTR);
        const float qscale = P.inv_sqrt_d * 1.4426950408889634f;
#pragma unroll
        for (int i = 0; i < QI; ++i) {
            const int rr = QPI * i + lane / PAIRS;
            *reinterpret_cast<uint4*>(sQ + rr * KSTR + pj * 16) = qa[i];
            *reinterpret_cast<uint4*>(sQ + rr * KSTR + (pj + PAIRS) * 16) = qb[i];
        }
        uint4 xa[STEPS / 2], xb[STEPS / 2];
        lds_sync_wave();
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int t = 0; t < STEPS / 2; ++t) {
            xa[t] = ld16(sQ + c * KSTR + 32 * t + 16 * half);
            xb[t] = ld16(sQ + c * KSTR + D + 32 * t + 16 * half);
        }
        const char* tab = smem + OFF_T + (position(qrow) - gB0) * TROW;
        if (P.k == 0) {                                     // (as many positions as rows: each wavefront's in its own area)
            char* const sT = smem + wave * TAREA;
            const int tq_last = r_last - w_first;
            u32x4 tq[TPC / 2];
#pragma unroll
            for (int i = 0; i < TPC / 2; ++i) {
                const int u = lane + 64 * i;
                tq[i] = reinterpret_cast<const u32x4*>(P.table)[(size_t)(unsigned)(w_first + min(u / TPC, tq_last)) * TPC + u % TPC];
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < TPC / 2; ++i) *reinterpret_cast<u32x4*>(sT + (lane + 64 * i) / TPC * TROW + (lane + 64 * i) % TPC * 16) = tq[i];
            lds_sync_wave();
            __builtin_amdgcn_wave_barrier();
            tab = sT + min(c, tq_last) * TROW;
        }
#pragma unroll
        for (int t = 0; t < STEPS / 2; ++t) {
            float ra[8], rb[8];
            rotate(xa[t], xb[t], reinterpret_cast<const float4*>(tab) + (2 * t + half) * 4, qscale, ra, rb);
            unsigned hi[4];
            qh[t] = split_hi(ra, hi);
            ql[t] = split_lo(ra, hi);
            qh[t + STEPS / 2] = split_hi(rb, hi);
            ql[t + STEPS / 2] = split_lo(rb, hi);
        }
    }

    // of this lane's query: the reference of the exponentials (both halves agree) and the half's sum.  The reference starts at
    // the lowest finite number, not at -inf: as long as a row has seen no key, or only keys whose scores overflowed to -inf,
    // their exponentials against it are exp2(-inf) = 0, not exp2(-inf + inf)
    float m_run = -3.402823466e38f, l_run = 0.f;
    f32x16 o[NJ];                                           // O^T: column 32 j + 8 (i / 4) + 4 half + i % 4 of this lane's query
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[j][i] = 0.f;
    // The parts of a tile's work.  Scores: kf(step) = the 32 K rows as MFMA operand (key c, bytes [32 step + 16 half, +16));
    // the lane's i-th score is that of key 8 (i / 4) + i % 4 + 4 half
    auto scores = [&](auto kf) __attribute__((always_inline)) {
        f32x16 x;
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = 0.f;
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            const bf16x8 f = kf(st);
            x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, qh[st], x, 0, 0, 0);
            x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, ql[st], x, 0, 0, 0);
        }
        return x;
    };
    auto mask = [&](f32x16& x, int lo, int hi) __attribute__((always_inline)) {   // keys lo .. hi (counted from 4 half) are visible
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int key = 8 * (i / 4) + i % 4;
            x[i] = (key >= lo && key <= hi) ? x[i] : -INFINITY;
        }
    };
    // the reference follows the maximum only when that has moved up by more than GA_LAZY (in units of ln 2): sums and outputs
    // are relative to the same reference, so the quotient is the same, and most tiles need no rescaling
    auto highest = [&](const f32x16& x, float mt) __attribute__((always_inline)) {   // of the query's scores, and mt
#pragma unroll
        for (int i = 0; i < 16; ++i) mt = fmaxf(mt, x[i]);
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mt), __float_as_uint(mt), false, false);
        return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    };
    auto follow = [&](float mt) __attribute__((always_inline)) {
        const bool moved = mt > m_run + GA_LAZY;            // (also the first finite scores of a row)
        if (__any(moved)) {
            const float m_new = moved ? mt : m_run;
            const float alpha = moved ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.f;
            l_run *= alpha;
            m_run = m_new;
#pragma unroll
            for (int j = 0; j < NJ; ++j) o[j] *= alpha;
        }
    };
    // exponentials against m, P.V: vf(j, m) = V^T as operand, columns 32 j + c, keys 16 m + 4 half + 0..3 and 16 m + 8 + 4 half + 0..3
    // (of the tile's first 16 keys or of all 32)
    auto accumulate = [&](const f32x16& x, float m, auto halves, auto vf) __attribute__((always_inline)) {
        float pr[2][8];
        float l0 = 0.f, l1 = 0.f;
#pragma unroll
        for (int i = 0; i < 8 * halves; ++i) {
            const float e = __builtin_amdgcn_exp2f(x[i] - m);
            pr[i / 8][i % 8] = e;
            if (i & 1) l1 += e; else l0 += e;
        }
        l_run += l0 + l1;
        bf16x8 ph[2], pl[2];
#pragma unroll
        for (int m2 = 0; m2 < halves; ++m2) {
            unsigned hi8[4];
            ph[m2] = split_hi(pr[m2], hi8);
            pl[m2] = split_lo(pr[m2], hi8);
        }
#pragma unroll
        for (int j = 0; j < NJ; j += 2)
#pragma unroll
            for (int m2 = 0; m2 < halves; ++m2) {
                const bf16x8 va = vf(j, m2), vb = vf(j + 1, m2);
                o[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, ph[m2], o[j], 0, 0, 0);
                o[j + 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vb, ph[m2], o[j + 1], 0, 0, 0);
                o[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pl[m2], o[j], 0, 0, 0);
                o[j + 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vb, pl[m2], o[j + 1], 0, 0, 0);
            }
    };
    const int vkey = (lane & 15) >> 2, vhi = (lane >> 4) & 1;   // V^T from rows in LDS: 16 lanes read 4 keys x 32 bytes and get 4 keys of a column each
    auto transposed = [&](const char* a, int rows8) __attribute__((always_inline)) {
        const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)a);
        const s16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(a + rows8));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    // ---- the [MASK] keys of the own groups: rows in LDS, K rotated (and rounded as cached keys are); 16-byte K pieces stand at
    // piece ^ key, 32-byte V chunks at chunk ^ f(key).  A wavefront's queries see rows among their own 32 and, where its
    // first row is not the first of its group, among the 16 before
    if (P.k > 0) {
        uint4 rk[OI][2];
#pragma unroll
        for (int i = 0; i < OI; ++i) {
            float ra[8], rb[8];
            rotate(ok[i][0], ok[i][1], table_lds(position(own_row(i))), 1.f, ra, rb);
            unsigned hi[4];
            rk[i][0] = __builtin_bit_cast(uint4, split_hi(ra, hi));
            rk[i][1] = __builtin_bit_cast(uint4, split_hi(rb, hi));
        }
        __syncthreads();                                    // table and query areas have been read
#pragma unroll
        for (int i = 0; i < OI; ++i) {
            const int orow = OPI * i + tid / PAIRS;
            const int ksw = D == 128 ? orow & 15 : (orow >> 1) & 7, vsw = D == 128 ? (orow & 3) << 1 : orow & 2;
            char* const kd = smem + orow * (2 * D) + ((pj ^ ksw) << 4);
            char* const vd = smem + OFF_OV + orow * (2 * D) + (((pj >> 1) ^ vsw) << 5) + ((pj & 1) << 4);
            if (OPI * i + OPI <= OROWS || orow < OROWS) {
                *reinterpret_cast<uint4*>(kd) = rk[i][0];
                *reinterpret_cast<uint4*>(smem + ((kd - smem) ^ (PAIRS * 16))) = rk[i][1];
                *reinterpret_cast<uint4*>(vd) = ov[i][0];
                *reinterpret_cast<uint4*>(smem + OFF_OV + ((vd - smem - OFF_OV) ^ (PAIRS * 16))) = ov[i][1];
            }
        }
        __syncthreads();
        const int kro = c * (2 * D) + ((half ^ (D == 128 ? c & 15 : (c >> 1) & 7)) << 4);
        const int vro = (4 * half + vkey) * (2 * D) + ((vhi ^ (D == 128 ? vkey << 1 : vkey & 2)) << 5) + (lane & 3) * 8;
        if (active) {
            // both tiles' scores, one reference, then the values: of the tile before, the 16 keys that are not the own tile's, too
            auto own_scores = [&](int first, int last, f32x16& x) __attribute__((always_inline)) {   // first: layout row of the tile's first key
                const char* kt = smem + (first - R0 + 16) * (2 * D);
                x = scores([&](int st) __attribute__((always_inline)) { return __builtin_bit_cast(bf16x8, ld16(kt + (kro ^ (st << 5)))); });
                mask(x, qg * K1 + 1 - first - 4 * half, last - first - 4 * half);
            };
            auto own_values = [&](int first, int j, int m2) __attribute__((always_inline)) {
                return transposed(smem + (first - R0 + 16) * (2 * D) + OFF_OV + m2 * 16 * 2 * D + (vro ^ (j << 6)), 8 * 2 * D);
            };
            f32x16 x;
            own_scores(r0, qrow, x);
            if (wg0 * K1 != r0) {
                f32x16 y;
                own_scores(r0 - 16, min(qrow, r0 - 1), y);
                float mt = y[0];
#pragma unroll
                for (int i = 1; i < 8; ++i) mt = fmaxf(mt, y[i]);
                follow(highest(x, mt));
                accumulate(y, m_run, std::integral_constant<int, 1>{}, [&](int j, int m2) __attribute__((always_inline)) { return own_values(r0 - 16, j, m2); });
            } else {
                follow(highest(x, x[0]));
            }
            accumulate(x, m_run, std::integral_constant<int, 2>{}, [&](int j, int m2) __attribute__((always_inline)) { return own_values(r0, j, m2); });
        }
    }
    __syncthreads();                                        // the stages' buffers are free

    // ---- the real tokens.  K is staged one tile further than V: a tile's scores are worked out while the tile before is
    // exponentiated and multiplied with its values
    store_k(0, k0);
    store_k(1, k1);
    store_v(0, v0);
    const int kr = c * KSTR + half * 16, vr = OFF_V + (4 * half + vkey) * VSTR + vhi * 32 + (lane & 3) * 8;
    auto stage_scores = [&](int t) __attribute__((always_inline)) {
        const char* a = smem + (t & 1) * KBUF + kr;
        return scores([&](int st) __attribute__((always_inline)) { return __builtin_bit_cast(bf16x8, ld16(a + 32 * st)); });
    };
    __syncthreads();
    f32x16 s = stage_scores(0);
    __syncthreads();
    const int real_end = active ? wg1 / 32 + 1 : 0, whole_end = (wg0 + 1) / 32;   // tiles this wavefront's queries see some of, all of
    auto visible = [&](int t, f32x16& x) __attribute__((always_inline)) { mask(x, 0, qg - 32 * t - 4 * half); };
    auto stage = [&](int t) __attribute__((always_inline)) {
        store_k(t, kst);                                    // (tile t + 2's, into the buffer of tile t, whose scores are known)
        store_v(t + 1, vst);
        load_k(t + 3, kst);
        load_v(t + 2, vst);
    };
    auto values = [&](int t) __attribute__((always_inline)) {
        accumulate(s, m_run, std::integral_constant<int, 2>{}, [&](int j, int m2) __attribute__((always_inline)) { return transposed(smem + (t & 1) * VBUF + vr + j * 64 + m2 * 16 * VSTR, 8 * VSTR); });
    };
    int t = 0;
    if (real_end > 0) {
        if (whole_end == 0) visible(0, s);
        follow(highest(s, s[0]));
        auto step = [&](auto masked) __attribute__((always_inline)) {
            stage(t);
            f32x16 sn = stage_scores(t + 1);
            values(t);
            if constexpr (masked) visible(t + 1, sn);
            const float mt = highest(sn, sn[0]);
            s = sn;
            follow(mt);
            __syncthreads();
        };
        for (; t + 1 < min(whole_end, real_end); ++t) step(std::false_type{});
        for (; t + 1 < real_end; ++t) step(std::true_type{});
        stage(t);
        values(t);
        __syncthreads();
        ++t;
    }
    for (; t < n_real; ++t) {
        stage(t);
        __syncthreads();
    }

    // ---- output: OCOLS columns at a time by way of the wavefront's LDS area, divided by the rows' sums
    const auto lw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
    const float den = __uint_as_float(lw[0]) + __uint_as_float(lw[1]), inv = 1.f / den;   // (every row sees at least its own real token)
    float z[2] = {0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < 16; i += 2) z[i / 2 & 1] = abs_max3(z[i / 2 & 1], o[j][i], o[j][i + 1]);
    const u64 zb = __ballot(den == den && !(z[0] < INFINITY && z[1] < INFINITY) && r0 + c < P.rows);
    constexpr int PCS = OCOLS / 4;                          // 16-byte pieces of a row
    char* const sO = smem + wave * (32 * OCOLS * 4);
    float* obase = P.out + ((size_t)seq * P.rows * P.nq + h) * D;
#pragma unroll
    for (int j0 = 0; j0 < NJ; j0 += OCOLS / 32) {
#pragma unroll
        for (int j = 0; j < OCOLS / 32; ++j)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                f32x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = o[j0 + j][4 * i4 + e] * inv;
                *reinterpret_cast<f32x4*>(sO + (c * PCS + ((8 * j + 2 * i4 + half) ^ (c & (PCS - 1)))) * 16) = w;
            }
        lds_sync_wave();
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < PCS / 2; ++u) {
            const int rr = (64 / PCS) * u + lane / PCS, pc = lane % PCS;
            const f32x4 w = *reinterpret_cast<const f32x4*>(sO + (rr * PCS + (pc ^ (rr & (PCS - 1)))) * 16);
            if (r0 + rr < P.rows) stg_stream16_q(obase + (size_t)(r0 + rr) * P.nq * D + 32 * j0 + 4 * pc, w);
        }
        lds_sync_wave();
        __builtin_amdgcn_wave_barrier();
    }
    const unsigned alone = (unsigned)(zb | zb >> 32);
    if (alone) ga_rows_alone<bf16_t, D>(ga_args(), seq, h, r0, alone, lane);
}

size_t a256(size_t v) { return (v + 255) & ~(size_t)255; }

int check(const ps_group_attn_args* a) {
    if (!a) return PS_ERR_NULL;
    if (a->seqs < 1 || a->tokens < 1 || a->k < 0 || a->n_heads < 1 || a->n_kv_heads < 1 || a->head_dim < 1) return PS_ERR_SHAPE;
    if (a->dtype != PS_F32 && a->dtype != PS_BF16) return PS_ERR_SHAPE;
    if (a->n_heads % a->n_kv_heads != 0 || !(a->rope_base > 0.f)) return PS_ERR_SHAPE;
    if (a->head_dim != 64 && a->head_dim != 128) return PS_ERR_UNSUPPORTED;
    if (a->k > 15 || (long long)a->tokens + a->k > (1 << 20)) return PS_ERR_UNSUPPORTED;
    if (a->n_heads > 65535 || a->seqs > 65535) return PS_ERR_UNSUPPORTED;
    if ((long long)(a->k + 1) * a->n_kv_heads * a->head_dim * 4 > (1LL << 27)) return PS_ERR_UNSUPPORTED;   // 32-bit offsets inside a key tile
    if (a->dtype == PS_F32 && ((long long)a->tokens * (a->k + 1) + GF_ROWS - 1) / GF_ROWS * a->n_heads > GA_MAX_WG) return PS_ERR_UNSUPPORTED;   // (its rows would be terabytes)
    return PS_OK;
}

struct GaLayout { size_t table, k_rot, total; };
GaLayout layout(const ps_group_attn_args* a) {
    GaLayout L;
    const size_t rows = (size_t)a->tokens * (a->k + 1), esz = a->dtype == PS_BF16 ? 2 : 4;
    L.table = 0;
    L.k_rot = a256((size_t)(a->tokens + a->k) * (a->head_dim / 2) * sizeof(float2));
    L.total = L.k_rot + a256((size_t)a->seqs * rows * a->n_kv_heads * a->head_dim * esz);
    return L;
}

// How a call is launched: the attention's kernel with its grid, and the rotation's
enum { GA_F32 = 0, GA_TILES = 1, GA_WIDE = 2, GA_F32_32 = 3, GA_F32_SHORT = 4 };   // (GA_F32_32: ga_attn_f32_kernel with blocks of 32 rows)
struct GaLaunch {
    int kernel;
    int threads;          // of the attention's workgroups (the rotation's: 256)
    dim3 rope, attn;
};
dim3 grid_xy(long long workgroups, int z) {
    const unsigned x = (unsigned)std::min(workgroups, (long long)GA_GRID_X);   // (HIP's own host min is that of ints)
    return dim3(x, (unsigned)((workgroups + x - 1) / x), z);
}
GaLaunch plan(const GaParams& P, int dtype, int head_dim) {
    GaLaunch L;
    L.threads = GA_THREADS;
    if (dtype == PS_BF16) {
        // The wide kernel, except where the real tokens' keys are a single stage and the groups' own rows are most of the work:
        // there the 16-row kernel, whose workgroups are half as long, is the faster one as long as
        // - groups straddle the wide kernel's 32-row tiles, which then looks at the 16 rows before a tile, too;
        // - its workgroups, which are up to three times as many, find a compute unit each;
        // - rotating all key rows for it, not only the real tokens', costs no time: up to 8192 rows.
        // us, 16-row / wide kernel, whole calls at head_dim 128: T 16, k 8, 8 heads 12.9 / 13.9; T 32, k 8, 32 / 8 heads (256 workgroups)
        // 13.5 / 14.8; T 32, k 4, 8 heads 13.7 / 13.9; T 8, k 10, 8 heads 13.0 / 13.7; T 1, k 4 11.0 / 12.2; but k 3 (T 24) 13.8 / 13.0,
        // k 7 (T 24) 14.0 / 13.1, k 15 (T 24) 14.7 / 13.3; 4 x T 16, k 8, 32 / 8 heads (512 workgroups) 16.8 / 14.9; T 32, k 10,
        // 32 heads (11264 key rows) 15.5 / 14.6, 4 x T 16, k 4, 32 heads (10240) 16.0 / 14.4; 8 x T 32, k 8, 40 heads 50 / 35
        const long long blocks = (long long)((P.rows + GW_ROWS - 1) / GW_ROWS) * P.nq * P.seqs;
        const long long tile_wg = (long long)((P.ntiles + GA_WAVES - 1) / GA_WAVES) * P.nq * P.seqs, key_rows = (long long)P.seqs * P.rows * P.nkv;
        const bool tiles = P.T <= 32 && P.k >= 4 && (P.T == 1 || 32 % (P.k + 1) != 0) && tile_wg <= 256 && key_rows <= 8192;
        L.kernel = blocks > GA_MAX_WG || tiles ? GA_TILES : GA_WIDE;
        L.attn = L.kernel == GA_WIDE ? grid_xy(blocks, 1) : dim3((P.ntiles + GA_WAVES - 1) / GA_WAVES, P.nq, P.seqs);
    } else {
        // (both sides of the line stand at ga_attn_f32)
        const bool is_short = (long long)((P.rows + 31) / 32) * P.nq * P.seqs <= (head_dim == 64 ? 704 : 400);
        const int rows = is_short ? 32 : 16 * GF_QT(head_dim);
        const long long blocks = (long long)((P.rows + rows - 1) / rows) * P.nq;
        L.kernel = is_short ? GA_F32_SHORT : rows == 32 ? GA_F32_32 : GA_F32;
        L.threads = is_short ? 512 : 128 * GF_QT(head_dim);
        L.attn = grid_xy(blocks, P.seqs);
    }
    // the rotation: a workgroup per position; where positions are few, several (of at most one item per thread each) share one's rows
    const long long items = (long long)P.seqs * P.nkv * (head_dim / 8) * (L.kernel == GA_WIDE ? 1 : P.k + 1);
    L.rope = dim3(P.T + P.k, (unsigned)std::max(1LL, std::min((items + 255) / 256, 2048LL / (P.T + P.k))));
    return L;
}

template <typename WT, int D>
int launch(const GaParams& P, const GaLaunch& L, hipStream_t s) {
    if constexpr (Traits<WT>::BF) {
        if (L.kernel == GA_WIDE) {
            hipLaunchKernelGGL((ga_rope_kernel<WT, D, false>), L.rope, dim3(256), 0, s, P);
            hipLaunchKernelGGL((ga_attn_wide_kernel<D>), L.attn, dim3(GA_THREADS), 0, s, P);
        } else {
            hipLaunchKernelGGL((ga_rope_kernel<WT, D, true>), L.rope, dim3(256), 0, s, P);
            hipLaunchKernelGGL((ga_attn_bf16_kernel<D>), L.attn, dim3(GA_THREADS), 0, s, P);
        }
    } else {
        hipLaunchKernelGGL((ga_rope_kernel<WT, D, true>), L.rope, dim3(256), 0, s, P);
        if (L.kernel == GA_F32_SHORT) hipLaunchKernelGGL((ga_attn_f32_short_kernel<D>), L.attn, dim3(L.threads), 0, s, P);
        else hipLaunchKernelGGL((ga_attn_f32_kernel<D>), L.attn, dim3(L.threads), 0, s, P);
    }
    return hipGetLastError() == hipSuccess ? PS_OK : PS_ERR_DEVICE;
}

// everything but the pointers
GaParams shape(const ps_group_attn_args* a) {
    GaParams P = {};
    P.seqs = a->seqs; P.T = a->tokens; P.k = a->k; P.nq = a->n_heads; P.nkv = a->n_kv_heads;
    P.rows = a->tokens * (a->k + 1);
    P.gpt = 16 / (a->k + 1);
    P.k1_magic = (unsigned)((0x100000000ull + a->k) / (unsigned)(a->k + 1));
    P.ntiles = (a->tokens + P.gpt - 1) / P.gpt;
    P.by_heads = ga_div((unsigned)P.nq * (unsigned)P.seqs);   // (up to 65535^2: beyond an int)
    P.by_slots = ga_div((unsigned)P.nkv * (unsigned)P.seqs);
    P.by_nkv = ga_div(P.nkv);
    P.group = P.nq / P.nkv;
    P.inv_sqrt_d = (float)(1.0 / sqrt((double)a->head_dim));
    P.log2_base = log2((double)a->rope_base);
    return P;
}

}   // namespace

extern "C" size_t ps_group_attention_workspace_bytes(const ps_group_attn_args* a) {
    return check(a) == PS_OK ? layout(a).total : 0;
}

extern "C" int ps_group_attention(const ps_group_attn_args* a, void* stream) {
    const int st = check(a);
    if (st != PS_OK) return st;
    if (!a->q || !a->k_ || !a->v || !a->out || !a->workspace) return PS_ERR_NULL;
    const GaLayout L = layout(a);
    if (a->workspace_bytes < L.total || ((uintptr_t)a->workspace & 255)) return PS_ERR_WORKSPACE;
    GaParams P = shape(a);
    const GaLaunch G = plan(P, a->dtype, a->head_dim);
    P.q = a->q; P.k_ = a->k_; P.v = a->v; P.out = a->out;
    char* ws = (char*)a->workspace;
    P.table = (float2*)(ws + L.table); P.k_rot = ws + L.k_rot;
    hipStream_t s = (hipStream_t)stream;
    if (a->dtype == PS_BF16) return a->head_dim == 128 ? launch<bf16_t, 128>(P, G, s) : launch<bf16_t, 64>(P, G, s);
    return a->head_dim == 128 ? launch<float, 128>(P, G, s) : launch<float, 64>(P, G, s);
}

// see ps_draft_debug.h
extern "C" int ps_train_debug_launch(const ps_group_attn_args* a, unsigned* out) {
    const int st = check(a);
    if (st != PS_OK) return st;
    if (!out) return PS_ERR_NULL;
    const GaLaunch G = plan(shape(a), a->dtype, a->head_dim);
    const unsigned v[8] = {(unsigned)G.kernel, G.attn.x, G.attn.y, G.attn.z, (unsigned)G.threads, G.rope.x, G.rope.y, 256u};
    for (int i = 0; i < 8; ++i) out[i] = v[i];
    return PS_OK;
}
