// Dense contractions of the path in fp32, on the bfloat16 matrix cores (v_mfma_f32_32x32x16_bf16), gfx950.
//
//   forward   A_p^l  = act( Z_p W^l (+ X_p W_s^l) + b^l )        [n_p x d_in] [d_in x d_out]
//   backward  dZ_p   = dY_p (W^l)^T                              [n_p x d_out][d_out x d_in]
//             grad W^l += Z_p^T dY_p                             reduction over the n_p rows
//
// The fp32 matrix instruction does 64 flop per cycle and SIMD, the bfloat16 one 1024.  Every fp32
// operand is split on its way into LDS into three bfloat16 numbers whose sum it is, exactly
//     x = h + m + l,   h = round(x), m = round(x - h), l = x - h - m    (8 + 8 + 8 significant bits)
// and a product is taken as the six terms
//     l h' + m m' + h l' + m h' + h m' + h h'      (each exact in fp32, accumulated in fp32).
// What is left out (m l' + l m' + l l') is at most 2^-25 of |x y| and has no sign of its own; the six
// terms of 16 k are added in 6 steps where the fp32 instruction rounds 8 times.
// What the split cannot represent - infinities, NaN, magnitudes that round up to infinity - makes
// the element's sum a NaN or an infinity; such elements are computed again as a chain of fp32 fused
// multiply-adds (bad elements only, see the end of the kernel).
//
// One workgroup of 4 wavefronts (2 x 2) owns a BM x BN tile of C.  K is walked in steps of BK
// through a double-buffered LDS stage.  The unit of loading, splitting and LDS is eight consecutive k
// of one row of the operand: one lane's share of an MFMA operand, 16 bytes in each of the three planes.
// K past a segment's end is zero-filled in LDS, never in memory; rows past m or n repeat the last one
// and are not stored.
//
// Bound by the splitting beside the matrix work: per stage and wavefront 24 matrix instructions of 32
// cycles and about 150 vector instructions of 4.  Against the fp32 instruction (same tiles), ms:
//   forward   1.2 M rows  256 x 256   1.55 -> 1.05      3 M rows  128 x 128   1.11 -> 0.86
//   backward  1.2 M rows  256 x 256   1.56 -> 1.06      3 M rows  128 x 172   1.47 -> 1.18
//   gradient  1.2 M rows  256 x 256   1.61 -> 1.14      3 M rows  128 x 128   1.11 -> 0.81
// Relative error against 64 bits (normal inputs): 2.9e-7 -> 2.4e-7 (K = 256), 1.4e-7 -> 1.1e-7
// (K = 64), gradient over 1.2 M rows 8.4e-7 -> 7.3e-7.  Magnitudes below 1e-34 lose bits: the
// matrix cores read bfloat16 denormals (here those of m and l) as zero.
#include "gnn_internal.h"
#include <cfloat>
#include <cstdlib>

namespace gnnmi {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kThreads = 256;
constexpr int BK = 16;
constexpr int GP = BK / 8;          // groups of eight k in a stage
// Rows of a plane are 16 bytes, one group of k after the other; the pad puts the groups that the
// lanes of a k-fast store write together into different banks (the reads are consecutive anyway).
constexpr int PADR = 16 / GP;

struct Operand {         // a matrix operand restricted to one K segment
    const float* p;
    int64_t ld;
};

__device__ inline uint32_t to_bf16x2(float a, float b)      // v_cvt_pk_bf16_f32: to nearest even
{
    const floatx2 f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}
// x minus one half of a pair, in one v_dot2_f32_bf16: the other half times 0 is 0, or NaN for an infinity.
// (The pairs (-1, 0) and (0, -1) are kept from the compiler: as a literal the first becomes the inline
// constant -1.0, which the instruction reads as the second.)
__device__ inline float minus_half(float x, uint32_t pair, uint32_t selector)
{
    asm("" : "+s"(selector));
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), __builtin_bit_cast(bf16x2, selector), x, false);
}
__device__ inline float minus_low(float x, uint32_t pair) { return minus_half(x, pair, 0x0000BF80u); }
__device__ inline float minus_high(float x, uint32_t pair) { return minus_half(x, pair, 0xBF800000u); }
__device__ inline void split2(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l)
{
    h = to_bf16x2(a, b);
    const float a1 = minus_low(a, h), b1 = minus_high(b, h);
    m = to_bf16x2(a1, b1);
    l = to_bf16x2(minus_low(a1, m), minus_high(b1, m));
}

// One operand's stage of BT rows x BK k: x[j] is the j-th k of this thread's group.  (BT = 64 has
// work for half of the wavefronts, from wavefront `first` on.)  Consecutive threads take the groups of
// a row of a k-fast operand, else consecutive rows, whose elements of one k are consecutive in memory.
template <int BT, bool KFAST, bool VEC>
struct Stage {
    static constexpr int GROUPS = BT * GP;
    static_assert(GROUPS <= kThreads, "one group per thread");
    static constexpr int PLANE = GP * (BT + PADR);             // 16-byte units
    float x[8];
    const float* q;        // k-fast: this thread's group of the next stage; else: its first row of k (uniform)
    int64_t ld;
    int32_t row, group;
    uint32_t col;          // else: element of that row, in bytes
    bool on;

    __device__ inline Stage(int first)
    {
        const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64) - (GROUPS < kThreads ? first : 0);
        const int t = 64 * w + (int)(threadIdx.x & 63);
        on = GROUPS == kThreads || (w >= 0 && w < GROUPS / 64);
        row = KFAST ? t / GP : t % BT;
        group = KFAST ? t % GP : 64 * w / BT;
    }
    // rows past the end read the last one
    __device__ inline void begin(const Operand& o, int64_t row0, int64_t nrows, int64_t k0)
    {
        const int64_t r = row0 + row < nrows ? row0 + row : nrows - 1;
        ld = o.ld;
        q = o.p + (KFAST ? r * ld + k0 + 8 * group : (k0 + 8 * group) * ld);
        col = 4u * (uint32_t)r;
    }
    __device__ inline float at(int32_t j) const
    {
        return KFAST ? q[j] : *reinterpret_cast<const float*>(reinterpret_cast<const char*>(q + j * ld) + col);
    }
    __device__ inline void advance() { q += KFAST ? BK : BK * ld; }
    // `left`: k of the segment from this stage on.  Loads past its end are clamped to its last k.
    __device__ inline void load(int32_t left)
    {
        if (GROUPS < kThreads && !on) return;
        const int32_t mine = left - 8 * group;
        if (KFAST && VEC) {
            const float4 a = *reinterpret_cast<const float4*>(q + (mine >= 4 ? 0 : mine - 4));
            const float4 b = *reinterpret_cast<const float4*>(q + (mine >= 8 ? 4 : mine - 4));
            x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
            x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = at(j < mine ? j : mine - 1);
        }
    }
    // flip: the sign bit, or 0.  Of the k past the segment's end one operand (ZERO) is zeroed: the other
    // repeats an element of the same row, which, were it infinite, has made the row's sums so already.
    template <bool ZERO>
    __device__ inline void store(uint4* S, int32_t left, uint32_t flip)
    {
        if (GROUPS < kThreads && !on) return;
        if (ZERO) {
            const int32_t mine = left - 8 * group;
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = (KFAST && VEC ? (j & 4) : j) < mine ? x[j] : 0.f;
        }
        uint32_t h[4], m[4], l[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float a = __uint_as_float(__float_as_uint(x[2 * j]) ^ flip);
            const float b = __uint_as_float(__float_as_uint(x[2 * j + 1]) ^ flip);
            split2(a, b, h[j], m[j], l[j]);
        }
        uint4* d = S + group * (BT + PADR) + row;
        d[0] = make_uint4(h[0], h[1], h[2], h[3]);
        d[PLANE] = make_uint4(m[0], m[1], m[2], m[3]);
        d[2 * PLANE] = make_uint4(l[0], l[1], l[2], l[3]);
    }
};

struct GemmArgs {
    Operand a[2], b[2];      // up to two K segments
    int32_t kseg[2];         // K of each segment (second may be 0)
    float* c;
    int64_t ldc;
    int64_t m;               // rows of C
    int32_t n;               // columns of C
    const float* bias;
    int32_t relu;
    int32_t accumulate;
    const float* add;        // added before the activation, may be null
    int64_t ldadd;
    int64_t split_chunk;     // K per split (multiple of BK); 0 = no split
    int64_t split_stride;    // elements between the partial C of consecutive splits
    const int2* splits;      // K range of every split (null: split_chunk apart)
    int32_t nt_1d;           // > 0: one-dimensional grid over (M tile, N tile), see tile_of_block
};

// Which tile a workgroup of a one-dimensional grid owns.  Workgroups are dealt to the 8 XCDs
// round-robin, each XCD with its own L2: block b runs on XCD b % 8 as that XCD's (b / 8)-th
// workgroup.  The workgroups of one XCD walk all N tiles of an M tile before the next M tile,
// so the rows of A they share are fetched into that L2 once instead of once per N tile.
__device__ inline bool tile_of_block(int64_t b, int64_t mt, int32_t nt, int64_t& mtile, int32_t& ntile)
{
    const int64_t slot = b >> 3;
    ntile = (int32_t)(slot % nt);
    mtile = (slot / nt) * 8 + (b & 7);
    return mtile < mt;
}

// A_KFAST: A(m,k) = a[m*lda + k]   (else a[k*lda + m])
// B_KFAST: B(k,n) = b[n*ldb + k]   (else b[k*ldb + n])
// An element of C is the same sum in the same order whatever the tile.
template <int BM, int BN, bool A_KFAST, bool B_KFAST, bool VEC_A, bool VEC_B>
__global__ __launch_bounds__(kThreads, 3) void k_gemm(const GemmArgs g)
{
    constexpr int WM = BM / 2, WN = BN / 2;   // wave tile
    constexpr int TM = WM / 32, TN = WN / 32; // 32x32 MFMA tiles per wave
    using StageA = Stage<BM, A_KFAST, VEC_A>;
    using StageB = Stage<BN, B_KFAST, VEC_B>;
    __shared__ __attribute__((aligned(16))) uint4 As[2][3 * StageA::PLANE];
    __shared__ __attribute__((aligned(16))) uint4 Bs[2][3 * StageB::PLANE];

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wm0 = (wave >> 1) * WM, wn0 = (wave & 1) * WN;
    int64_t mtile = blockIdx.x;
    int32_t ntile = blockIdx.y;
    if (g.nt_1d > 0 && !tile_of_block(blockIdx.x, (g.m + BM - 1) / BM, g.nt_1d, mtile, ntile)) return;
    const int64_t m0 = mtile * BM;
    const int32_t n0 = ntile * BN;

    // K range of this workgroup (split-K only with a single segment)
    int64_t kbeg = 0, kend0 = g.kseg[0];
    float* cbase = g.c;
    if (g.split_chunk > 0) {
        kbeg = (int64_t)blockIdx.z * g.split_chunk;
        kend0 = kbeg + g.split_chunk < kend0 ? kbeg + g.split_chunk : kend0;
        if (g.splits) {
            kbeg = g.splits[blockIdx.z].x;
            kend0 = g.splits[blockIdx.z].y;
        }
        cbase += (int64_t)blockIdx.z * g.split_stride;
    }
    const int32_t tiles0 = kend0 > kbeg ? (int32_t)((kend0 - kbeg + BK - 1) / BK) : 0;
    const int32_t ntiles = tiles0 + (g.kseg[1] + BK - 1) / BK;

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    StageA sa(0);
    StageB sb(BM == 64 ? 2 : 0);
    int32_t left = 0;                  // k of the segment from the stage that is loaded next
    auto begin = [&](int seg) {
        const int64_t k0 = seg == 0 ? kbeg : 0;
        left = (int32_t)((seg == 0 ? kend0 : (int64_t)g.kseg[1]) - k0);
        sa.begin(g.a[seg], m0, g.m, k0);
        sb.begin(g.b[seg], n0, g.n, k0);
    };
    // The matrix cores round sums down, not to nearest: a bias of half a unit per step, which the many
    // partial sums of a weight gradient would add up (gradient over 1.2 M rows: relative error 2.7e-6
    // instead of 8e-7).  So A, and the sums with it, changes its sign for the second and third quarter
    // of the stages: + - - +, in which a bias that grows with the sums cancels.
    const int32_t turn0 = ntiles / 4, turn1 = turn0 + ntiles / 2;       // (the last stage is a positive one)
    auto negative = [&](int32_t t) { return t >= turn0 && t < turn1; };
    auto store = [&](int32_t t) {
        sa.template store<false>(As[t & 1], left, negative(t) ? 0x80000000u : 0u);
        sb.template store<true>(Bs[t & 1], left, 0u);
        sa.advance();
        sb.advance();
        left -= BK;
    };
    const int half = lane >> 5, xl = lane & 31;
    auto multiply = [&](int32_t t) {
        const uint4* ap = As[t & 1] + half * (BM + PADR) + wm0 + xl;
        const uint4* bp = Bs[t & 1] + half * (BN + PADR) + wn0 + xl;
        bf16x8 av[3][TM], bv[3][TN];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
#pragma unroll
            for (int i = 0; i < TM; ++i) av[p][i] = __builtin_bit_cast(bf16x8, ap[p * StageA::PLANE + 32 * i]);
#pragma unroll
            for (int j = 0; j < TN; ++j) bv[p][j] = __builtin_bit_cast(bf16x8, bp[p * StageB::PLANE + 32 * j]);
        }
        constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};   // small terms first
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[PA[q]][i], bv[PB[q]][j], acc[i][j], 0, 0, 0);
    };
    auto negate = [&] {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = -acc[i][j][r];
    };

    if (ntiles > 0) {
        begin(tiles0 > 0 ? 0 : 1);
        sa.load(left);
        sb.load(left);
        store(0);
        __syncthreads();
        for (int32_t t = 0; t + 1 < ntiles; ++t) {
            if (negative(t) != negative(t - 1)) negate();
            if (t + 1 == tiles0) begin(1);
            sa.load(left);
            sb.load(left);
            // keep the loads where they are: left alone, the scheduler sinks them below the
            // MFMA block, right in front of the wait that precedes the LDS store
            __builtin_amdgcn_sched_barrier(0);
            multiply(t);
            store(t + 1);
            __syncthreads();
        }
        if (negative(ntiles - 2)) negate();
        multiply(ntiles - 1);
    }

    // elements whose sum is no finite number (0 times it is NaN)
    uint64_t bad = 0;
    float zero = 0.f;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) zero = fmaf(acc[i][j][r], 0.f, zero);
    if (zero != 0.f) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (!(fabsf(acc[i][j][r]) <= FLT_MAX)) bad |= 1ull << ((i * TN + j) * 16 + r);
    }

    // epilogue: lane holds C[8 (r/4) + 4 (lane/32) + r%4][lane%32] of each 32x32 tile
    const bool plain = !g.relu && !g.accumulate && !g.add;
    auto put = [&](int64_t row, int32_t col, float v) {
        float* dst = cbase + row * g.ldc + col;
        if (g.add) v += g.add[row * g.ldadd + col];
        if (g.relu) v = v > 0.f ? v : 0.f;
        if (g.accumulate) v += *dst;
        *dst = v;
    };
    const bool inside = m0 + BM <= g.m && __builtin_amdgcn_ballot_w64(bad != 0) == 0;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int32_t col = n0 + wn0 + 32 * j + (lane & 31);
            if (col >= g.n) continue;
            const float bv = g.bias ? g.bias[col] : 0.f;
            const int64_t row0 = m0 + wm0 + 32 * i + 4 * (lane >> 5);
            float* dst = cbase + row0 * g.ldc + col;
            if (inside && plain) {
#pragma unroll
                for (int r = 0; r < 16; ++r) dst[(8 * (r >> 2) + (r & 3)) * g.ldc] = acc[i][j][r] + bv;
            } else if (inside) {
                // (what is added is read before anything is stored, sixteen loads in flight: element by
                // element the aggregate of a GraphSAGE layer cost 33 us on 40,000 rows of 256)
                float v[16], o[16];
                auto load16 = [&](const float* p, int64_t ld) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[r] = p[row0 * ld + col + (8 * (r >> 2) + (r & 3)) * ld];
                };
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] = acc[i][j][r] + bv;
                if (g.add) {
                    load16(g.add, g.ldadd);
#pragma unroll
                    for (int r = 0; r < 16; ++r) v[r] += o[r];
                }
                if (g.relu) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) v[r] = v[r] > 0.f ? v[r] : 0.f;
                }
                if (g.accumulate) {
                    load16(cbase, g.ldc);
#pragma unroll
                    for (int r = 0; r < 16; ++r) v[r] += o[r];
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) dst[(8 * (r >> 2) + (r & 3)) * g.ldc] = v[r];
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int64_t o = 8 * (r >> 2) + (r & 3);
                    if (row0 + o < g.m && !((bad >> ((i * TN + j) * 16 + r)) & 1)) put(row0 + o, col, acc[i][j][r] + bv);
                }
            }
        }
    while (bad) {
        const int e = __ffsll((unsigned long long)bad) - 1;
        bad &= bad - 1;
        const int r = e & 15, j = (e >> 4) % TN, i = (e >> 4) / TN;
        const int32_t col = n0 + wn0 + 32 * j + (lane & 31);
        const int64_t row = m0 + wm0 + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (col >= g.n || row >= g.m) continue;
        float v = 0.f;
        for (int seg = 0; seg < 2; ++seg) {
            const int64_t ke = seg == 0 ? kend0 : (int64_t)g.kseg[1];
            const Operand a = g.a[seg], b = g.b[seg];
            for (int64_t k = seg == 0 ? kbeg : 0; k < ke; ++k)
                v = fmaf(A_KFAST ? a.p[row * a.ld + k] : a.p[k * a.ld + row],
                         B_KFAST ? b.p[col * b.ld + k] : b.p[k * b.ld + col], v);
        }
        put(row, col, v + (g.bias ? g.bias[col] : 0.f));
    }
}

// c[i] += sum_s partial[s * stride + i].  A block covers 64 groups of four consecutive
// elements; its four wavefronts each add a quarter of the splits (ascending, eight loads in
// flight) and the four sums are combined through LDS in wavefront order, so the result does
// not depend on timing.  (One thread per group over all splits left most of the chip idle: a
// 256 x 256 gradient is only 64 such blocks of 256 threads.)
// With `groups` a launch holds the splits of several partitions: block row y sums those of group y,
// the same way, and leaves the sum in group_sum at the group's place (m n floats each); k_add_groups
// then adds the groups to c one after the other, as one launch per partition would.
__global__ __launch_bounds__(256) void k_reduce_partials(const float* __restrict__ partial,
                                                         int32_t splits, int64_t stride,
                                                         float* __restrict__ c, int64_t ldc,
                                                         int32_t m, int32_t n, const TnGroup* __restrict__ groups,
                                                         float* __restrict__ group_sum)
{
    constexpr int U = 8;
    __shared__ float4 sm[4][64];
    const int64_t total = (int64_t)m * n;
    if (groups) {
        const TnGroup q = groups[blockIdx.y];
        partial += (int64_t)q.first * stride;
        splits = q.count;
        group_sum += (int64_t)q.slot * total;
    }
    const int grp = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int64_t i = ((int64_t)blockIdx.x * 64 + grp) * 4;
    const int32_t per = (splits + 3) / 4;
    const int32_t zb = q * per, ze = zb + per < splits ? zb + per : splits;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    if (i < total) {
        const bool full = (i + 3 < total) && (stride % 4 == 0);
        if (full) {
            for (int32_t z0 = zb; z0 < ze; z0 += U) {
                float4 x[U];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    x[u] = z0 + u < ze
                               ? *reinterpret_cast<const float4*>(partial + (int64_t)(z0 + u) * stride + i)
                               : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int u = 0; u < U; ++u) { acc[0] += x[u].x; acc[1] += x[u].y; acc[2] += x[u].z; acc[3] += x[u].w; }
            }
        } else {
            for (int32_t z = zb; z < ze; ++z)
                for (int e = 0; e < 4; ++e)
                    if (i + e < total) acc[e] += partial[(int64_t)z * stride + i + e];
        }
    }
    sm[q][grp] = make_float4(acc[0], acc[1], acc[2], acc[3]);
    __syncthreads();
    if (q != 0 || i >= total) return;
    float4 t = sm[0][grp];
    for (int w = 1; w < 4; ++w) { t.x += sm[w][grp].x; t.y += sm[w][grp].y; t.z += sm[w][grp].z; t.w += sm[w][grp].w; }
    const float out[4] = {t.x, t.y, t.z, t.w};
    for (int e = 0; e < 4; ++e) {
        const int64_t j2 = i + e;
        if (j2 >= total) break;
        if (groups) {
            group_sum[j2] = out[e];
        } else {
            const int64_t r = j2 / n, cc = j2 - r * n;
            c[r * ldc + cc] += out[e];
        }
    }
}

// c[r, j] = (((c[r, j] + sums[0]) + sums[1]) + ...): the groups in order, eight loads in flight
__global__ __launch_bounds__(256) void k_add_groups(const float* __restrict__ sums, int32_t ngroups, int64_t stride,
                                                    float* __restrict__ c, int64_t ldc, int32_t m, int32_t n)
{
    constexpr int U = 8;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)m * n) return;
    const int64_t r = i / n;
    float* dst = c + r * ldc + (i - r * n);
    float v = *dst;
    for (int32_t g0 = 0; g0 < ngroups; g0 += U) {
        float x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = g0 + u < ngroups ? sums[(int64_t)(g0 + u) * stride + i] : 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (g0 + u < ngroups) v += x[u];
    }
    *dst = v;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

template <bool A_KFAST, bool B_KFAST>
void launch_gemm(const GemmArgs& g, int splits, hipStream_t s)
{
    if (g.m <= 0 || g.n <= 0) return;
    // 16-byte loads along k need aligned rows and whole vectors; decided per operand (operands whose m
    // or n index is the contiguous one are read element by element, consecutive lanes side by side)
    bool va = A_KFAST, vb = B_KFAST;
    for (int i = 0; i < 2; ++i) {
        if (g.kseg[i] == 0) continue;
        va = va && aligned16(g.a[i].p) && g.a[i].ld % 4 == 0 && g.kseg[i] % 4 == 0;
        vb = vb && aligned16(g.b[i].p) && g.b[i].ld % 4 == 0 && g.kseg[i] % 4 == 0;
    }
    const bool big_m = g.m > 64, big_n = g.n > 64;
    static const bool xcd_map = [] {
        const char* e = getenv("GNNMI_GEMM_XCD_MAP");
        return !(e && e[0] == '0');
    }();
#define GNN_GEMM(BM, BN, VA, VB)                                                                \
    do {                                                                                        \
        const int64_t mt = (g.m + BM - 1) / BM;                                                 \
        const int32_t nt = (g.n + BN - 1) / BN;                                                 \
        GemmArgs ga = g;                                                                        \
        if (splits == 1 && nt > 1 && xcd_map) {                                                 \
            ga.nt_1d = nt;                                                                      \
            hipLaunchKernelGGL((k_gemm<BM, BN, A_KFAST, B_KFAST, VA, VB>),                      \
                               dim3((unsigned)((mt + 7) / 8 * 8 * nt)), dim3(kThreads), 0, s, ga); \
        } else {                                                                                \
            hipLaunchKernelGGL((k_gemm<BM, BN, A_KFAST, B_KFAST, VA, VB>),                      \
                               dim3((unsigned)mt, (unsigned)nt, (unsigned)splits), dim3(kThreads), 0, s, ga); \
        }                                                                                       \
    } while (0)
    // the last 128-wide column tile would be less than half used: 64-wide tiles waste less
    // (172 columns: 192 computed instead of 256, 0.57 -> 0.55 ms on 1.2 M rows, K = 128)
    const bool tail64 = splits == 1 && (g.n + 63) / 64 * 64 < (g.n + 127) / 128 * 128;
    // 64 x 64 tiles where all of them are resident at once, five to a CU: tiles of 128 x 128 would leave
    // CUs idle or alone with the latency of a stage (256 columns, K = 256, 64 / 128: 3,000 rows 16 / 27 us,
    // 15,600 rows 28 / 31 us, 40,000 rows - 2,504 tiles - 58 / 48 us)
    const bool few = ((g.m + 63) / 64) * ((g.n + 63) / 64) * splits <= 5 * 256;
#define GNN_GEMM_TILE(VA, VB)                                     \
    do {                                                          \
        if (few) GNN_GEMM(64, 64, VA, VB);                        \
        else if (big_m && big_n && tail64) GNN_GEMM(128, 64, VA, VB); \
        else if (big_m && big_n) GNN_GEMM(128, 128, VA, VB);      \
        else if (big_m) GNN_GEMM(128, 64, VA, VB);                \
        else if (big_n) GNN_GEMM(64, 128, VA, VB);                \
        else GNN_GEMM(64, 64, VA, VB);                            \
    } while (0)
    if constexpr (A_KFAST && B_KFAST) {
        if (va && vb) GNN_GEMM_TILE(true, true);
        else if (va) GNN_GEMM_TILE(true, false);
        else if (vb) GNN_GEMM_TILE(false, true);
        else GNN_GEMM_TILE(false, false);
    } else if constexpr (A_KFAST) {
        if (va) GNN_GEMM_TILE(true, false);
        else GNN_GEMM_TILE(false, false);
    } else {
        GNN_GEMM_TILE(false, false);
    }
#undef GNN_GEMM_TILE
#undef GNN_GEMM
}

}  // namespace

void launch_gemm_nn(const GemmSeg* segs, int nseg, float* c, int64_t ldc, int64_t m, int32_t n,
                    const GemmEpilogue& ep, hipStream_t s)
{
    GemmArgs g{};
    for (int i = 0; i < 2; ++i) {
        if (i < nseg) {
            g.a[i] = {segs[i].a, segs[i].lda};
            g.b[i] = {segs[i].b, segs[i].ldb};
            g.kseg[i] = segs[i].k;
        } else {
            g.a[i] = g.a[0];
            g.b[i] = g.b[0];
            g.kseg[i] = 0;
        }
    }
    g.c = c; g.ldc = ldc; g.m = m; g.n = n;
    g.bias = ep.bias; g.relu = ep.relu; g.accumulate = ep.accumulate;
    g.add = ep.add; g.ldadd = ep.ldadd;
    launch_gemm<true, false>(g, 1, s);
}

void launch_gemm_nt(const float* a, int64_t lda, const float* b, int64_t ldb, float* c,
                    int64_t ldc, int64_t m, int32_t n, int32_t k, const GemmEpilogue& ep,
                    hipStream_t s)
{
    GemmArgs g{};
    g.a[0] = g.a[1] = {a, lda};
    g.b[0] = g.b[1] = {b, ldb};
    g.kseg[0] = k; g.kseg[1] = 0;
    g.c = c; g.ldc = ldc; g.m = m; g.n = n;
    g.bias = ep.bias; g.relu = ep.relu; g.accumulate = ep.accumulate;
    g.add = ep.add; g.ldadd = ep.ldadd;
    launch_gemm<true, true>(g, 1, s);
}

void launch_gemm_nt2(const GemmSeg* segs, int nseg, float* c, int64_t ldc, int64_t m, int32_t n,
                     const GemmEpilogue& ep, hipStream_t s)
{
    GemmArgs g{};
    for (int i = 0; i < 2; ++i) {
        const GemmSeg& sg = segs[i < nseg ? i : 0];
        g.a[i] = {sg.a, sg.lda};
        g.b[i] = {sg.b, sg.ldb};
        g.kseg[i] = i < nseg ? sg.k : 0;
    }
    g.c = c; g.ldc = ldc; g.m = m; g.n = n;
    g.bias = ep.bias; g.relu = ep.relu; g.accumulate = ep.accumulate;
    g.add = ep.add; g.ldadd = ep.ldadd;
    launch_gemm<true, true>(g, 1, s);
}

int64_t gemm_tn_chunk(int64_t rows, int32_t m, int32_t n)
{
    const int64_t tiles = (int64_t)((m + 127) / 128) * ((n + 127) / 128);
    int64_t chunk = (rows * tiles / 2048 + BK - 1) / BK * BK;
    chunk = chunk < 128 ? 128 : chunk;
    return chunk > 2048 ? 2048 : chunk;
}

void launch_gemm_tn(const float* a, int64_t lda, const float* b, int64_t ldb, float* c,
                    int64_t ldc, int32_t m, int32_t n, int64_t kdim, int64_t chunk, float* partial,
                    hipStream_t s, const TnParts* parts, bool f32_instruction)
{
    if (kdim <= 0 || m <= 0 || n <= 0) return;
    const int splits = parts ? parts->nchunks : (int)((kdim + chunk - 1) / chunk);
    GemmArgs g{};
    g.a[0] = g.a[1] = {a, lda};
    g.b[0] = g.b[1] = {b, ldb};
    g.kseg[0] = (int32_t)kdim; g.kseg[1] = 0;
    g.c = partial; g.ldc = n; g.m = m; g.n = n;
    g.split_chunk = chunk;
    g.split_stride = (int64_t)m * n;
    g.splits = parts ? parts->chunks : nullptr;
    if (f32_instruction) launch_gemm_f32_tn(a, lda, b, ldb, c, ldc, m, n, kdim, chunk, partial, s, parts);
    else launch_gemm<false, false>(g, splits, s);
    if (parts) {
        float* sums = partial + (int64_t)splits * m * n;
        launch_reduce_groups(partial, (int64_t)m * n, m, n, *parts, sums, s);
        launch_add_groups(sums, parts->nslots, (int64_t)m * n, c, ldc, m, n, s);
    } else {
        launch_reduce_partials(partial, splits, (int64_t)m * n, c, ldc, m, n, s);
    }
}

void launch_reduce_partials(const float* partial, int splits, int64_t stride, float* c, int64_t ldc,
                            int32_t m, int32_t n, hipStream_t s)
{
    int64_t blocks = ((int64_t)m * n + 255) / 256;
    hipLaunchKernelGGL(k_reduce_partials, dim3((unsigned)blocks), dim3(256), 0, s, partial, splits,
                       stride, c, ldc, m, n, (const TnGroup*)nullptr, (float*)nullptr);
}

void launch_reduce_groups(const float* partial, int64_t stride, int32_t m, int32_t n, const TnParts& parts,
                          float* sums, hipStream_t s)
{
    const int64_t blocks = ((int64_t)m * n + 255) / 256;
    if (parts.ngroups <= 0) return;
    hipLaunchKernelGGL(k_reduce_partials, dim3((unsigned)blocks, (unsigned)parts.ngroups), dim3(256), 0, s, partial, 0,
                       stride, (float*)nullptr, 0, m, n, parts.groups, sums);
}

void launch_add_groups(const float* sums, int32_t ngroups, int64_t stride, float* c, int64_t ldc, int32_t m, int32_t n,
                       hipStream_t s)
{
    if (ngroups <= 0) return;
    hipLaunchKernelGGL(k_add_groups, dim3((unsigned)(((int64_t)m * n + 255) / 256)), dim3(256), 0, s, sums, ngroups,
                       stride, c, ldc, m, n);
}

}  // namespace gnnmi
