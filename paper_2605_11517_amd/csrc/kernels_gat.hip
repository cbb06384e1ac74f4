// Kernels of the graph-attention layers (LeakyReLU slope 0.2; Velickovic et al.,
// the model family the paper evaluates next to GCN and GraphSAGE).  A layer transforms first:
// H = A^{l-1} W, s_src = H a_src, s_dst = H a_dst per vertex; a partition then gathers the rows
// of H and the scores s_src of its boundary vertices, computes the attention weight of every
// entry of T_p and aggregates with them (the aggregation kernel of the other models, with the
// attention weights as entry weights).  The backward pass regathers, recomputes the attention
// weights and needs one more edge-wise kernel: the dot product dY[v] . H[u] per entry.
//
// Several heads: the per-vertex scores of all heads of a vertex lie side by side (nh floats per
// vertex, so one fetch of a neighbour's scores serves every head), the per-entry arrays (attention
// weights, edge-wise products) are kept head after head, `hs` floats apart, and the row-wise
// passes take the heads of a row in blocks of up to four.
//
// Row-wise scalar passes: a wavefront takes a range item of short rows - rows of up to 128
// entries four at a time, a group of 16 lanes each, longer ones one after the other with the
// whole wavefront; long rows (more than 512 entries) are cut into the aggregation kernel's
// segments, one wavefront per segment, and combined per row in segment order.  All reductions
// are shuffles and fixed-order sums, so results are reproducible.
#include "gnn_internal.h"

namespace gnnmi {
namespace {

constexpr int kWave = 64;
constexpr int kBlock = 256;
constexpr float kSlope = 0.2f;

__device__ inline float wave_sum(float v)
{
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) v += __shfl_xor(v, m, kWave);
    return v;
}
__device__ inline float wave_max(float v)
{
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) v = fmaxf(v, __shfl_xor(v, m, kWave));
    return v;
}
// BLOCK: every thread of the workgroup calls these the same number of times
template <bool BLOCK> __device__ inline float red_sum(float v, float* sm)
{
    v = wave_sum(v);
    if (!BLOCK) return v;
    __syncthreads();
    if (threadIdx.x % kWave == 0) sm[threadIdx.x / kWave] = v;
    __syncthreads();
    return (sm[0] + sm[1]) + (sm[2] + sm[3]);
}
struct GatRows {
    const int64_t* rp;          // row pointers of the partition's rows (absolute positions)
    const int32_t* col;         // local columns (absolute positions)
    int64_t e0;                 // first absolute position of the partition
    int64_t n_own;
    const float* ssrc_own;      // s_src of the partition's own rows, nh floats per row
    const float* ssrc_bnd;      // s_src of its boundary rows (staged), nh floats per row
    const float* sdst_own;      // nh floats per row
    int32_t nh;                 // heads
    int64_t hs;                 // floats between two heads' per-entry arrays
    // work decomposition
    const int32_t* range_rows;
    int64_t nranges;
    const int32_t* long_row;
    int64_t nlong;
    int32_t segment;            // longer rows are handled segment by segment
    __device__ float ssrc(int32_t c, int32_t h) const
    {
        return c < n_own ? ssrc_own[(int64_t)c * nh + h] : ssrc_bnd[(int64_t)(c - n_own) * nh + h];
    }
};

__device__ inline float lrelu(float x) { return x > 0.f ? x : kSlope * x; }

// head h = blockIdx.y: s_src[r nh + h] = H_h[r,:] . a_src_h, s_dst[r nh + h] = H_h[r,:] . a_dst_h with
// H_h = H + h head_off (rows ld floats apart) and the head's f entries of the attention vectors;
// one wavefront per row and head
__global__ __launch_bounds__(kBlock) void k_gat_scores(const float* __restrict__ H, int32_t ld, int32_t f,
                                                       int64_t rows, const float* __restrict__ a_src,
                                                       const float* __restrict__ a_dst,
                                                       float* __restrict__ ssrc, float* __restrict__ sdst,
                                                       int32_t nh, int64_t head_off)
{
    const int lane = threadIdx.x % kWave;
    const int64_t r = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (r >= rows) return;
    const int32_t hd = blockIdx.y;
    H += hd * head_off;
    a_src += hd * f;
    a_dst += hd * f;
    ssrc += hd;
    sdst += hd;
    float s1 = 0.f, s2 = 0.f;
    for (int j = lane; j < f; j += kWave) {
        const float h = H[r * ld + j];
        s1 += h * a_src[j];
        s2 += h * a_dst[j];
    }
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if (lane == 0) {
        ssrc[r * nh] = s1;
        sdst[r * nh] = s2;
    }
}

// attention weights of one short row (at most kSpmmSegmentMax = 8 x 64 entries):
// att[e - e0] = softmax over the row's entries of LeakyReLU(s_src(col) + s_dst(row)).  Every
// lane keeps its up to eight scores in registers, so the scores are gathered once.
constexpr int kPerLane = kSpmmSegmentMax / kWave;

// The row-wise passes take HB heads of a row at a time (h0 .. h0 + HB - 1, those below nh):
// the scores of the HB heads of a neighbour lie side by side and are fetched together (VEC: as
// one 16-byte vector; needs HB = 4 and nh a multiple of 4), and the HB reductions run beside
// each other instead of one after the other.
// The same for heads lying side by side in rows of nh f floats, f a power of two between 4 and
// 256: one wavefront per row reads the whole row (a 16-byte vector per lane and 256-column block)
// and the f / 4 lanes of a head add up their products.
__global__ __launch_bounds__(kBlock) void k_gat_scores_side(const float* __restrict__ H, int32_t ld, int32_t f,
                                                            int64_t rows, const float* __restrict__ a_src,
                                                            const float* __restrict__ a_dst,
                                                            float* __restrict__ ssrc, float* __restrict__ sdst,
                                                            int32_t nh)
{
    const int lane = threadIdx.x % kWave;
    const int64_t r = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (r >= rows) return;
    const int32_t d = nh * f;
    const int gl = f / 4;                       // lanes per head
    for (int32_t c0 = 0; c0 < d; c0 += 4 * kWave) {
        const int32_t c = c0 + 4 * lane;
        float s1 = 0.f, s2 = 0.f;
        if (c < d) {
            const float4 h = *reinterpret_cast<const float4*>(H + r * ld + c);
            const float4 as = *reinterpret_cast<const float4*>(a_src + c);
            const float4 ad = *reinterpret_cast<const float4*>(a_dst + c);
            s1 = (h.x * as.x + h.y * as.y) + (h.z * as.z + h.w * as.w);
            s2 = (h.x * ad.x + h.y * ad.y) + (h.z * ad.z + h.w * ad.w);
        }
        for (int m = 1; m < gl; m <<= 1) {
            s1 += __shfl_xor(s1, m, kWave);
            s2 += __shfl_xor(s2, m, kWave);
        }
        if (c < d && lane % gl == 0) {
            ssrc[r * nh + c / f] = s1;
            sdst[r * nh + c / f] = s2;
        }
    }
}

template <int HB, bool VEC>
__device__ inline void load_scores(const GatRows& g, int32_t c, int32_t h0, int nhb, float (&out)[HB])
{
    const float* p = c < g.n_own ? g.ssrc_own + (int64_t)c * g.nh + h0
                                 : g.ssrc_bnd + (int64_t)(c - g.n_own) * g.nh + h0;
    if (VEC) {
        static_assert(!VEC || HB == 4, "vector loads take four heads");
        const float4 v = *reinterpret_cast<const float4*>(p);
        out[0] = v.x; out[1 % HB] = v.y; out[2 % HB] = v.z; out[3 % HB] = v.w;
    } else {
#pragma unroll
        for (int b = 0; b < HB; ++b) out[b] = b < nhb ? p[b] : 0.f;
    }
}

template <int HB, bool VEC>
__device__ inline void att_row_wave(const GatRows& g, int32_t row, int32_t h0, float* __restrict__ att_all)
{
    const int t = threadIdx.x % kWave;
    const int nhb = g.nh - h0 < HB ? g.nh - h0 : HB;
    const int64_t eb = g.rp[row], ee = g.rp[row + 1];
    const int niter = (int)((ee - eb + kWave - 1) / kWave);
    float sd[HB], m[HB];
#pragma unroll
    for (int b = 0; b < HB; ++b) {
        sd[b] = b < nhb ? g.sdst_own[(int64_t)row * g.nh + h0 + b] : 0.f;
        m[b] = -INFINITY;
    }
    float x[HB][kPerLane];
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) {
#pragma unroll
        for (int b = 0; b < HB; ++b) x[b][i] = -INFINITY;
        if (i < niter) {
            const int64_t e = eb + t + (int64_t)i * kWave;
            if (e < ee) {
                float sc[HB];
                load_scores<HB, VEC>(g, g.col[e], h0, nhb, sc);
#pragma unroll
                for (int b = 0; b < HB; ++b) x[b][i] = lrelu(sc[b] + sd[b]);
            }
#pragma unroll
            for (int b = 0; b < HB; ++b) m[b] = fmaxf(m[b], x[b][i]);
        }
    }
    float s[HB];
#pragma unroll
    for (int b = 0; b < HB; ++b) {
        m[b] = wave_max(m[b]);
        s[b] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < kPerLane; ++i)
        if (i < niter) {
#pragma unroll
            for (int b = 0; b < HB; ++b) {
                x[b][i] = expf(x[b][i] - m[b]);          // exp(-inf) = 0 for the lanes past the row end
                s[b] += x[b][i];
            }
        }
#pragma unroll
    for (int b = 0; b < HB; ++b) s[b] = 1.f / wave_sum(s[b]);
#pragma unroll
    for (int i = 0; i < kPerLane; ++i)
        if (i < niter) {
            const int64_t e = eb + t + (int64_t)i * kWave;
            if (e < ee) {
#pragma unroll
                for (int b = 0; b < HB; ++b)
                    if (b < nhb) att_all[(h0 + b) * g.hs + (e - g.e0)] = x[b][i] * s[b];
            }
        }
}

// after the edge-wise dot products dal[e] = dY[row] . H[col]: t = sum att dal;
// dpre[e] = att (dal - t) LeakyReLU'(x)  (gradient of the pre-activation score);
// gs_dst[row] = sum of those.  The pairs (att, dpre) of an entry are written side by side for
// all heads, pair[((e - e0) nh + h) 2 + {0, 1}]: the transposed pass fetches an entry's values by
// position, and finds those of every head in one place.
template <int HB, bool VEC>
__device__ inline void bwd_row_wave(const GatRows& g, int32_t row, int32_t h0, const float* __restrict__ att_all,
                                    const float* __restrict__ dal_all, float* __restrict__ pair,
                                    float* __restrict__ gs_dst_own)
{
    static_assert(HB == 1 || HB == 2 || HB == 4, "blocks of one, two or four heads");
    const int t = threadIdx.x % kWave;
    const int nhb = g.nh - h0 < HB ? g.nh - h0 : HB;
    const int64_t eb = g.rp[row], ee = g.rp[row + 1];
    const int niter = (int)((ee - eb + kWave - 1) / kWave);
    float sd[HB], tv[HB];
    unsigned pos[HB];           // bit i: the score of the lane's i-th entry is positive
#pragma unroll
    for (int b = 0; b < HB; ++b) {
        sd[b] = b < nhb ? g.sdst_own[(int64_t)row * g.nh + h0 + b] : 0.f;
        tv[b] = 0.f;
        pos[b] = 0u;
    }
    float a[HB][kPerLane], d[HB][kPerLane];
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) {
#pragma unroll
        for (int b = 0; b < HB; ++b) { a[b][i] = 0.f; d[b][i] = 0.f; }
        if (i < niter) {
            const int64_t e = eb + t + (int64_t)i * kWave;
            if (e < ee) {
                float sc[HB];
                load_scores<HB, VEC && HB == 4>(g, g.col[e], h0, nhb, sc);
#pragma unroll
                for (int b = 0; b < HB; ++b)
                    if (b < nhb) {
                        a[b][i] = att_all[(h0 + b) * g.hs + (e - g.e0)];
                        d[b][i] = dal_all[(h0 + b) * g.hs + (e - g.e0)];
                        if (sc[b] + sd[b] > 0.f) pos[b] |= 1u << i;
                    }
            }
#pragma unroll
            for (int b = 0; b < HB; ++b) tv[b] += a[b][i] * d[b][i];
        }
    }
    float ds[HB];
#pragma unroll
    for (int b = 0; b < HB; ++b) {
        tv[b] = wave_sum(tv[b]);
        ds[b] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < kPerLane; ++i)
        if (i < niter) {
            const int64_t e = eb + t + (int64_t)i * kWave;
            float dp[HB];
#pragma unroll
            for (int b = 0; b < HB; ++b) {
                dp[b] = a[b][i] * (d[b][i] - tv[b]) * ((pos[b] >> i) & 1u ? 1.f : kSlope);
                ds[b] += dp[b];
            }
            if (e < ee) {
                float* q = pair + ((e - g.e0) * g.nh + h0) * 2;
                if (VEC) {          // whole blocks of an even number of heads: 16-byte stores
#pragma unroll
                    for (int b = 0; b + 1 < HB; b += 2)
                        *reinterpret_cast<float4*>(q + 2 * b) = make_float4(a[b][i], dp[b], a[b + 1][i], dp[b + 1]);
                } else {
#pragma unroll
                    for (int b = 0; b < HB; ++b)
                        if (b < nhb) *reinterpret_cast<float2*>(q + 2 * b) = make_float2(a[b][i], dp[b]);
                }
            }
        }
#pragma unroll
    for (int b = 0; b < HB; ++b) {
        ds[b] = wave_sum(ds[b]);
        if (t == 0 && b < nhb) gs_dst_own[(int64_t)row * g.nh + h0 + b] = ds[b];
    }
}

// Rows of at most kGroupRow entries: a group of 16 lanes per row, four rows of the range item
// at a time (a wavefront that walks its rows one after the other waits three dependent memory
// round trips per row - row pointer, columns, scores - with nothing else in flight).  Every lane
// of the wavefront runs the same number of row steps; lanes without a row take an empty one.
constexpr int kGroup = 16;
constexpr int kGroupRow = kGroup * kPerLane;      // 128 entries

template <int HB, bool VEC>
__device__ inline void att_rows_groups(const GatRows& g, int32_t r0, int32_t r1, float* __restrict__ att_all)
{
    const int lane = threadIdx.x % kWave, gl = lane % kGroup, grp = lane / kGroup;
    for (int32_t i0 = r0; i0 < r1; i0 += kWave / kGroup) {
        const int32_t row = i0 + grp;
        int64_t eb = 0, ee = 0;
        if (row < r1) {
            eb = g.rp[row];
            ee = g.rp[row + 1];
            if (ee - eb > (g.segment < kGroupRow ? g.segment : kGroupRow)) ee = eb;   // longer rows: afterwards
        }
        const int niter = (int)((ee - eb + kGroup - 1) / kGroup);
        int32_t cols[kPerLane];
#pragma unroll
        for (int i = 0; i < kPerLane; ++i) {
            const int64_t e = eb + gl + (int64_t)i * kGroup;
            cols[i] = e < ee ? g.col[e] : -1;
        }
        for (int32_t h0 = 0; h0 < g.nh; h0 += HB) {
            const int nhb = g.nh - h0 < HB ? g.nh - h0 : HB;
            float sd[HB], m[HB], sum[HB];
#pragma unroll
            for (int b = 0; b < HB; ++b) {
                sd[b] = (b < nhb && row < r1) ? g.sdst_own[(int64_t)row * g.nh + h0 + b] : 0.f;
                m[b] = -INFINITY;
                sum[b] = 0.f;
            }
            float x[HB][kPerLane];
#pragma unroll
            for (int i = 0; i < kPerLane; ++i) {
#pragma unroll
                for (int b = 0; b < HB; ++b) x[b][i] = -INFINITY;
                if (i < niter && cols[i] >= 0) {
                    float sc[HB];
                    load_scores<HB, VEC>(g, cols[i], h0, nhb, sc);
#pragma unroll
                    for (int b = 0; b < HB; ++b) x[b][i] = lrelu(sc[b] + sd[b]);
                }
#pragma unroll
                for (int b = 0; b < HB; ++b) m[b] = fmaxf(m[b], x[b][i]);
            }
#pragma unroll
            for (int b = 0; b < HB; ++b) {
#pragma unroll
                for (int k = 1; k < kGroup; k <<= 1) m[b] = fmaxf(m[b], __shfl_xor(m[b], k, kWave));
            }
#pragma unroll
            for (int i = 0; i < kPerLane; ++i)
                if (i < niter) {
#pragma unroll
                    for (int b = 0; b < HB; ++b) {
                        x[b][i] = expf(x[b][i] - m[b]);      // exp(-inf) = 0 past the row end
                        sum[b] += x[b][i];
                    }
                }
#pragma unroll
            for (int b = 0; b < HB; ++b) {
#pragma unroll
                for (int k = 1; k < kGroup; k <<= 1) sum[b] += __shfl_xor(sum[b], k, kWave);
                sum[b] = 1.f / sum[b];
            }
#pragma unroll
            for (int i = 0; i < kPerLane; ++i)
                if (i < niter && cols[i] >= 0) {
                    const int64_t e = eb + gl + (int64_t)i * kGroup;
#pragma unroll
                    for (int b = 0; b < HB; ++b)
                        if (b < nhb) att_all[(h0 + b) * g.hs + (e - g.e0)] = x[b][i] * sum[b];
                }
        }
    }
}

// The backward scalars of such rows, the same way (see bwd_row_wave for what is computed).
template <int HB, bool VEC>
__device__ inline void bwd_rows_groups(const GatRows& g, int32_t r0, int32_t r1, const float* __restrict__ att_all,
                                       const float* __restrict__ dal_all, float* __restrict__ pair,
                                       float* __restrict__ gs_dst_own)
{
    const int lane = threadIdx.x % kWave, gl = lane % kGroup, grp = lane / kGroup;
    for (int32_t i0 = r0; i0 < r1; i0 += kWave / kGroup) {
        const int32_t row = i0 + grp;
        int64_t eb = 0, ee = 0;
        if (row < r1) {
            eb = g.rp[row];
            ee = g.rp[row + 1];
            if (ee - eb > (g.segment < kGroupRow ? g.segment : kGroupRow)) ee = eb;   // longer rows: afterwards
        }
        const int niter = (int)((ee - eb + kGroup - 1) / kGroup);
        int32_t cols[kPerLane];
#pragma unroll
        for (int i = 0; i < kPerLane; ++i) {
            const int64_t e = eb + gl + (int64_t)i * kGroup;
            cols[i] = e < ee ? g.col[e] : -1;
        }
        for (int32_t h0 = 0; h0 < g.nh; h0 += HB) {
            const int nhb = g.nh - h0 < HB ? g.nh - h0 : HB;
            float sd[HB], tv[HB], ds[HB];
            unsigned pos[HB];
#pragma unroll
            for (int b = 0; b < HB; ++b) {
                sd[b] = (b < nhb && row < r1) ? g.sdst_own[(int64_t)row * g.nh + h0 + b] : 0.f;
                tv[b] = 0.f;
                ds[b] = 0.f;
                pos[b] = 0u;
            }
            float a[HB][kPerLane], d[HB][kPerLane];
#pragma unroll
            for (int i = 0; i < kPerLane; ++i) {
#pragma unroll
                for (int b = 0; b < HB; ++b) { a[b][i] = 0.f; d[b][i] = 0.f; }
                if (i < niter && cols[i] >= 0) {
                    const int64_t e = eb + gl + (int64_t)i * kGroup;
                    float sc[HB];
                    load_scores<HB, VEC && HB == 4>(g, cols[i], h0, nhb, sc);
#pragma unroll
                    for (int b = 0; b < HB; ++b)
                        if (b < nhb) {
                            a[b][i] = att_all[(h0 + b) * g.hs + (e - g.e0)];
                            d[b][i] = dal_all[(h0 + b) * g.hs + (e - g.e0)];
                            if (sc[b] + sd[b] > 0.f) pos[b] |= 1u << i;
                        }
                }
#pragma unroll
                for (int b = 0; b < HB; ++b) tv[b] += a[b][i] * d[b][i];
            }
#pragma unroll
            for (int b = 0; b < HB; ++b) {
#pragma unroll
                for (int k = 1; k < kGroup; k <<= 1) tv[b] += __shfl_xor(tv[b], k, kWave);
            }
#pragma unroll
            for (int i = 0; i < kPerLane; ++i)
                if (i < niter) {
                    float dp[HB];
#pragma unroll
                    for (int b = 0; b < HB; ++b) {
                        dp[b] = a[b][i] * (d[b][i] - tv[b]) * ((pos[b] >> i) & 1u ? 1.f : kSlope);
                        ds[b] += dp[b];
                    }
                    if (cols[i] >= 0) {
                        const int64_t e = eb + gl + (int64_t)i * kGroup;
                        float* q = pair + ((e - g.e0) * g.nh + h0) * 2;
                        if (VEC) {
#pragma unroll
                            for (int b = 0; b + 1 < HB; b += 2)
                                *reinterpret_cast<float4*>(q + 2 * b) =
                                    make_float4(a[b][i], dp[b], a[b + 1][i], dp[b + 1]);
                        } else {
#pragma unroll
                            for (int b = 0; b < HB; ++b)
                                if (b < nhb) *reinterpret_cast<float2*>(q + 2 * b) = make_float2(a[b][i], dp[b]);
                        }
                    }
                }
#pragma unroll
            for (int b = 0; b < HB; ++b) {
#pragma unroll
                for (int k = 1; k < kGroup; k <<= 1) ds[b] += __shfl_xor(ds[b], k, kWave);
                if (gl == 0 && b < nhb && ee > eb) gs_dst_own[(int64_t)row * g.nh + h0 + b] = ds[b];
            }
        }
    }
}

// MODE 0: attention weights; MODE 1: backward scalars.  One range item of short rows per
// wavefront; long rows are skipped here and handled segment by segment below.
template <int MODE, int HB, bool VEC>
__global__ __launch_bounds__(kBlock) void k_gat_rows(const GatRows g, float* __restrict__ att,
                                                     float* __restrict__ dal, float* __restrict__ pair,
                                                     float* __restrict__ gs_dst_own)
{
    const int64_t item = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (item >= g.nranges) return;
    const int32_t r1 = g.range_rows[item + 1];
    if constexpr (MODE == 0) att_rows_groups<HB, VEC>(g, g.range_rows[item], r1, att);
    else bwd_rows_groups<HB, VEC>(g, g.range_rows[item], r1, att, dal, pair, gs_dst_own);
    for (int32_t row = g.range_rows[item]; row < r1; ++row) {
        const int64_t len = g.rp[row + 1] - g.rp[row];
        if (len > g.segment || len <= kGroupRow) continue;
        for (int32_t h0 = 0; h0 < g.nh; h0 += HB) {
            if constexpr (MODE == 0) att_row_wave<HB, VEC>(g, row, h0, att);
            else bwd_row_wave<HB, VEC>(g, row, h0, att, dal, pair, gs_dst_own);
        }
    }
}

// ---- long rows, segment-parallel --------------------------------------------------------------
// A long row is cut into segments of at most kSpmmSegmentMax entries (the aggregation kernel's work
// items); one wavefront handles one segment with its entries in registers, a second small
// kernel combines the segments of each row in segment order, a third applies the result.
struct GatSegs {
    const int32_t* seg_row;
    const int64_t* seg_begin;
    const int32_t* seg_len;
    int64_t nsegs;
    const int32_t* long_row;
    const int32_t* long_first;
    const int32_t* long_nseg;
    int64_t nlong;
};

// STEP 0: per segment local max m and sum of exp(x - m); att <- exp(x - m)
// STEP 1: att *= factor[segment]
// STEP 2: per segment sum of att * dal
// STEP 3: dpre = att (dal - t[segment]) LeakyReLU'(x) written beside att into `pair` (see
//         bwd_row_wave); per segment sum of those
// Per-entry arrays of head h lie hs floats on, per-segment arrays 2 nsegs (stat) / nsegs (factor)
// floats on.  Steps 0 and 3 take the heads in blocks of HB as the row-wise passes do.
template <int STEP, int HB, bool VEC>
__global__ __launch_bounds__(kBlock) void k_gat_segments(const GatRows g, const GatSegs q,
                                                         float* __restrict__ att_all, float* __restrict__ dal_all,
                                                         float* __restrict__ stat_all,
                                                         const float* __restrict__ factor_all,
                                                         float* __restrict__ pair)
{
    const int t = threadIdx.x % kWave;
    const int64_t sgi = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (sgi >= q.nsegs) return;
    const int32_t row = q.seg_row[sgi];
    const int64_t eb = q.seg_begin[sgi], ee = eb + q.seg_len[sgi];
    if constexpr (STEP == 0) {
        for (int32_t h0 = 0; h0 < g.nh; h0 += HB) {
            const int nhb = g.nh - h0 < HB ? g.nh - h0 : HB;
            float sd[HB], m[HB], sum[HB];
#pragma unroll
            for (int b = 0; b < HB; ++b) {
                sd[b] = b < nhb ? g.sdst_own[(int64_t)row * g.nh + h0 + b] : 0.f;
                m[b] = -INFINITY;
                sum[b] = 0.f;
            }
            float x[HB][kPerLane];
#pragma unroll
            for (int i = 0; i < kPerLane; ++i) {
                const int64_t e = eb + t + (int64_t)i * kWave;
#pragma unroll
                for (int b = 0; b < HB; ++b) x[b][i] = -INFINITY;
                if (e < ee) {
                    float sc[HB];
                    load_scores<HB, VEC>(g, g.col[e], h0, nhb, sc);
#pragma unroll
                    for (int b = 0; b < HB; ++b) x[b][i] = lrelu(sc[b] + sd[b]);
                }
#pragma unroll
                for (int b = 0; b < HB; ++b) m[b] = fmaxf(m[b], x[b][i]);
            }
#pragma unroll
            for (int b = 0; b < HB; ++b) m[b] = wave_max(m[b]);
#pragma unroll
            for (int i = 0; i < kPerLane; ++i) {
                const int64_t e = eb + t + (int64_t)i * kWave;
#pragma unroll
                for (int b = 0; b < HB; ++b) {
                    const float ex = expf(x[b][i] - m[b]);
                    if (e < ee && b < nhb) att_all[(h0 + b) * g.hs + (e - g.e0)] = ex;
                    sum[b] += ex;
                }
            }
#pragma unroll
            for (int b = 0; b < HB; ++b) {
                sum[b] = wave_sum(sum[b]);
                if (t == 0 && b < nhb) {
                    float* stat = stat_all + (int64_t)(h0 + b) * 2 * q.nsegs;
                    stat[2 * sgi] = m[b];
                    stat[2 * sgi + 1] = sum[b];
                }
            }
        }
    } else if constexpr (STEP == 3) {
        static_assert(STEP != 3 || HB == 1 || HB == 2 || HB == 4, "blocks of one, two or four heads");
        for (int32_t h0 = 0; h0 < g.nh; h0 += HB) {
            const int nhb = g.nh - h0 < HB ? g.nh - h0 : HB;
            float sd[HB], tv[HB], ds[HB];
#pragma unroll
            for (int b = 0; b < HB; ++b) {
                sd[b] = b < nhb ? g.sdst_own[(int64_t)row * g.nh + h0 + b] : 0.f;
                tv[b] = b < nhb ? factor_all[(int64_t)(h0 + b) * q.nsegs + sgi] : 0.f;
                ds[b] = 0.f;
            }
#pragma unroll
            for (int i = 0; i < kPerLane; ++i) {
                const int64_t e = eb + t + (int64_t)i * kWave;
                if (e < ee) {
                    float sc[HB], av[HB], dp[HB];
                    load_scores<HB, VEC && HB == 4>(g, g.col[e], h0, nhb, sc);
#pragma unroll
                    for (int b = 0; b < HB; ++b) {
                        av[b] = 0.f; dp[b] = 0.f;
                        if (b < nhb) {
                            av[b] = att_all[(h0 + b) * g.hs + (e - g.e0)];
                            dp[b] = av[b] * (dal_all[(h0 + b) * g.hs + (e - g.e0)] - tv[b]) *
                                    (sc[b] + sd[b] > 0.f ? 1.f : kSlope);
                            ds[b] += dp[b];
                        }
                    }
                    float* qp = pair + ((e - g.e0) * g.nh + h0) * 2;
                    if (VEC) {          // whole blocks of an even number of heads: 16-byte stores
#pragma unroll
                        for (int b = 0; b + 1 < HB; b += 2)
                            *reinterpret_cast<float4*>(qp + 2 * b) = make_float4(av[b], dp[b], av[b + 1], dp[b + 1]);
                    } else {
#pragma unroll
                        for (int b = 0; b < HB; ++b)
                            if (b < nhb) *reinterpret_cast<float2*>(qp + 2 * b) = make_float2(av[b], dp[b]);
                    }
                }
            }
#pragma unroll
            for (int b = 0; b < HB; ++b) {
                ds[b] = wave_sum(ds[b]);
                if (t == 0 && b < nhb) stat_all[(int64_t)(h0 + b) * 2 * q.nsegs + sgi] = ds[b];
            }
        }
    } else {
        for (int32_t h = 0; h < g.nh; ++h) {
            float* __restrict__ att = att_all + h * g.hs;
            if (STEP == 1) {
                const float f = factor_all[(int64_t)h * q.nsegs + sgi];
                for (int64_t e = eb + t; e < ee; e += kWave) att[e - g.e0] *= f;
            } else {
                const float* __restrict__ dal = dal_all + h * g.hs;
                float tv = 0.f;
                for (int64_t e = eb + t; e < ee; e += kWave) tv += att[e - g.e0] * dal[e - g.e0];
                tv = wave_sum(tv);
                if (t == 0) stat_all[(int64_t)h * 2 * q.nsegs + sgi] = tv;
            }
        }
    }
}

// One wavefront per long row, its segments in ascending order, head after head.
// STEP 0: from (m, sum) per segment: factor[segment] = exp(m_seg - M) / S
// STEP 2: factor[segment] = sum of the row's stat (the row's t)
// STEP 3: gs_dst_own[row] = sum of the row's stat
template <int STEP>
__global__ __launch_bounds__(kBlock) void k_gat_combine(const GatSegs q, int32_t nh,
                                                        const float* __restrict__ stat_all,
                                                        float* __restrict__ factor_all,
                                                        float* __restrict__ gs_dst_own)
{
    const int t = threadIdx.x % kWave;
    const int64_t i = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (i >= q.nlong) return;
    const int32_t first = q.long_first[i], ns = q.long_nseg[i];
    for (int32_t h = 0; h < nh; ++h) {
        const float* __restrict__ stat = stat_all + (int64_t)h * 2 * q.nsegs;
        float* __restrict__ factor = factor_all ? factor_all + (int64_t)h * q.nsegs : nullptr;
        if (STEP == 0) {
            float M = -INFINITY;
            for (int32_t j = t; j < ns; j += kWave) M = fmaxf(M, stat[2 * (int64_t)(first + j)]);
            M = wave_max(M);
            float S = 0.f;
            for (int32_t j = t; j < ns; j += kWave)
                S += stat[2 * (int64_t)(first + j) + 1] * expf(stat[2 * (int64_t)(first + j)] - M);
            S = wave_sum(S);
            const float inv = 1.f / S;
            for (int32_t j = t; j < ns; j += kWave) factor[first + j] = expf(stat[2 * (int64_t)(first + j)] - M) * inv;
        } else {
            float v = 0.f;
            for (int32_t j = t; j < ns; j += kWave) v += stat[first + j];
            v = wave_sum(v);
            if (STEP == 2) {
                for (int32_t j = t; j < ns; j += kWave) factor[first + j] = v;
            } else if (t == 0) {
                gs_dst_own[(int64_t)q.long_row[i] * nh + h] = v;
            }
        }
    }
}

// Rows of the transposed operator (the entries of R_p = [own ; boundary] as sources), every head:
// tw_att[h hs + pos - e0] = att of entry tperm[pos] (entry weights of the transposed aggregation)
// and gs_src[(owner row of i) nh + h] += sum over the row of dpre of entry tperm[pos], both read
// from the pairs the backward scalar pass wrote (pair[(entry nh + h) 2 + {0, 1}] = att, dpre: the
// values of all heads of an entry lie in one place, a fetch by position finds them together).
struct GatTRows {
    const int64_t* trp;
    const int32_t* tperm;
    int64_t e0;
    int64_t n_own, base_row;
    const int32_t* bnd;         // library rows of the boundary vertices
    int32_t nh;                 // heads: gs_src holds nh floats per vertex,
    int64_t hs;                 // tw_att one array per head, hs floats apart
    const int32_t* range_rows;
    int64_t nranges;
    int32_t segment;
};
// Sum of the score gradients of four heads h0 .. h0 + 3 (those below h0 + nhb) over the transposed
// entries [eb, ee), by a group of 16 lanes: entries 16 apart per lane, then a shuffle tree.  Every
// pass over transposed rows sums a row, a segment or a piece this way.  The attention weights of
// those entries are written to tw_att on the way.  EVEN: nh is even, two heads' pairs are read as
// one 16-byte vector.
constexpr int kTHeads = 4;
template <bool EVEN>
__device__ inline void trow_sum(const float* __restrict__ pair, const int32_t* __restrict__ tperm, int64_t eb, int64_t ee,
                                int gl, int32_t nh, int32_t h0, int nhb, float* __restrict__ tw_att, int64_t hs,
                                int64_t e0, float (&sum)[kTHeads])
{
    constexpr int GW = kGroup, HB = kTHeads;
#pragma unroll
    for (int b = 0; b < HB; ++b) sum[b] = 0.f;
    for (int64_t e = eb + gl; e < ee; e += GW) {
        const float* q = pair + ((int64_t)tperm[e] * nh + h0) * 2;
        float av[HB], dv[HB];
        if (EVEN) {
#pragma unroll
            for (int b = 0; b < HB; b += 2) {
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                if (b < nhb) v = *reinterpret_cast<const float4*>(q + 2 * b);
                av[b] = v.x; dv[b] = v.y; av[b + 1] = v.z; dv[b + 1] = v.w;
            }
        } else {
#pragma unroll
            for (int b = 0; b < HB; ++b) {
                float2 v = make_float2(0.f, 0.f);
                if (b < nhb) v = *reinterpret_cast<const float2*>(q + 2 * b);
                av[b] = v.x; dv[b] = v.y;
            }
        }
#pragma unroll
        for (int b = 0; b < HB; ++b)
            if (b < nhb) {
                tw_att[(h0 + b) * hs + e - e0] = av[b];
                sum[b] += dv[b];
            }
    }
#pragma unroll
    for (int b = 0; b < HB; ++b)
#pragma unroll
        for (int m = 1; m < GW; m <<= 1) sum[b] += __shfl_xor(sum[b], m, kWave);
}

// Long transposed rows (a hub as a source: up to 10^5 destinations in one partition) are cut
// into the aggregation's segments like the long forward rows: 16 lanes per segment, then one
// wavefront per row adds the segments' sums.  (A workgroup per row walked a hub's entries in a
// hundred dependent steps: 245 us per launch, whatever the heads.)
template <bool EVEN>
__global__ __launch_bounds__(kBlock) void k_gat_tsegs(const GatTRows g, const GatSegs q,
                                                      const float* __restrict__ pair, float* __restrict__ tw_att,
                                                      float* __restrict__ stat)
{
    const int gl = threadIdx.x % kGroup;
    const int64_t sgi = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kGroup;
    if (sgi >= q.nsegs) return;
    const int64_t eb = q.seg_begin[sgi], ee = eb + q.seg_len[sgi];
    for (int32_t h0 = 0; h0 < g.nh; h0 += kTHeads) {
        const int nhb = g.nh - h0 < kTHeads ? g.nh - h0 : kTHeads;
        float sum[kTHeads];
        trow_sum<EVEN>(pair, g.tperm, eb, ee, gl, g.nh, h0, nhb, tw_att, g.hs, g.e0, sum);
#pragma unroll
        for (int b = 0; b < kTHeads; ++b)
            if (gl == 0 && b < nhb) stat[(int64_t)(h0 + b) * q.nsegs + sgi] = sum[b];
    }
}
__global__ __launch_bounds__(kBlock) void k_gat_tcombine(const GatTRows g, const GatSegs q,
                                                         const float* __restrict__ stat, float* __restrict__ gs_src)
{
    const int t = threadIdx.x % kWave;
    const int64_t i = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (i >= q.nlong) return;
    const int32_t first = q.long_first[i], ns = q.long_nseg[i], row = q.long_row[i];
    const int64_t r = row < g.n_own ? g.base_row + row : (int64_t)g.bnd[row - g.n_own];
    for (int32_t h = 0; h < g.nh; ++h) {
        float v = 0.f;
        for (int32_t j = t; j < ns; j += kWave) v += stat[(int64_t)h * q.nsegs + first + j];
        v = wave_sum(v);
        if (t == 0) gs_src[r * g.nh + h] += v;
    }
}
template <bool EVEN>
__global__ __launch_bounds__(kBlock) void k_gat_trows(const GatTRows g, const float* __restrict__ pair,
                                                      float* __restrict__ tw_att, float* __restrict__ gs_src)
{
    // transposed rows are short (a source feeds about ten destinations of a partition): a
    // group of 16 lanes takes a row, four rows of the item at a time, four heads at a time
    const int lane = threadIdx.x % kWave, gl = lane % kGroup, grp = lane / kGroup;
    const int64_t item = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (item >= g.nranges) return;
    const int32_t r1 = g.range_rows[item + 1];
    for (int32_t i = g.range_rows[item] + grp; i < r1; i += kWave / kGroup) {
        const int64_t eb = g.trp[i], ee = g.trp[i + 1];
        if (ee <= eb || ee - eb > g.segment) continue;      // long rows: the other kernels
        const int64_t r = i < g.n_own ? g.base_row + i : (int64_t)g.bnd[i - g.n_own];
        for (int32_t h0 = 0; h0 < g.nh; h0 += kTHeads) {
            const int nhb = g.nh - h0 < kTHeads ? g.nh - h0 : kTHeads;
            float sum[kTHeads];
            trow_sum<EVEN>(pair, g.tperm, eb, ee, gl, g.nh, h0, nhb, tw_att, g.hs, g.e0, sum);
#pragma unroll
            for (int b = 0; b < kTHeads; ++b)
                if (gl == 0 && b < nhb) gs_src[r * g.nh + h0 + b] += sum[b];
        }
    }
}

// The same over the whole graph's transpose (MergedItems): gs_src of a row is the sum over its
// pieces in order, stored once.  A group of 16 lanes takes a row of at most one segment, piece by
// piece, or one unit of a longer row.
template <bool EVEN>
__global__ __launch_bounds__(kBlock) void k_gat_merged_rows(const MergedItems it, const float* __restrict__ pair,
                                                            float* __restrict__ tw_att, float* __restrict__ gs_src,
                                                            int32_t nh, int64_t hs, float* __restrict__ stat)
{
    const int lane = threadIdx.x % kWave, gl = lane % kGroup, grp = lane / kGroup;
    const int64_t item = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kGroup;
    if (item >= it.nunits + it.nrows) return;
    float sum[kTHeads];
    if (item < it.nunits) {
        const int64_t eb = it.unit_begin[item], ee = eb + (it.unit_len[item] & 0xFFFF);
        for (int32_t h0 = 0; h0 < nh; h0 += kTHeads) {
            const int nhb = nh - h0 < kTHeads ? nh - h0 : kTHeads;
            trow_sum<EVEN>(pair, it.perm, eb, ee, gl, nh, h0, nhb, tw_att, hs, 0, sum);
#pragma unroll
            for (int b = 0; b < kTHeads; ++b)
                if (gl == 0 && b < nhb) stat[(int64_t)(h0 + b) * it.nunits + item] = sum[b];
        }
        return;
    }
    const int32_t row = it.rows[item - it.nunits] & 0x7FFFFFFF;
    const int64_t r_end = it.rp[row + 1];
    for (int32_t h0 = 0; h0 < nh; h0 += kTHeads) {
        const int nhb = nh - h0 < kTHeads ? nh - h0 : kTHeads;
        float tot[kTHeads] = {0.f, 0.f, 0.f, 0.f};
        for (int64_t e = it.rp[row]; e < r_end;) {
            int64_t pe = e;
            for (;;) {                                   // end of this piece (the row's last entry ends one)
                const bool end = pe + gl < r_end && it.col[pe + gl] < 0;
                const unsigned ends = (unsigned)(__ballot(end) >> (grp * kGroup)) & 0xFFFFu;
                if (ends) { pe += __ffs((int)ends); break; }
                pe += kGroup;
                if (pe >= r_end) { pe = r_end; break; }
            }
            trow_sum<EVEN>(pair, it.perm, e, pe, gl, nh, h0, nhb, tw_att, hs, 0, sum);
#pragma unroll
            for (int b = 0; b < kTHeads; ++b) tot[b] += sum[b];
            e = pe;
        }
#pragma unroll
        for (int b = 0; b < kTHeads; ++b)
            if (gl == 0 && b < nhb) gs_src[(int64_t)row * nh + h0 + b] = tot[b];
    }
}
// the longer rows from their units: a piece of several units as k_gat_tcombine adds segments
__global__ __launch_bounds__(kBlock) void k_gat_merged_combine(const MergedItems it, const float* __restrict__ stat,
                                                               float* __restrict__ gs_src, int32_t nh)
{
    const int t = threadIdx.x % kWave;
    const int64_t i = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (i >= it.nlong * nh) return;
    const int32_t h = (int32_t)(i % nh);
    const int64_t li = i / nh;
    const int64_t row = it.long_row[li] & 0x7FFFFFFF;
    const int64_t first = it.long_first[li];
    const int32_t nu = it.long_nunits[li];
    const float* st = stat + (int64_t)h * it.nunits + first;
    float tot = 0.f;
    for (int32_t u = 0; u < nu;) {
        // units u .. ue - 1 are one piece
        int32_t ue = u;
        for (;;) {
            const bool end = ue + t < nu && it.unit_len[first + ue + t] < 0;
            const unsigned long long ends = __ballot(end);
            if (ends) { ue += __ffsll((unsigned long long)ends); break; }
            ue += kWave;
            if (ue >= nu) { ue = nu; break; }
        }
        if (ue == u + 1) {
            tot += st[u];
        } else {
            float v = 0.f;
            for (int32_t j = u + t; j < ue; j += kWave) v += st[j];
            tot += wave_sum(v);
        }
        u = ue;
    }
    if (t == 0) gs_src[row * nh + h] = tot;
}

// Edge-wise dot products: dal[e - e0] = dY[row,:] . src(col[e])[:] with src the partition's own
// rows of H or the staged boundary rows.  One wavefront per work item (a segment of a long row
// or a range of short rows); the 64 lanes form 64 / G slots of G lanes, a slot handles one entry
// at a time with NV 16-byte vectors per lane and sums its G partial products with shuffles.
struct GatDotArgs {
    const int64_t* rp;
    const int32_t* col;
    int64_t e0, n_own;
    const float* a_rows;
    const float* b_rows;
    const float* dy;            // [n_own, ld]
    int32_t ld;                 // row stride of H, staging and dy (multiple of 4)
    int32_t d;                  // columns of those rows the products run over (multiple of 4)
    float* dal;
    // nslice > 1: one launch for the heads of a layer whose heads lie side by side: workgroup b
    // takes head b % nslice, i.e. columns [head d, (head + 1) d) of every row and the head's array
    // of products, dal_stride floats on (consecutive workgroups, on different XCDs, read different
    // columns of the same source rows)
    int32_t nslice;
    int64_t dal_stride;
    SpmmItems it;
};
template <int G, int NV>
__device__ inline void dot_entries(const GatDotArgs& g, int32_t row, int64_t eb, int64_t ee, int lane)
{
    constexpr int S = kWave / G;
    constexpr int U = 4;
    const int slot = lane / G, gl = lane % G;
    float4 y[NV];
    int cv[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int c = (v * G + gl) * 4;
        cv[v] = c < g.d ? c : -1;
        y[v] = cv[v] >= 0 ? *reinterpret_cast<const float4*>(g.dy + (int64_t)row * g.ld + c)
                          : make_float4(0.f, 0.f, 0.f, 0.f);
        if (cv[v] < 0) cv[v] = 0;
    }
    if (eb >= ee) return;
    // the column indices of a batch are fetched one batch ahead, so that the row loads of a batch
    // do not wait for an index load first
    int32_t cnext[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t ee_u = eb + u * S + slot;
        cnext[u] = g.col[ee_u < ee ? ee_u : ee - 1];
    }
    for (int64_t e = eb; e < ee; e += S * U) {
        float acc[U];
        const float* src[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t c = cnext[u];
            src[u] = c < g.n_own ? g.a_rows + (int64_t)c * g.ld : g.b_rows + ((int64_t)c - g.n_own) * g.ld;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t ee_u = e + S * U + u * S + slot;
            cnext[u] = g.col[ee_u < ee ? ee_u : ee - 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            acc[u] = 0.f;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const float4 h = *reinterpret_cast<const float4*>(src[u] + cv[v]);
                acc[u] += (h.x * y[v].x + h.y * y[v].y) + (h.z * y[v].z + h.w * y[v].w);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float a = acc[u];
#pragma unroll
            for (int m = 1; m < G; m <<= 1) a += __shfl_xor(a, m, kWave);
            const int64_t ee_u = e + u * S + slot;
            if (gl == 0 && ee_u < ee) g.dal[ee_u - g.e0] = a;
        }
    }
}
template <int G, int NV>
__global__ __launch_bounds__(kBlock) void k_gat_dots(GatDotArgs g)
{
    const int lane = threadIdx.x % kWave;
    unsigned blk = blockIdx.x;
    if (g.nslice > 1) {
        const int64_t hd = blk % (unsigned)g.nslice;
        blk /= (unsigned)g.nslice;
        g.a_rows += hd * g.d;
        g.b_rows += hd * g.d;
        g.dy += hd * g.d;
        g.dal += hd * g.dal_stride;
    }
    const int64_t item = (int64_t)blk * (kBlock / kWave) + threadIdx.x / kWave;
    if (item < g.it.nsegs) {
        const int64_t eb = g.it.seg_begin[item];
        dot_entries<G, NV>(g, g.it.seg_row[item], eb, eb + g.it.seg_len[item], lane);
        return;
    }
    const int64_t ri = item - g.it.nsegs;
    if (ri >= g.it.nranges) return;
    const int32_t r1 = g.it.range_rows[ri + 1];
    for (int32_t row = g.it.range_rows[ri]; row < r1; ++row) {
        const int64_t eb = g.rp[row], ee = g.rp[row + 1];
        if (ee - eb > g.it.segment) continue;
        dot_entries<G, NV>(g, row, eb, ee, lane);
    }
}

// The same for rows of 5 to 16 vectors (a head of eight in a layer of 256: 1.02 -> 0.74 ms on 6 M entries): a slot of G lanes takes an item
// of its own, a segment or a whole short row, the short rows longest first.  Bound by rows in flight; a
// wavefront that walks one row of twenty entries keeps a third of its lanes busy.  Eight entries at a
// time: their partial products are summed across the lanes and transposed in one go (a sum in the order
// of the loop above, entry u ending in lane u), 7 shuffles and one store instead of 24 and 8.
template <int G>
__global__ __launch_bounds__(kBlock) void k_gat_dots_slots(GatDotArgs g)
{
    static_assert(G == 8 || G == 16, "eight entries, eight or sixteen lanes");
    constexpr int S = kWave / G, U = 8;
    const int lane = threadIdx.x % kWave, slot = lane / G, gl = lane % G;
    unsigned blk = blockIdx.x;
    if (g.nslice > 1) {
        const int64_t hd = blk % (unsigned)g.nslice;
        blk /= (unsigned)g.nslice;
        g.a_rows += hd * g.d;
        g.b_rows += hd * g.d;
        g.dy += hd * g.d;
        g.dal += hd * g.dal_stride;
    }
    const int64_t item = ((int64_t)blk * (kBlock / kWave) + threadIdx.x / kWave) * S + slot;
    int64_t eb = 0;
    int32_t len = 0, row = 0;
    if (item < g.it.nsegs) {
        eb = g.it.seg_begin[item];
        len = g.it.seg_len[item];
        row = g.it.seg_row[item];
    } else if (item < g.it.nsegs + g.it.nshort) {
        row = g.it.rows_sorted[item - g.it.nsegs] & 0x7FFFFFFF;
        eb = g.rp[row];
        len = (int32_t)(g.rp[row + 1] - eb);
    }
    int32_t maxlen = len;
#pragma unroll
    for (int m = G; m < kWave; m <<= 1) maxlen = max(maxlen, __shfl_xor(maxlen, m, kWave));
    // lanes past the row's end multiply by zero what they read from column 0
    const bool live = gl * 4 < g.d;
    const int cv = live ? gl * 4 : 0;
    const float4 y = live ? *reinterpret_cast<const float4*>(g.dy + (int64_t)row * g.ld + cv) : make_float4(0.f, 0.f, 0.f, 0.f);
    // a slot that has ended repeats its last entry (no entry at all: row 0), without storing
    auto column = [&](int32_t e) { return len > 0 ? g.col[eb + (e < len ? e : len - 1)] : 0; };
    int32_t next = column(gl % U);
    for (int32_t e0 = 0; e0 < maxlen; e0 += U) {
        const int32_t mine = next;
        float4 h[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t c = __shfl(mine, slot * G + u, kWave);
            const float* src = c < g.n_own ? g.a_rows + (int64_t)c * g.ld : g.b_rows + ((int64_t)c - g.n_own) * g.ld;
            h[u] = *reinterpret_cast<const float4*>(src + cv);
        }
        next = column(e0 + U + gl % U);
        float a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float acc = 0.f;
            acc += (h[u].x * y.x + h[u].y * y.y) + (h[u].z * y.z + h[u].w * y.w);
            a[u] = acc;
        }
#pragma unroll
        for (int m = 1, n = U / 2; m < U; m <<= 1, n >>= 1)
#pragma unroll
            for (int j = 0; j < n; ++j) {
                const bool odd = (gl & m) != 0;
                const float keep = odd ? a[2 * j + 1] : a[2 * j], send = odd ? a[2 * j] : a[2 * j + 1];
                a[j] = keep + __shfl_xor(send, m, kWave);
            }
        if (G == 16) a[0] += __shfl_xor(a[0], 8, kWave);
        if (gl < U && e0 + gl < len) g.dal[eb + e0 + gl - g.e0] = a[0];
    }
}

// gH[r, j] += gs_src[r nh] a_src[j] + gs_dst[r nh] a_dst[j] for the rows of one partition (one
// head: its scores are nh floats apart), and the per-block partial column sums
// sum_r gs_src[r] H[r, j] (first f columns of `partial` rows) and sum_r gs_dst[r] H[r, j] (next f
// columns), 256 rows per block.  Bound by memory: one read of H, one read and write of gH.  A thread
// takes four columns (a 16-byte vector; H and gH have rows of ld floats, a multiple of 4, zeros
// past f) of every (256 / vectors per row)-th row with four rows in flight; the row groups are
// combined through LDS in order.  (One thread per column, one row after the other: 115 us on 9,400
// rows of 256 columns.)  The four columns of a vector belong to one head.
__global__ __launch_bounds__(kBlock) void k_gat_rank1(float* __restrict__ gH, const float* __restrict__ H,
                                                      int32_t ld, int32_t f, int64_t rows,
                                                      const float* __restrict__ gs_src,
                                                      const float* __restrict__ gs_dst,
                                                      const float* __restrict__ a_src,
                                                      const float* __restrict__ a_dst,
                                                      float* __restrict__ partial, int32_t nh, int32_t fh,
                                                      const int2* __restrict__ blk)
{
    constexpr int U = 4;
    __shared__ float4 sm[kBlock][2];
    int64_t r0 = (int64_t)blockIdx.x * 256;
    int64_t r1 = r0 + 256 < rows ? r0 + 256 : rows;
    if (blk) {
        r0 = blk[blockIdx.x].x;
        r1 = blk[blockIdx.x].y;
    }
    const int cw = (f + 3) / 4;
    for (int cc = 0; cc < cw; cc += kBlock) {
        const int cwe = cw - cc < kBlock ? cw - cc : kBlock;
        const int rpp = kBlock / cwe, rsub = threadIdx.x / cwe;
        const int j = 4 * (cc + (int)threadIdx.x % cwe);
        float4 p1 = make_float4(0.f, 0.f, 0.f, 0.f), p2 = p1;
        if (rsub < rpp) {
            float as[4], ad[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                as[e] = j + e < f ? a_src[j + e] : 0.f;
                ad[e] = j + e < f ? a_dst[j + e] : 0.f;
            }
            const int32_t hd = j / fh;
            for (int64_t r = r0 + rsub; r < r1; r += (int64_t)rpp * U) {
                float gs[U], gd[U];
                float4 h[U], g[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int64_t rr = r + (int64_t)u * rpp < r1 ? r + (int64_t)u * rpp : r;
                    gs[u] = gs_src[rr * nh + hd];
                    gd[u] = gs_dst[rr * nh + hd];
                    h[u] = *reinterpret_cast<const float4*>(H + rr * ld + j);
                    g[u] = *reinterpret_cast<const float4*>(gH + rr * ld + j);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int64_t rr = r + (int64_t)u * rpp;
                    if (rr >= r1) break;
                    g[u].x += gs[u] * as[0] + gd[u] * ad[0];
                    g[u].y += gs[u] * as[1] + gd[u] * ad[1];
                    g[u].z += gs[u] * as[2] + gd[u] * ad[2];
                    g[u].w += gs[u] * as[3] + gd[u] * ad[3];
                    *reinterpret_cast<float4*>(gH + rr * ld + j) = g[u];
                    p1.x += gs[u] * h[u].x; p1.y += gs[u] * h[u].y; p1.z += gs[u] * h[u].z; p1.w += gs[u] * h[u].w;
                    p2.x += gd[u] * h[u].x; p2.y += gd[u] * h[u].y; p2.z += gd[u] * h[u].z; p2.w += gd[u] * h[u].w;
                }
            }
        }
        sm[threadIdx.x][0] = p1;
        sm[threadIdx.x][1] = p2;
        __syncthreads();
        if (rsub == 0) {
            for (int q = 1; q < rpp; ++q) {
                const float4 o1 = sm[q * cwe + threadIdx.x][0], o2 = sm[q * cwe + threadIdx.x][1];
                p1.x += o1.x; p1.y += o1.y; p1.z += o1.z; p1.w += o1.w;
                p2.x += o2.x; p2.y += o2.y; p2.z += o2.z; p2.w += o2.w;
            }
            const float s1[4] = {p1.x, p1.y, p1.z, p1.w}, s2[4] = {p2.x, p2.y, p2.z, p2.w};
            float* out = partial + (int64_t)blockIdx.x * 2 * f;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (j + e < f) {
                    out[j + e] = s1[e];
                    out[f + j + e] = s2[e];
                }
        }
        __syncthreads();
    }
}

}  // namespace

void launch_gat_scores(const float* H, int32_t ld, int32_t f, int64_t rows, const float* a_src,
                       const float* a_dst, float* ssrc, float* sdst, int32_t nh, int64_t head_off, hipStream_t s)
{
    if (rows <= 0) return;
    const int64_t blocks = (rows + kBlock / kWave - 1) / (kBlock / kWave);
    const bool aligned = ((reinterpret_cast<uintptr_t>(H) | reinterpret_cast<uintptr_t>(a_src) |
                           reinterpret_cast<uintptr_t>(a_dst)) & 15) == 0 && ld % 4 == 0;
    if (nh > 1 && head_off == f && f >= 4 && f <= 256 && (f & (f - 1)) == 0 && aligned) {
        hipLaunchKernelGGL(k_gat_scores_side, dim3((unsigned)blocks), dim3(kBlock), 0, s, H, ld, f, rows, a_src, a_dst,
                           ssrc, sdst, nh);
        return;
    }
    hipLaunchKernelGGL(k_gat_scores, dim3((unsigned)blocks, (unsigned)nh), dim3(kBlock), 0, s, H, ld, f, rows, a_src,
                       a_dst, ssrc, sdst, nh, head_off);
}

static GatRows make_rows(const GatRowsHost& h)
{
    GatRows g;
    g.rp = h.rp; g.col = h.col; g.e0 = h.e0; g.n_own = h.n_own;
    g.ssrc_own = h.ssrc_own; g.ssrc_bnd = h.ssrc_bnd; g.sdst_own = h.sdst_own;
    g.nh = h.nh; g.hs = h.hs;
    g.range_rows = h.items.range_rows; g.nranges = h.items.nranges;
    g.long_row = h.items.long_row; g.nlong = h.items.nlong;
    g.segment = h.items.segment;
    return g;
}

static GatSegs make_segs(const GatRowsHost& h)
{
    GatSegs q;
    q.seg_row = h.items.seg_row; q.seg_begin = h.items.seg_begin; q.seg_len = h.items.seg_len;
    q.nsegs = h.items.nsegs;
    q.long_row = h.items.long_row; q.long_first = h.items.long_first; q.long_nseg = h.items.long_nseg;
    q.nlong = h.items.nlong;
    return q;
}

// `segwork`: 3 floats per head and segment of the partition's long rows
void launch_gat_attention(const GatRowsHost& h, float* att, float* segwork, hipStream_t s)
{
    const GatRows g = make_rows(h);
    if (g.nranges > 0) {
        const dim3 grid((unsigned)((g.nranges + 3) / 4)), b(kBlock);
        float* none = nullptr;
        if (g.nh == 1) hipLaunchKernelGGL((k_gat_rows<0, 1, false>), grid, b, 0, s, g, att, none, none, none);
        else if (g.nh % 4 == 0) hipLaunchKernelGGL((k_gat_rows<0, 4, true>), grid, b, 0, s, g, att, none, none, none);
        else hipLaunchKernelGGL((k_gat_rows<0, 4, false>), grid, b, 0, s, g, att, none, none, none);
    }
    const GatSegs q = make_segs(h);
    if (q.nsegs > 0 && q.nlong > 0) {
        float* stat = segwork;
        float* factor = segwork + 2 * q.nsegs * g.nh;
        float* none = nullptr;
        const dim3 gs((unsigned)((q.nsegs + 3) / 4)), gl((unsigned)((q.nlong + 3) / 4)), b(kBlock);
        const float* nof = nullptr;
        if (g.nh == 1) hipLaunchKernelGGL((k_gat_segments<0, 1, false>), gs, b, 0, s, g, q, att, none, stat, nof, none);
        else if (g.nh % 4 == 0) hipLaunchKernelGGL((k_gat_segments<0, 4, true>), gs, b, 0, s, g, q, att, none, stat, nof, none);
        else hipLaunchKernelGGL((k_gat_segments<0, 4, false>), gs, b, 0, s, g, q, att, none, stat, nof, none);
        hipLaunchKernelGGL((k_gat_combine<0>), gl, b, 0, s, q, g.nh, (const float*)stat, factor, none);
        hipLaunchKernelGGL((k_gat_segments<1, 1, false>), gs, b, 0, s, g, q, att, none, none, (const float*)factor, none);
    }
}

void launch_gat_bwd_scalars(const GatRowsHost& h, const float* att, const float* dal, float* pair,
                            float* gs_dst_own, float* segwork, hipStream_t s)
{
    const GatRows g = make_rows(h);
    float* a = const_cast<float*>(att);
    float* d = const_cast<float*>(dal);
    if (g.nranges > 0) {
        const dim3 grid((unsigned)((g.nranges + 3) / 4)), b(kBlock);
        if (g.nh == 1) hipLaunchKernelGGL((k_gat_rows<1, 1, false>), grid, b, 0, s, g, a, d, pair, gs_dst_own);
        else if (g.nh % 4 == 0) hipLaunchKernelGGL((k_gat_rows<1, 4, true>), grid, b, 0, s, g, a, d, pair, gs_dst_own);
        else if (g.nh % 2 == 0) hipLaunchKernelGGL((k_gat_rows<1, 2, true>), grid, b, 0, s, g, a, d, pair, gs_dst_own);
        else hipLaunchKernelGGL((k_gat_rows<1, 2, false>), grid, b, 0, s, g, a, d, pair, gs_dst_own);
    }
    const GatSegs q = make_segs(h);
    if (q.nsegs > 0 && q.nlong > 0) {
        float* stat = segwork;
        float* factor = segwork + 2 * q.nsegs * g.nh;
        float* none = nullptr;
        const dim3 gs((unsigned)((q.nsegs + 3) / 4)), gl((unsigned)((q.nlong + 3) / 4)), b(kBlock);
        hipLaunchKernelGGL((k_gat_segments<2, 1, false>), gs, b, 0, s, g, q, a, d, stat, (const float*)nullptr, none);
        hipLaunchKernelGGL((k_gat_combine<2>), gl, b, 0, s, q, g.nh, (const float*)stat, factor, none);
        if (g.nh == 1)
            hipLaunchKernelGGL((k_gat_segments<3, 1, false>), gs, b, 0, s, g, q, a, d, stat, (const float*)factor, pair);
        else if (g.nh % 4 == 0)
            hipLaunchKernelGGL((k_gat_segments<3, 4, true>), gs, b, 0, s, g, q, a, d, stat, (const float*)factor, pair);
        else if (g.nh % 2 == 0)
            hipLaunchKernelGGL((k_gat_segments<3, 2, true>), gs, b, 0, s, g, q, a, d, stat, (const float*)factor, pair);
        else
            hipLaunchKernelGGL((k_gat_segments<3, 2, false>), gs, b, 0, s, g, q, a, d, stat, (const float*)factor, pair);
        hipLaunchKernelGGL((k_gat_combine<3>), gl, b, 0, s, q, g.nh, (const float*)stat, none, gs_dst_own);
    }
}

void launch_gat_transposed(const int64_t* trp, const int32_t* tperm, int64_t e0, int64_t n_own,
                           int64_t base_row, const int32_t* bnd, const SpmmItems& items, const float* pair,
                           float* tw_att, float* gs_src, int32_t nh, int64_t hs, float* segwork, hipStream_t s)
{
    GatTRows g;
    g.trp = trp; g.tperm = tperm; g.e0 = e0; g.n_own = n_own; g.base_row = base_row; g.bnd = bnd;
    g.nh = nh; g.hs = hs;
    g.range_rows = items.range_rows; g.nranges = items.nranges;
    g.segment = items.segment;
    if (g.nranges > 0) {
        const dim3 grid((unsigned)((g.nranges + 3) / 4)), b(kBlock);
        if (nh % 2 == 0) hipLaunchKernelGGL((k_gat_trows<true>), grid, b, 0, s, g, pair, tw_att, gs_src);
        else hipLaunchKernelGGL((k_gat_trows<false>), grid, b, 0, s, g, pair, tw_att, gs_src);
    }
    if (items.nlong > 0 && items.nsegs > 0) {
        GatSegs q;
        q.seg_row = items.seg_row; q.seg_begin = items.seg_begin; q.seg_len = items.seg_len; q.nsegs = items.nsegs;
        q.long_row = items.long_row; q.long_first = items.long_first; q.long_nseg = items.long_nseg;
        q.nlong = items.nlong;
        const dim3 grid((unsigned)((q.nsegs * kGroup + kBlock - 1) / kBlock));
        if (nh % 2 == 0) hipLaunchKernelGGL((k_gat_tsegs<true>), grid, dim3(kBlock), 0, s, g, q, pair, tw_att, segwork);
        else hipLaunchKernelGGL((k_gat_tsegs<false>), grid, dim3(kBlock), 0, s, g, q, pair, tw_att, segwork);
        hipLaunchKernelGGL(k_gat_tcombine, dim3((unsigned)((q.nlong + 3) / 4)), dim3(kBlock), 0, s, g, q,
                           (const float*)segwork, gs_src);
    }
}

void launch_gat_dots(const int64_t* rp, const int32_t* col, int64_t e0, int64_t n_own, const float* a_rows,
                     const float* b_rows, const float* dy, int32_t d, int32_t ld, float* dal, const SpmmItems& items,
                     hipStream_t s, int32_t nslice, int64_t dal_stride)
{
    const int64_t nitems = items.nsegs + items.nranges;
    if (nitems <= 0) return;
    if (nslice < 1) nslice = 1;
    GatDotArgs g;
    g.rp = rp; g.col = col; g.e0 = e0; g.n_own = n_own; g.a_rows = a_rows; g.b_rows = b_rows; g.dy = dy;
    g.ld = ld; g.d = d; g.dal = dal; g.it = items;
    g.nslice = nslice; g.dal_stride = dal_stride;
    const dim3 grid((unsigned)((nitems + 3) / 4 * nslice)), block(kBlock);
    const int vecs = d / 4;
    auto slots = [&](int per_wave) { return dim3((unsigned)((items.nsegs + items.nshort + 4 * per_wave - 1) / (4 * per_wave) * nslice)); };
    if (vecs <= 4) hipLaunchKernelGGL((k_gat_dots<4, 1>), grid, block, 0, s, g);
    else if (vecs <= 8) hipLaunchKernelGGL((k_gat_dots_slots<8>), slots(8), block, 0, s, g);
    else if (vecs <= 16) hipLaunchKernelGGL((k_gat_dots_slots<16>), slots(4), block, 0, s, g);
    else if (vecs <= 32) hipLaunchKernelGGL((k_gat_dots<32, 1>), grid, block, 0, s, g);
    // 1 KB rows: four 16-lane slots with four vectors per lane keep 16 source rows in flight per
    // wavefront and need four shuffle steps per entry (one 64-lane slot: 4 rows, six steps)
    else if (vecs <= 64) hipLaunchKernelGGL((k_gat_dots<16, 4>), grid, block, 0, s, g);
    else if (vecs <= 128) hipLaunchKernelGGL((k_gat_dots<64, 2>), grid, block, 0, s, g);
    else hipLaunchKernelGGL((k_gat_dots<64, 4>), grid, block, 0, s, g);
}

int64_t gat_rank1_partial_floats(int64_t rows, int32_t f) { return ((rows + 255) / 256) * 2 * (int64_t)f; }

void launch_gat_rank1(float* gH, const float* H, int32_t ld, int32_t f, int64_t rows, const float* gs_src,
                      const float* gs_dst, int32_t nh, int32_t fh, const float* a_src, const float* a_dst,
                      float* partial, hipStream_t s, const RowBlocks* rb)
{
    if (rows <= 0) return;
    const dim3 grid((unsigned)(rb ? rb->nblocks : (rows + 255) / 256)), b(kBlock);
    hipLaunchKernelGGL(k_gat_rank1, grid, b, 0, s, gH, H, ld, f, rows, gs_src, gs_dst, a_src, a_dst, partial, nh, fh,
                       rb ? rb->rows : (const int2*)nullptr);
}

void launch_gat_merged(const MergedItems& it, const float* pair, float* tw_att, float* gs_src, int32_t nh, int64_t hs,
                       float* stat, hipStream_t s)
{
    const int64_t items = it.nunits + it.nrows;
    if (items <= 0) return;
    const dim3 grid((unsigned)((items * kGroup + kBlock - 1) / kBlock)), b(kBlock);
    if (nh % 2 == 0) hipLaunchKernelGGL((k_gat_merged_rows<true>), grid, b, 0, s, it, pair, tw_att, gs_src, nh, hs, stat);
    else hipLaunchKernelGGL((k_gat_merged_rows<false>), grid, b, 0, s, it, pair, tw_att, gs_src, nh, hs, stat);
    if (it.nlong > 0)
        hipLaunchKernelGGL(k_gat_merged_combine, dim3((unsigned)((it.nlong * nh + 3) / 4)), b, 0, s, it,
                           (const float*)stat, gs_src, nh);
}

}  // namespace gnnmi
