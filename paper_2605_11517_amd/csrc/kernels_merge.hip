// Set-up kernels of the whole-graph schedule: the transposed operator of the whole graph from the
// per-partition transposes (see MergedItems), and the forward plan in rows of the graph.  They run
// once per gnn_bind; every access is bounded by the arrays' own row pointers.
#include "gnn_internal.h"

namespace gnnmi {
namespace {

constexpr int kBlock = 256;
constexpr int kWave = 64;

__global__ __launch_bounds__(kBlock) void k_merge_count(int64_t nrows, int32_t k, const int64_t* __restrict__ toff,
                                                        const int64_t* __restrict__ off, const int64_t* __restrict__ boff,
                                                        const int32_t* __restrict__ bnd, const int64_t* __restrict__ trp,
                                                        int32_t* __restrict__ cnt, int32_t segment)
{
    const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (j >= nrows) return;
    int32_t lo = 0, hi = k;                       // toff[lo] <= j < toff[hi]
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) / 2;
        if (toff[mid] <= j) lo = mid;
        else hi = mid;
    }
    const int64_t i = j - toff[lo], np = off[lo + 1] - off[lo];
    const int64_t u = i < np ? off[lo] + i : (int64_t)bnd[boff[lo] + i - np];
    const int32_t len = (int32_t)(trp[j + 1] - trp[j]);
    if (len > 0) atomicAdd(&cnt[u], len);         // integers: any order gives the same count
    if (len > segment) atomicOr(&cnt[u], (int32_t)kLongPiece);
}

// one wavefront per row of partition p's transpose
__global__ __launch_bounds__(kBlock) void k_merge_fill(int64_t r0, int64_t np, int64_t nb, const int32_t* __restrict__ bnd,
                                                       const int64_t* __restrict__ trp, const int32_t* __restrict__ tcol,
                                                       const float* __restrict__ tw, const int32_t* __restrict__ tperm,
                                                       int64_t fwd0, const int64_t* __restrict__ rp,
                                                       int64_t* __restrict__ cursor, int32_t* __restrict__ col,
                                                       float* __restrict__ w, int32_t* __restrict__ perm,
                                                       uint8_t* __restrict__ self_first)
{
    const int lane = threadIdx.x % kWave;
    const int64_t i = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (i >= np + nb) return;
    const int64_t u = i < np ? r0 + i : (int64_t)bnd[i - np];
    const int64_t e0 = trp[i], len = trp[i + 1] - e0;
    const int64_t at = cursor[u];
    const bool self = self_first && i < np;
    for (int64_t j = lane; j < len; j += kWave) {
        uint32_t c = (uint32_t)(tcol[e0 + j] + (int32_t)r0);
        if (j == len - 1) c |= kPieceEnd | (self ? kSelfNext : 0u);
        col[at + j] = (int32_t)c;
        if (tw) w[at + j] = tw[e0 + j];
        else perm[at + j] = (int32_t)(fwd0 + tperm[e0 + j]);
    }
    if (lane == 0) {
        cursor[u] = at + len;
        if (self && len == 0) {
            // the self term follows the last piece so far, or comes first
            if (at > rp[u]) col[at - 1] = (int32_t)((uint32_t)col[at - 1] | kSelfNext);
            else self_first[u] = 1;
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_merge_mask_count(int64_t n, const int64_t* __restrict__ rp,
                                                             const int32_t* __restrict__ col,
                                                             const uint8_t* __restrict__ mask, int32_t* __restrict__ cnt,
                                                             int32_t segment)
{
    const int lane = threadIdx.x % kWave;
    const int64_t u = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (u >= n) return;
    const int64_t e1 = rp[u + 1];
    int32_t c = 0, piece = 0;                     // entries kept: of the row, of the piece so far
    bool long_piece = false;
    for (int64_t e = rp[u]; e < e1; e += kWave) {
        const int32_t v = e + lane < e1 ? col[e + lane] : 0;
        const unsigned long long on = __ballot(e + lane < e1 && mask[v & kMergedColumn] != 0);
        unsigned long long ends = __ballot(v < 0);
        c += __popcll(on);
        int from = 0;
        while (ends) {                            // pieces that end in this chunk
            const int at = __ffsll((unsigned long long)ends) - 1;
            ends &= ends - 1;
            const unsigned long long upto = at == 63 ? ~0ull : (1ull << (at + 1)) - 1ull;
            piece += __popcll(on & upto & ~((1ull << from) - 1ull));
            long_piece = long_piece || piece > segment;
            piece = 0;
            from = at + 1;
            if (from == 64) break;
        }
        if (from < 64) piece += __popcll(on & ~((1ull << from) - 1ull));
    }
    if (lane == 0) cnt[u] = c | (long_piece ? (int32_t)kLongPiece : 0);
}

// end of the piece that starts at e (the position after its last entry)
__device__ inline int64_t piece_end(const int32_t* __restrict__ col, int64_t e, int64_t e_end, int lane)
{
    for (int64_t pe = e; pe < e_end; pe += kWave) {
        const int32_t c = pe + lane < e_end ? col[pe + lane] : 0;
        const unsigned long long ends = __ballot(c < 0);
        if (ends) return pe + __ffsll((unsigned long long)ends);
    }
    return e_end;
}

__global__ __launch_bounds__(kBlock) void k_merge_mask_fill(int64_t n, const int64_t* __restrict__ rp,
                                                            const int32_t* __restrict__ col, const float* __restrict__ w,
                                                            const uint8_t* __restrict__ mask,
                                                            const int64_t* __restrict__ out_rp,
                                                            int32_t* __restrict__ out_col, float* __restrict__ out_w,
                                                            const uint8_t* __restrict__ self_in, uint8_t* __restrict__ self_out)
{
    const int lane = threadIdx.x % kWave;
    const int64_t u = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (u >= n) return;
    const int64_t e_end = rp[u + 1];
    int64_t dst = out_rp[u];
    const int64_t dst0 = dst;
    bool first = self_in && self_in[u] != 0;
    uint32_t last = 0;                       // the entry written last, flags included
    for (int64_t e = rp[u]; e < e_end;) {
        const int64_t pe = piece_end(col, e, e_end, lane);
        const bool self = ((uint32_t)col[pe - 1] & kSelfNext) != 0;
        const int64_t piece0 = dst;
        for (int64_t b = e; b < pe; b += kWave) {
            const bool in = b + lane < pe;
            const int32_t c = in ? col[b + lane] & kMergedColumn : 0;
            const bool on = in && mask[c] != 0;
            const unsigned long long kept = __ballot(on);
            if (!kept) continue;
            if (on) {
                const int64_t at = dst + __popcll(kept & ((1ull << lane) - 1ull));
                out_col[at] = c;
                out_w[at] = w[b + lane];
            }
            dst += __popcll(kept);
            last = (uint32_t)__shfl(c, 63 - __clzll((long long)kept), kWave);
        }
        if (dst > piece0) last |= kPieceEnd;
        if (self) {
            if (dst > dst0) last |= kSelfNext;
            else first = true;
        }
        // (written again with its flags by one lane: stores of a wavefront keep their order)
        if (lane == 0 && dst > dst0 && (dst > piece0 || self)) out_col[dst - 1] = (int32_t)last;
        e = pe;
    }
    if (lane == 0 && self_out) self_out[u] = first ? 1 : 0;
}

__global__ __launch_bounds__(kBlock) void k_merge_units(int64_t nlong, const int32_t* __restrict__ long_row,
                                                        const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                        int32_t segment, int32_t* __restrict__ nunits,
                                                        const int32_t* __restrict__ first, int64_t* __restrict__ begin,
                                                        int32_t* __restrict__ len)
{
    const int lane = threadIdx.x % kWave;
    const int64_t i = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (i >= nlong) return;
    const int32_t u = long_row[i] & 0x7FFFFFFF;
    const int64_t e_end = rp[u + 1];
    int32_t total = 0;
    for (int64_t e = rp[u]; e < e_end;) {
        const int64_t pe = piece_end(col, e, e_end, lane);
        const int32_t segs = (int32_t)((pe - e + segment - 1) / segment);
        if (begin) {
            const uint32_t self = (uint32_t)col[pe - 1] & kSelfNext;
            for (int32_t s = lane; s < segs; s += kWave) {
                const int64_t b = e + (int64_t)s * segment;
                const uint32_t l = (uint32_t)(pe - b < segment ? pe - b : segment);
                begin[first[i] + total + s] = b;
                len[first[i] + total + s] = (int32_t)(l | (s == segs - 1 ? (kPieceEnd | self) : 0u));
            }
        }
        total += segs;
        e = pe;
    }
    if (!begin && lane == 0) nunits[i] = total;
}

__global__ __launch_bounds__(kBlock) void k_merge_mark(int32_t* __restrict__ list, int64_t count,
                                                       const uint8_t* __restrict__ self_first)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < count && self_first[list[i]]) list[i] = (int32_t)((uint32_t)list[i] | 0x80000000u);
}

__global__ __launch_bounds__(kBlock) void k_offset_copy(const int32_t* __restrict__ src, int32_t* __restrict__ dst,
                                                        int64_t count, int32_t add)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < count) dst[i] = src[i] + add;
}

__global__ __launch_bounds__(kBlock) void k_staged_columns(const int32_t* __restrict__ lcol, int32_t* __restrict__ wcol,
                                                           int64_t count, int32_t n_own, int32_t base, int32_t other)
{
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= count) return;
    const int32_t c = lcol[e];
    wcol[e] = c < n_own ? base + c : other + (c - n_own);
}

dim3 per_thread(int64_t n) { return dim3((unsigned)((n + kBlock - 1) / kBlock)); }
dim3 per_wave(int64_t n) { return dim3((unsigned)((n + kBlock / kWave - 1) / (kBlock / kWave))); }

}  // namespace

void launch_merge_count(int64_t nrows, int32_t k, const int64_t* toff, const int64_t* off, const int64_t* boff,
                        const int32_t* bnd, const int64_t* trp, int32_t* cnt, int32_t segment, hipStream_t s)
{
    if (nrows > 0)
        hipLaunchKernelGGL(k_merge_count, per_thread(nrows), dim3(kBlock), 0, s, nrows, k, toff, off, boff, bnd, trp, cnt,
                           segment);
}

void launch_merge_fill(int64_t r0, int64_t np, int64_t nb, const int32_t* bnd, const int64_t* trp, const int32_t* tcol,
                       const float* tw, const int32_t* tperm, int64_t e0, const int64_t* rp, int64_t* cursor, int32_t* col,
                       float* w, int32_t* perm, uint8_t* self_first, hipStream_t s)
{
    if (np + nb > 0)
        hipLaunchKernelGGL(k_merge_fill, per_wave(np + nb), dim3(kBlock), 0, s, r0, np, nb, bnd, trp, tcol, tw, tperm, e0, rp,
                           cursor, col, w, perm, self_first);
}

void launch_merge_mask_count(int64_t n, const int64_t* rp, const int32_t* col, const uint8_t* mask, int32_t* cnt,
                             int32_t segment, hipStream_t s)
{
    hipLaunchKernelGGL(k_merge_mask_count, per_wave(n), dim3(kBlock), 0, s, n, rp, col, mask, cnt, segment);
}

void launch_merge_mask_fill(int64_t n, const int64_t* rp, const int32_t* col, const float* w, const uint8_t* mask,
                            const int64_t* out_rp, int32_t* out_col, float* out_w, const uint8_t* self_in,
                            uint8_t* self_out, hipStream_t s)
{
    hipLaunchKernelGGL(k_merge_mask_fill, per_wave(n), dim3(kBlock), 0, s, n, rp, col, w, mask, out_rp, out_col, out_w,
                       self_in, self_out);
}

void launch_merge_units(int64_t nlong, const int32_t* long_row, const int64_t* rp, const int32_t* col, int32_t segment,
                        int32_t* nunits, const int32_t* first, int64_t* begin, int32_t* len, hipStream_t s)
{
    if (nlong > 0)
        hipLaunchKernelGGL(k_merge_units, per_wave(nlong), dim3(kBlock), 0, s, nlong, long_row, rp, col, segment, nunits,
                           first, begin, len);
}

void launch_merge_mark(int32_t* list, int64_t count, const uint8_t* self_first, hipStream_t s)
{
    if (count > 0) hipLaunchKernelGGL(k_merge_mark, per_thread(count), dim3(kBlock), 0, s, list, count, self_first);
}

void launch_offset_copy(const int32_t* src, int32_t* dst, int64_t count, int32_t add, hipStream_t s)
{
    if (count > 0) hipLaunchKernelGGL(k_offset_copy, per_thread(count), dim3(kBlock), 0, s, src, dst, count, add);
}

void launch_staged_columns(const int32_t* lcol, int32_t* wcol, int64_t count, int64_t n_own, int64_t base, int64_t other,
                           hipStream_t s)
{
    if (count > 0)
        hipLaunchKernelGGL(k_staged_columns, per_thread(count), dim3(kBlock), 0, s, lcol, wcol, count, (int32_t)n_own,
                           (int32_t)base, (int32_t)other);
}

}  // namespace gnnmi
