// Whole-graph schedule of the resident epoch.
//
// The paper walks a layer partition by partition because a partition is what fits the device.  Where
// the whole graph's intermediates fit, one launch per step of a layer does the work of k launches:
// a partition of a few thousand rows neither fills 256 CUs nor outlasts the latency of one launch
// (GraphSAGE 100-256-256-47 on 40,000 vertices in 8 partitions: 369 kernels per epoch, none with
// more than 80 workgroups).  The schedule is the resident one on a second context with one
// partition, the graph, that shares every buffer; what differs is kept in tables and in the
// transposed operator, so that every sum is taken in the order of the partition-by-partition
// schedule and results are its bits:
//   - weight gradients are split and summed partition by partition (TnParts), as are the column
//     sums of the bias gradients and the loss (RowBlocks);
//   - the transposed aggregation runs over the whole graph's transpose (MergedItems), whose rows
//     hold the partitions' contributions one after the other;
//   - boundary rows, where they pass through staging, lie there side by side for all partitions.
// The per-partition entry points, the streaming schedule and profiled epochs that gather through
// staging are not touched.
#include <cstdlib>
#include <new>

#include "gnn_ctx.h"

namespace gnnmi {

namespace {

// Device memory the schedule may add to the workspace and staging of the partition-by-partition one.
constexpr int64_t kWholeLimitBytes = (int64_t)40 << 30;

void free_merged(DevMeta::Merged& m)
{
    for (void* p : {(void*)m.rp, (void*)m.col, (void*)m.w, (void*)m.rows, (void*)m.unit_begin, (void*)m.unit_len,
                    (void*)m.long_row, (void*)m.long_first, (void*)m.long_nunits, (void*)m.partial, (void*)m.self_first, (void*)m.perm})
        if (p) (void)hipFree(p);
    m = DevMeta::Merged{};
}

void free_tables(WholeTables& t)
{
    if (t.rb.rows) (void)hipFree((void*)t.rb.rows);
    if (t.rb.groups) (void)hipFree((void*)t.rb.groups);
    if (t.rb.loss_rows) (void)hipFree((void*)t.rb.loss_rows);
    for (auto& kv : t.splits)
        for (TnParts* p : {&kv.second.wide, &kv.second.narrow}) {
            if (p->chunks) (void)hipFree((void*)p->chunks);
            if (p->groups) (void)hipFree((void*)p->groups);
        }
    t = WholeTables{};
}

// the inner context's own device arrays (the rest of its DevMeta belongs to the outer one)
void free_inner(gnn_ctx* w)
{
    free_merged(w->D.merged);
    free_merged(w->D.merged_masked);
    DevMeta::Plan& f = w->D.fwd;
    for (void* p : {(void*)f.range_rows, (void*)f.seg_row, (void*)f.long_row, (void*)f.long_first, (void*)f.rows_sorted,
                    (void*)w->D.lcol})
        if (p) (void)hipFree(p);
    free_tables(w->tables);
    w->D = DevMeta{};
    w->bound = false;
}

struct Fail {};
void check(hipError_t e)
{
    if (e != hipSuccess) {
        (void)hipGetLastError();
        throw Fail{};
    }
}

template <typename T>
T* device_array(int64_t count)
{
    T* p = nullptr;
    check(hipMalloc((void**)&p, (size_t)std::max<int64_t>(1, count) * sizeof(T)));
    return p;
}
template <typename T>
T* to_device(const std::vector<T>& v)
{
    T* p = device_array<T>((int64_t)v.size());
    if (!v.empty()) {
        const hipError_t e = hipMemcpy(p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            (void)hipFree(p);
            check(e);
        }
    }
    return p;
}
// device memory of a build step, freed when the step ends
struct Temp {
    std::vector<void*> ptrs;
    template <typename T> T* keep(T* p) { ptrs.push_back((void*)p); return p; }
    ~Temp() { for (void* p : ptrs) (void)hipFree(p); }
};

// the forward plan of all partitions with rows, segments and ranges numbered through
void build_forward_plan(const gnn_ctx* c, gnn_ctx* w)
{
    const HostMeta::Plan& H = c->M.plan_fwd;
    const DevMeta::Plan& P = c->D.fwd;
    DevMeta::Plan& Q = w->D.fwd;
    const int32_t k = c->M.k;
    Q.range_rows = device_array<int32_t>(H.range_off[(size_t)k]);
    Q.rows_sorted = device_array<int32_t>(H.rows_off[(size_t)k]);
    Q.long_row = device_array<int32_t>(H.long_off[(size_t)k]);
    Q.long_first = device_array<int32_t>(H.long_off[(size_t)k]);
    Q.seg_row = device_array<int32_t>(H.seg_off[(size_t)k]);
    for (int32_t p = 0; p < k; ++p) {
        const int32_t r0 = (int32_t)c->M.off[(size_t)p];
        auto copy = [&](const int32_t* src, int32_t* dst, const std::vector<int64_t>& o, int32_t add) {
            launch_offset_copy(src + o[(size_t)p], dst + o[(size_t)p], o[(size_t)p + 1] - o[(size_t)p], add, nullptr);
        };
        copy(P.range_rows, Q.range_rows, H.range_off, r0);
        copy(P.rows_sorted, Q.rows_sorted, H.rows_off, r0);
        copy(P.long_row, Q.long_row, H.long_off, r0);
        copy(P.long_first, Q.long_first, H.long_off, (int32_t)H.seg_off[(size_t)p]);
        copy(P.seg_row, Q.seg_row, H.seg_off, r0);
    }
    // (shared: the segments' absolute positions and lengths, the long rows' segment counts)
    Q.seg_begin = P.seg_begin;
    Q.seg_len = P.seg_len;
    Q.long_nseg = P.long_nseg;
    check(hipGetLastError());
}

void build_staged_columns(const gnn_ctx* c, gnn_ctx* w)
{
    if (w->D.lcol || c->M.lcol.empty()) return;
    const HostMeta& M = c->M;
    w->D.lcol = device_array<int32_t>((int64_t)M.lcol.size());
    for (int32_t p = 0; p < M.k; ++p) {
        const int64_t r0 = M.off[(size_t)p], r1 = M.off[(size_t)p + 1];
        const int64_t e0 = M.rp[(size_t)r0], e1 = M.rp[(size_t)r1];
        launch_staged_columns(c->D.lcol + e0, w->D.lcol + e0, e1 - e0, r1 - r0, r0, M.n + M.boff[(size_t)p], nullptr);
    }
    check(hipGetLastError());
}

void build_tables(const gnn_ctx* c, gnn_ctx* w)
{
    const HostMeta& M = c->M;
    const int32_t k = M.k;
    WholeTables& T = w->tables;
    std::vector<int2> rows, groups, loss;
    std::vector<int32_t> first((size_t)k), count((size_t)k);
    for (int32_t p = 0; p < k; ++p) {
        const int64_t r0 = M.off[(size_t)p], r1 = M.off[(size_t)p + 1];
        first[(size_t)p] = (int32_t)rows.size();
        for (int64_t r = r0; r < r1; r += act_rows_per_block())
            rows.push_back(make_int2((int)r, (int)std::min<int64_t>(r1, r + act_rows_per_block())));
        count[(size_t)p] = (int32_t)rows.size() - first[(size_t)p];
        for (int64_t r = r0; r < r1; r += loss_rows_per_block())
            loss.push_back(make_int2((int)r, (int)std::min<int64_t>(r1, r + loss_rows_per_block())));
    }
    for (int32_t t = 0; t < k; ++t) {
        const int32_t p = M.sched[(size_t)t];
        if (count[(size_t)p] > 0) groups.push_back(make_int2(first[(size_t)p], count[(size_t)p]));
    }
    T.rb.nblocks = (int64_t)rows.size();
    T.rb.ngroups = (int32_t)groups.size();
    T.rb.nloss = (int64_t)loss.size();
    T.rb.rows = to_device(rows);
    T.rb.groups = to_device(groups);
    T.rb.loss_rows = to_device(loss);
    auto add_split = [&](int32_t m, int32_t n, int64_t lda, int64_t ldb) {
        const int64_t rows_g = c->grad_rows(), chunk = gemm_tn_chunk(rows_g, m, n);
        const int64_t wide = c->bf16() && gemm_bf16_tn_wide_ok(rows_g, m, n, lda, ldb)
                                 ? gemm_bf16_tn_wide_chunk(rows_g, m, n) : 0;
        if (T.splits.count({wide, chunk})) return;
        std::vector<int2> cw, cn;
        std::vector<TnGroup> gw, gn;
        int32_t slot = 0;
        auto cut = [](std::vector<int2>& cs, std::vector<TnGroup>& gs, int64_t a, int64_t b, int64_t step, int32_t& sl) {
            if (b <= a) return;
            TnGroup g{(int32_t)cs.size(), 0, sl++};
            for (int64_t r = a; r < b; r += step) cs.push_back(make_int2((int)r, (int)std::min(b, r + step)));
            g.count = (int32_t)cs.size() - g.first;
            gs.push_back(g);
        };
        for (int32_t t = 0; t < k; ++t) {
            const int32_t p = M.sched[(size_t)t];
            int64_t r0 = M.off[(size_t)p];
            const int64_t r1 = M.off[(size_t)p + 1];
            if (wide) {
                const int64_t whole_stages = r0 + (r1 - r0) / 64 * 64;
                cut(cw, gw, r0, whole_stages, wide, slot);
                r0 = whole_stages;
            }
            cut(cn, gn, r0, r1, chunk, slot);
        }
        WholeTables::Split& S = T.splits[{wide, chunk}];
        auto fill = [&](TnParts& P, const std::vector<int2>& cs, const std::vector<TnGroup>& gs) {
            P.nchunks = (int32_t)cs.size();
            P.ngroups = (int32_t)gs.size();
            P.nslots = slot;
            P.chunks = to_device(cs);
            P.groups = to_device(gs);
        };
        fill(S.wide, cw, gw);
        fill(S.narrow, cn, gn);
    };
    for (int32_t l = 1; l <= c->L; ++l) {
        const int32_t din = c->dims[(size_t)l - 1], dout = c->dims[(size_t)l];
        add_split(din, dout, din, dout);
        if (c->nheads(l) > 1) add_split(din, c->head_cols(l), din, c->head_cols(l));
    }
}

// Longest row of the merged operator that one slot sums.  A longer row's pieces are summed on their own
// and written and read once more, a row of d floats per piece: with 64 partitions a row of 300 entries
// is 60 pieces, and its sums are a fifth of what it fetches.  But a slot walks a row in dependent
// steps, which must not outlast the launch.  Transposed pass + combining in ms, rows cut above
// 64 / 128 / 256 / 512 / 1024 entries:
//   50 k entries (GCN 64-64-16)                         0.027 / 0.036 / 0.053
//   6.5 M entries (1024 bfloat16 columns)               2.51 / 2.45 / 2.15 / 2.11 / 2.12
//   52 M entries, 64 partitions (128 and 172 columns)   7.74 / 6.87 / 6.13 / 5.75 / 5.69
//   66 M entries (256 columns)                          9.64 / 8.88 / 8.63 / 8.42 / 8.23
int64_t merged_row_max(int64_t entries, int32_t segment)
{
    const int64_t most = entries < 2000000 ? 64 : entries < 8000000 ? 256 : entries < 30000000 ? 512 : 1024;
    return std::max<int64_t>(segment, most);
}

// Row pointers and work lists of a merged operator from the entries per row (device).
void finish_rows(const gnn_ctx* c, DevMeta::Merged& m, const int32_t* cnt_dev)
{
    const int64_t n = c->M.n;
    std::vector<int32_t> cnt((size_t)n);
    check(hipMemcpy(cnt.data(), cnt_dev, (size_t)n * sizeof(int32_t), hipMemcpyDeviceToHost));
    std::vector<int64_t> rp((size_t)n + 1);
    rp[0] = 0;
    for (int64_t u = 0; u < n; ++u) rp[(size_t)u + 1] = rp[(size_t)u] + (cnt[(size_t)u] & 0x7FFFFFFF);
    // (a row with a long piece is negative here: long whatever its length)
    const int32_t most = (int32_t)merged_row_max(rp[(size_t)n], c->M.segment);
    std::vector<int64_t> bucket((size_t)most + 2, 0);
    std::vector<int32_t> longs;
    for (int64_t u = 0; u < n; ++u) {
        const int32_t d = cnt[(size_t)u];
        if (d < 0 || d > most) longs.push_back((int32_t)u);
        else bucket[(size_t)(most - d) + 1]++;
    }
    for (size_t i = 1; i < bucket.size(); ++i) bucket[i] += bucket[i - 1];
    std::vector<int32_t> rows((size_t)(n - (int64_t)longs.size()));
    for (int64_t u = 0; u < n; ++u) {
        const int32_t d = cnt[(size_t)u];
        if (d >= 0 && d <= most) rows[(size_t)bucket[(size_t)(most - d)]++] = (int32_t)u;
    }
    m.entries = rp[(size_t)n];
    m.avg_len = (float)m.entries / (float)std::max<int64_t>(1, n);
    m.nrows = (int64_t)rows.size();
    m.nlong = (int64_t)longs.size();
    m.rp = to_device(rp);
    m.rows = to_device(rows);
    m.long_row = to_device(longs);
    m.col = device_array<int32_t>(m.entries);
    if (c->model == GNN_GAT) m.perm = device_array<int32_t>(m.entries);
    else m.w = device_array<float>(m.entries);
}

// Units of the long rows, room for their sums, and the self-term marks of both lists.
void finish_units(const gnn_ctx* c, DevMeta::Merged& m, int32_t width)
{
    m.long_nunits = device_array<int32_t>(m.nlong);
    launch_merge_units(m.nlong, m.long_row, m.rp, m.col, c->M.segment, m.long_nunits, nullptr, nullptr, nullptr, nullptr);
    std::vector<int32_t> cnt((size_t)m.nlong), first((size_t)m.nlong);
    check(hipGetLastError());
    if (m.nlong > 0)
        check(hipMemcpy(cnt.data(), m.long_nunits, (size_t)m.nlong * sizeof(int32_t), hipMemcpyDeviceToHost));
    int64_t total = 0;
    for (size_t i = 0; i < cnt.size(); ++i) {
        first[i] = (int32_t)total;
        total += cnt[i];
    }
    if (total >= ((int64_t)1 << 31)) throw Fail{};
    m.nunits = total;
    m.long_first = to_device(first);
    m.unit_begin = device_array<int64_t>(total);
    m.unit_len = device_array<int32_t>(total);
    m.partial = device_array<float>(total * width);
    launch_merge_units(m.nlong, m.long_row, m.rp, m.col, c->M.segment, m.long_nunits, m.long_first, m.unit_begin,
                       m.unit_len, nullptr);
    if (m.self_first) {
        launch_merge_mark(m.rows, m.nrows, m.self_first, nullptr);
        launch_merge_mark(m.long_row, m.nlong, m.self_first, nullptr);
    }
    check(hipGetLastError());
}

// widest row any transposed aggregation moves
int32_t transposed_width(const gnn_ctx* c)
{
    int32_t d = 4;
    for (int32_t l = 1; l <= c->L; ++l) d = std::max(d, c->transform_first(l) ? c->hrow(l) : c->dims[(size_t)l - 1]);
    return d;
}

void build_merged(const gnn_ctx* c, DevMeta::Merged& m)
{
    const HostMeta& M = c->M;
    const int64_t n = M.n;
    Temp tmp;
    int32_t* cnt = tmp.keep(device_array<int32_t>(n));
    launch_fill_zero(cnt, n * (int64_t)sizeof(int32_t), nullptr);
    const int64_t* toff = tmp.keep(to_device(M.toff));
    const int64_t* off = tmp.keep(to_device(M.off));
    const int64_t* boff = tmp.keep(to_device(M.boff));
    launch_merge_count(M.toff[(size_t)M.k], M.k, toff, off, boff, c->D.bnd, c->D.trp, cnt, c->M.segment, nullptr);
    check(hipGetLastError());
    finish_rows(c, m, cnt);
    int64_t* cursor = tmp.keep(device_array<int64_t>(n));
    check(hipMemcpy(cursor, m.rp, (size_t)n * sizeof(int64_t), hipMemcpyDeviceToDevice));
    if (c->model == GNN_SAGE_MEAN) {
        m.self_first = device_array<uint8_t>(n);
        launch_fill_zero(m.self_first, n, nullptr);
    }
    for (int32_t t = 0; t < M.k; ++t) {
        const int32_t p = M.sched[(size_t)t];
        const int64_t r0 = M.off[(size_t)p], np = M.off[(size_t)p + 1] - r0;
        launch_merge_fill(r0, np, M.boff[(size_t)p + 1] - M.boff[(size_t)p], c->D.bnd + M.boff[(size_t)p],
                          c->D.trp + M.toff[(size_t)p], c->D.tcol, c->D.tw, c->D.tperm, M.rp[(size_t)r0], m.rp, cursor,
                          m.col, m.w, m.perm, m.self_first, nullptr);
    }
    check(hipGetLastError());
    finish_units(c, m, transposed_width(c));
    check(hipDeviceSynchronize());
    m.ready = true;
}

void build_merged_masked(const gnn_ctx* c, const DevMeta::Merged& full, DevMeta::Merged& m)
{
    const int64_t n = c->M.n;
    Temp tmp;
    int32_t* cnt = tmp.keep(device_array<int32_t>(n));
    launch_merge_mask_count(n, full.rp, full.col, c->mask, cnt, c->M.segment, nullptr);
    check(hipGetLastError());
    finish_rows(c, m, cnt);
    if (full.self_first) m.self_first = device_array<uint8_t>(n);
    launch_merge_mask_fill(n, full.rp, full.col, full.w, c->mask, m.rp, m.col, m.w, full.self_first, m.self_first, nullptr);
    check(hipGetLastError());
    const int32_t width = c->transform_first(c->L) ? c->padded(c->L) : c->dims[(size_t)c->L - 1];
    finish_units(c, m, width);
    check(hipDeviceSynchronize());
    m.ready = true;
}

bool wanted(const gnn_ctx* c)
{
    // GNNMI_WHOLE=0: partition by partition (for measurements and tests; read per call)
    const char* e = std::getenv("GNNMI_WHOLE");
    if (e && e[0] == '0') return false;
    return c->built && !c->is_whole && !c->streaming() && c->M.k > 1 &&
           c->M.stats.nnz < ((int64_t)1 << 31) && c->M.n + c->M.stats.sum_boundary < ((int64_t)1 << 30) && c->M.n <= kWholeMaxRows;
}

void copy_settings(const gnn_ctx* c, gnn_ctx* w)
{
    w->order_mode = c->order_mode;
    w->keep_forward = c->keep_forward;
    w->heads = c->heads;
    w->fuse_gather = c->fuse_gather;
    w->masked_bwd = c->masked_bwd;
    w->dropout_p = c->dropout_p;
    w->dropout_seed = c->dropout_seed;
    w->dropout_epoch = c->dropout_epoch;
    w->prof = c->prof;
}

}  // namespace

void whole_free(gnn_ctx* c)
{
    if (!c->whole) return;
    free_inner(c->whole);
    for (hipEvent_t e : c->whole->events) (void)hipEventDestroy(e);
    delete c->whole;
    c->whole = nullptr;
    c->whole_ready = false;
}

void whole_layout(gnn_ctx* c)
{
    c->whole_ready = false;
    if (!wanted(c)) {
        whole_free(c);
        return;
    }
    gnn_ctx* w = c->whole;
    if (!w) {
        w = new gnn_ctx();                        // (bad_alloc: reported by the caller as out of memory)
        c->whole = w;
        w->is_whole = true;
    }
    const HostMeta& M = c->M;
    w->model = c->model; w->dtype = c->dtype; w->L = c->L; w->has_bias = c->has_bias; w->dims = c->dims;
    w->parts_k = M.k;
    copy_settings(c, w);
    HostMeta& N = w->M;
    N = HostMeta{};
    N.n = M.n; N.k = 1; N.model = M.model;
    N.off = {0, M.n};
    N.boff = {0, M.boff[(size_t)M.k]};
    N.sched = {0};
    N.segment = M.segment;
    N.stats = M.stats;
    N.stats.k = 1;
    N.stats.max_own = M.n;
    N.stats.max_boundary = M.boff[(size_t)M.k];
    N.stats.max_nnz = M.stats.nnz;
    const HostMeta::Plan& H = M.plan_fwd;
    N.plan_fwd.segment = H.segment;
    N.plan_fwd.range_off = {0, H.range_off[(size_t)M.k]};
    N.plan_fwd.seg_off = {0, H.seg_off[(size_t)M.k]};
    N.plan_fwd.long_off = {0, H.long_off[(size_t)M.k]};
    N.plan_fwd.rows_off = {0, H.rows_off[(size_t)M.k]};
    N.plan_fwd.max_segs = H.seg_off[(size_t)M.k];
    w->built = true;
    w->fwd_done.assign((size_t)w->L, 0);
    w->xf_fwd_done.assign((size_t)w->L, 0);
    w->att_done.assign((size_t)w->L, 0);
    w->z_done.assign((size_t)w->L, 0);
    w->xf_bwd_done.assign((size_t)w->L, 0);
    w->bwd_done.assign((size_t)w->L + 2, 0);
    compute_workspace(w);
    // the boundary rows of all partitions pass through staging only while the gather is not fused;
    // a context that fuses it takes the memory only where it is little
    c->whole_staged = !c->fuse_gather || w->ws.staging_bytes <= ((int64_t)1 << 30);
    const int64_t staging = c->whole_staged ? std::max(c->ws.staging_bytes, w->ws.staging_bytes) : c->ws.staging_bytes;
    const int64_t scratch = std::max(c->ws.scratch_bytes, w->ws.scratch_bytes);
    if (staging + scratch - c->ws.staging_bytes - c->ws.scratch_bytes > kWholeLimitBytes) {
        whole_free(c);
        return;
    }
    c->ws.staging_bytes = staging;
    c->ws.scratch_bytes = scratch;
}

void whole_bind(gnn_ctx* c)
{
    c->whole_ready = false;
    gnn_ctx* w = c->whole;
    if (!w) return;
    free_inner(w);
    DevMeta& D = w->D;
    D.rp = c->D.rp;
    D.ew = c->D.ew;
    D.rscale = c->D.rscale;
    D.bnd = c->D.bnd;
    D.order = c->D.order;
    w->feat = c->feat; w->act = c->act; w->gact = c->gact; w->w = c->w; w->gw = c->gw;
    w->labels = c->labels; w->mask = c->mask;
    w->staging = c->staging; w->scratch = c->scratch;
    w->hbuf = w->ghbuf = nullptr;
    w->dyall_buf = nullptr;
    if (w->ws.h_floats > 0) {
        w->hbuf = w->scratch + w->ws.h;
        w->ghbuf = w->scratch + w->ws.gh;
        if (w->ws.dyall >= 0) w->dyall_buf = (float*)(w->scratch + w->ws.dyall);
    }
    try {
        build_forward_plan(c, w);
        build_tables(c, w);
    } catch (const Fail&) {
        free_inner(w);
        return;
    } catch (const std::bad_alloc&) {
        free_inner(w);
        return;
    }
    w->bound = true;
    whole_update(c);
}

// (re)builds what depends on the gather-fusion and masked-backward switches
void whole_update(gnn_ctx* c)
{
    c->whole_ready = false;
    gnn_ctx* w = c->whole;
    if (!w || !w->bound) return;
    copy_settings(c, w);
    bool any_transposed = c->L >= 2;
    bool full_used = false;                   // by a layer below the output layer
    for (int32_t l = 1; l <= c->L; ++l) {
        const bool uses = l >= 2 || c->transform_first(l);
        any_transposed = any_transposed || uses;
        full_used = full_used || (uses && l < c->L);
    }
    const bool masked = c->masked_bwd && c->D.masked_t.ready;
    try {
        check(hipDeviceSynchronize());
        w->D.gcol = c->fuse_gather ? c->D.gcol : nullptr;
        if (!w->gather_fused() && c->whole_staged) build_staged_columns(c, w);
        free_merged(w->D.merged_masked);
        if (any_transposed) {
            if (!w->D.merged.ready || !w->D.merged.col) {
                free_merged(w->D.merged);
                build_merged(c, w->D.merged);
            }
            if (masked) {
                build_merged_masked(c, w->D.merged, w->D.merged_masked);
                if (!full_used) {
                    // nothing but the output layer aggregates transposed: the marker stays, the arrays go
                    free_merged(w->D.merged);
                    w->D.merged.ready = true;
                }
            }
        } else {
            w->D.merged.ready = true;
        }
        check(hipDeviceSynchronize());
    } catch (const Fail&) {
        free_merged(w->D.merged);
        free_merged(w->D.merged_masked);
        return;
    } catch (const std::bad_alloc&) {
        free_merged(w->D.merged);
        free_merged(w->D.merged_masked);
        return;
    }
    c->whole_ready = true;
}

bool whole_runs(const gnn_ctx* c)
{
    // (profiled epochs that gather through staging bracket the steps of every partition)
    if (!c->whole_ready || (!c->whole->gather_fused() && (c->prof != 0 || !c->whole_staged))) return false;
    const char* e = std::getenv("GNNMI_WHOLE");
    return !(e && e[0] == '0');
}

MergedItems merged_items(const DevMeta::Merged& m)
{
    MergedItems it;
    it.rp = m.rp; it.col = m.col; it.w = m.w; it.perm = m.perm; it.rows = m.rows; it.nrows = m.nrows;
    it.unit_begin = m.unit_begin; it.unit_len = m.unit_len; it.nunits = m.nunits;
    it.long_row = m.long_row; it.long_first = m.long_first; it.long_nunits = m.long_nunits; it.nlong = m.nlong;
    it.partial = m.partial; it.avg_len = m.avg_len;
    return it;
}

void run_spmm_merged(gnn_ctx* c, int32_t layer, const void* src, float* out, int32_t d, int self, hipStream_t s)
{
    const DevMeta::Merged& m = layer == c->L && c->D.merged_masked.ready ? c->D.merged_masked : c->D.merged;
    const MergedItems it = merged_items(m);
    {
        Timed t(c, s, GNN_K_SPMM_T);
        launch_spmm_merged(it, src, c->bf16() ? 1 : 0, out, d, self, s);
    }
    if (it.nlong > 0) {
        Timed t(c, s, GNN_K_SPMM_REDUCE);
        launch_spmm_merged_reduce(it, out, d, self, s);
    }
}

gnn_status whole_epoch(gnn_ctx* c, void* stream, float* loss_out)
{
    gnn_ctx* w = c->whole;
    copy_settings(c, w);
    w->events_used = 0;
    const gnn_status st = epoch_resident(w, stream, loss_out);
    // what the per-partition entry points may build on afterwards: the activations, the loss and the
    // kept aggregates (same place, same rows); H and everything staged is gone
    c->staged_layer = c->staged_p = -1;
    c->h_layer = 0;
    std::fill(c->xf_fwd_done.begin(), c->xf_fwd_done.end(), 0);
    const uint8_t done = st == GNN_OK ? 1 : 0;
    std::fill(c->fwd_done.begin(), c->fwd_done.end(), done);
    std::fill(c->xf_bwd_done.begin(), c->xf_bwd_done.end(), done);
    std::fill(c->z_done.begin(), c->z_done.end(), done);
    std::fill(c->att_done.begin(), c->att_done.end(), 0);
    std::fill(c->bwd_done.begin(), c->bwd_done.end(), done ? c->M.k : 0);
    c->loss_done = done != 0;
    if (st != GNN_OK) {
        c->err = w->err;
        return st;
    }
    if (c->prof)
        for (int i = 0; i < GNN_K_COUNT; ++i) {
            c->prof_ms[i] = w->prof_ms[i];
            c->prof_launches[i] = w->prof_launches[i];
        }
    return GNN_OK;
}

}  // namespace gnnmi
