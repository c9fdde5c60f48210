// knn_batch_search: many independent k-NN jobs of uneven sizes in one call.
//
// Every job follows the steps of knn_search (threshold from a corpus sample,
// fused product with candidate filtering, exact fallback of unusable rows,
// candidate selection, exact re-rank), so its output is the same.  What changes
// is how the work reaches the device:
//  * the fused products of all jobs run as ONE launch of (job part, row tile,
//    column tile) items that the host orders for the hardware's round-robin
//    dispatch over the eight XCDs: per XCD a queue of parts, longest first, a
//    part's column range split into eight contiguous chunks, one per XCD, so
//    each corpus tile is read by one XCD, where the part's row tiles reuse it
//    from L2.  The items run one per workgroup, or (queue form) a resident
//    grid takes them from eight per-XCD atomic queues in the same order;
//  * FP32 jobs that two-half operands serve, and BF16 / FP8 jobs, take the
//    pipelined 256 x 256 form of that launch (gemm_pipe.hip);
//  * jobs with short corpora take the whole corpus as their sample (plan.hpp);
//  * the steps around the products (norms, operands, samples, list flags,
//    certificates, re-rank) run as one launch per kernel instance over all jobs:
//    96 uneven jobs 23.0 -> 16.1 ms, 57 jobs of 41 queries and up to 6987 points
//    3.28 -> 1.05 ms against a launch per job and step;
//  * every step of a call is captured into one HIP graph on the first call and
//    replayed by later calls with the same job table; one synchronisation then
//    brings the counts of rows needing the exact fallback or re-run (rare) to the
//    host;
//  * with autotuning on, the tile shape and form of the grouped launch (of the
//    parts that are neither pipelined nor selected from their sample) are
//    the fastest of the candidates, timed on the batch itself with a threshold
//    of -inf (nothing is kept, so the timing run has no effect on the results).
// Jobs with more than kRowBlock queries are split into parts of at most that
// many rows; each part has its own candidate lists.  Parts whose threshold
// sample is their whole corpus have no product but the sample's.
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <string>
#include <vector>

#include "autotune.hpp"
#include "dist.hpp"
#include "handle.hpp"
#include "internal.hpp"
#include "knn.h"
#include "plan.hpp"

namespace knn {

knn_status_t fail_msg(knn_handle_t h, knn_status_t s, const std::string &msg);
unsigned long long *stats_ptr(knn_handle_t h);
void add_host_stats(knn_handle_t h, int64_t rows, int64_t fallback_rows);
void add_host_rerun(knn_handle_t h, int64_t rows);
void add_host_candidates(knn_handle_t h, int64_t n);
int handle_num_cu(knn_handle_t h);
const uint16_t *handle_net(knn_handle_t h);
hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t stream);
knn_status_t ensure_unit_ws(knn_handle_t h, size_t bytes, hipStream_t stream, void **out);
knn_status_t run_search(knn_handle_t h, const float *Q, int64_t m, const float *C, int64_t n, int d, int k, bool graph,
                        float *out_dist, int32_t *out_idx, hipStream_t stream, const knn_options_t *opt);

struct BatchJob {
    const float *Q, *C;
    int64_t m, n;
    int d, k;
    bool graph;
    float *out_dist;
    int32_t *out_idx;
    Plan p;
    double cost;  // 2 m n d
    float oscale = 1.0f;  // returned distance = oscale * squared distance (cosine / Pearson: 1/2)
    // per-job buffers
    float *cnorm = nullptr, *qn2 = nullptr;
    unsigned int *cmax2 = nullptr;
    void *Cq = nullptr, *Qq = nullptr;
    float *cs = nullptr, *qs = nullptr;
    // the threshold sample of the corpus (the corpus itself when not gathered)
    const float *Cs = nullptr, *csn = nullptr, *css = nullptr;
    const void *Csq = nullptr;
    int first_part = 0, nparts = 0;
};

struct BatchPart {
    int job;
    int64_t i0, mb;
    bool direct;    // the threshold sample is the whole corpus: its selection is the candidate list
    bool pipe;      // FILTER product in the grouped pipelined launch
    bool grouped;   // else in the grouped launch (or its own: FP32 with d % 4 != 0)
    bool spipe;     // sample product in the grouped pipelined launch (two-half operands)
    bool sgrouped;  // else in the grouped launch (or its own)
    float *Ds = nullptr;   // mb x S sample distances
    float *tv = nullptr;   // mb x (r + 1) selected sample keys (values, indices)
    int32_t *ti = nullptr;
    uint32_t *cnt = nullptr;
    uint64_t *cand = nullptr;
    int32_t *flags = nullptr;
    float *sv = nullptr;   // mb x kk selected candidates
    int32_t *si = nullptr;
    int32_t *ulist = nullptr;  // FP32: uncertified rows, re-run exactly
    float *tfix = nullptr;
};

// A multi-matrix selection launch: its segments and the segment of each row.
struct SegLaunch {
    int cap = 0;
    int64_t rows = 0;
    uint32_t cols = 0, k = 0;
    std::vector<SelectSeg> segs;
    std::vector<uint32_t> row_seg;
    SelectSeg *dsegs = nullptr;
    uint32_t *drow_seg = nullptr;
};

// Buffers shared by all jobs; every use of one is ordered on the stream.
struct BatchShared {
    float *Qf = nullptr, *Df = nullptr, *fv = nullptr, *qfs = nullptr;
    void *Qfq = nullptr;
    int32_t *fi = nullptr;
    void *selws = nullptr;
    size_t selws_bytes = 0;
    float *ninf = nullptr;
    uint32_t *zeros = nullptr;    // cmax2, nflag, nu and cnt_all, cleared by each call
    int64_t nzeros = 0;
    uint32_t *cnt_all = nullptr;  // the candidate counts of all parts, contiguous
    int64_t cnt_rows = 0;
    DistArgs *table = nullptr, *probe = nullptr, *stable = nullptr;
    GemmItem *items = nullptr, *sitems = nullptr;    // 128 x 128 .. tiles of gemm.hip
    GemmItem *pitems = nullptr, *psitems = nullptr;  // tiles of the pipelined product
    unsigned int *cmax2 = nullptr;                   // per job, the largest squared corpus norm
    uint32_t *nflag = nullptr;
    uint32_t *nu = nullptr;  // uncertified-row counts, one per part
    // the preparation, flag, certificate and re-rank steps of all jobs or parts
    PrepSeg *preps = nullptr;
    FlagSeg *flags = nullptr;
    CertifyArgs *certs = nullptr;
    RerankArgs *reranks = nullptr;
    uint32_t *preps_first = nullptr, *flags_first = nullptr, *certs_first = nullptr, *reranks_first = nullptr;
    uint32_t *queues = nullptr;  // the eight per-XCD item queues of the persistent product
};

// State of the last batch of a handle: its workspace, plan and graphs.
struct BatchState {
    std::vector<uint8_t> key;
    void *ws = nullptr;
    size_t ws_bytes = 0;
    uint32_t *nflag_host = nullptr;  // pinned: per part the flagged-row count, then the uncertified-row count
    size_t nflag_host_cap = 0;
    hipStream_t cap_stream = nullptr;
    std::vector<hipGraphExec_t> graphs;  // in launch order, see the segments
    bool eager = true;                   // replay eagerly (no graphs)
    bool timed = false;
    std::vector<BatchJob> jobs;
    std::vector<BatchPart> parts;
    std::vector<int> order;  // jobs, longest first
    BatchShared sh;
    int tile = kTileWide;
    bool queue = false;  // the product as a resident grid over per-XCD item queues
    size_t nitems = 0, nsitems = 0, npitems = 0, npsitems = 0;
    std::vector<SegClass> preps, flags, certs, reranks;  // their launches
    std::vector<SegLaunch> sample_sel;  // threshold selections, one launch per capacity class
    SegLaunch keys_sel;                 // candidate selections
    int smode = kPivotSample;
    const uint16_t *net = nullptr;
    int force = 0;

    void drop_graphs() {
        for (hipGraphExec_t g : graphs) hipGraphExecDestroy(g);
        graphs.clear();
    }
    ~BatchState() {
        drop_graphs();
        if (cap_stream) hipStreamDestroy(cap_stream);
        if (ws) hipFree(ws);
        if (nflag_host) hipHostFree(nflag_host);
    }
};

void batch_release(knn_handle_t h) {
    delete h->batch;
    h->batch = nullptr;
}

namespace {

// Items of the grouped launch for a tile shape, in dispatch order.  Eight
// queues, one per XCD, each holding the parts longest first; a part's column
// tiles are split into eight contiguous chunks (chunk q to queue q), each
// column tile followed by all of the part's row tiles (which then find it in
// their XCD's L2).  Workgroup b runs on XCD b % 8 and takes the next item of
// that queue; once a queue is empty its XCD takes items from the back of the
// fullest remaining queue (the shortest work there).
// Autotune candidates: a tile shape, plus this for the queue form.
constexpr int kQueueChoice = 16;

constexpr int kPipeForm = -2;  // tile argument: the pipelined product's tiles and parts

void build_items(const BatchState &b, int tile, std::vector<GemmItem> &items) {
    constexpr int kQueues = 8;
    int bm = kPipeTileDim, bn = kPipeTileDim;
    if (tile != kPipeForm) gemm_tile_dims(tile, &bm, &bn);
    std::vector<std::vector<GemmItem>> q(kQueues);
    for (int j : b.order) {
        const BatchJob &js = b.jobs[j];
        for (int pi = js.first_part; pi < js.first_part + js.nparts; ++pi) {
            const BatchPart &pt = b.parts[pi];
            if (tile == kPipeForm ? !pt.pipe : !pt.grouped) continue;
            const uint32_t tm_n = (uint32_t)((pt.mb + bm - 1) / bm);
            const uint32_t tn_n = (uint32_t)((js.n + bn - 1) / bn);
            for (int qi = 0; qi < kQueues; ++qi) {
                const uint32_t c0 = (uint32_t)((uint64_t)tn_n * qi / kQueues);
                const uint32_t c1 = (uint32_t)((uint64_t)tn_n * (qi + 1) / kQueues);
                for (uint32_t tn = c0; tn < c1; ++tn)
                    for (uint32_t tm = 0; tm < tm_n; ++tm) q[qi].push_back(GemmItem{(uint32_t)pi, tm, tn});
            }
        }
    }
    size_t total = 0;
    for (const auto &x : q) total += x.size();
    items.clear();
    items.reserve(total);
    std::vector<size_t> head(kQueues, 0), tail(kQueues);
    for (int qi = 0; qi < kQueues; ++qi) tail[qi] = q[qi].size();
    for (size_t t = 0; t < total; ++t) {
        const int qi = (int)(t % kQueues);
        if (head[qi] < tail[qi]) {
            items.push_back(q[qi][head[qi]++]);
            continue;
        }
        int best = -1;
        for (int o = 0; o < kQueues; ++o)
            if (head[o] < tail[o] && (best < 0 || tail[o] - head[o] > tail[best] - head[best])) best = o;
        items.push_back(q[best][--tail[best]]);
    }
}

size_t max_items(const BatchState &b) {
    // the 128 x 128 tile gives the most items
    size_t n = 0;
    for (const BatchPart &pt : b.parts)
        if (pt.grouped) n += (size_t)((pt.mb + 127) / 128) * (size_t)((b.jobs[pt.job].n + 127) / 128);
    return n;
}

// Items of the grouped sample products (128 x 128 tiles, or the pipelined
// product's), part after part.
void build_sample_items(const BatchState &b, bool pipe, std::vector<GemmItem> &items) {
    items.clear();
    const int t = pipe ? kPipeTileDim : 128;
    for (size_t pi = 0; pi < b.parts.size(); ++pi) {
        const BatchPart &pt = b.parts[pi];
        if (pipe ? !pt.spipe : !pt.sgrouped) continue;
        const uint32_t tm_n = (uint32_t)((pt.mb + t - 1) / t), tn_n = (uint32_t)((b.jobs[pt.job].p.S + t - 1) / t);
        for (uint32_t tm = 0; tm < tm_n; ++tm)
            for (uint32_t tn = 0; tn < tn_n; ++tn) items.push_back(GemmItem{(uint32_t)pi, tm, tn});
    }
}

// The threshold selections of all parts (k = r + 1 over their S sample
// distances), one launch per capacity class, and the candidate selections of
// the filtered parts (k = kk over their candidate lists), one launch.
void plan_selects(BatchState &b) {
    b.sample_sel.clear();
    // a sample row that fits the on-chip capacity is selected there directly
    // (no pivot sample, no streaming), so short rows go to the class that holds them
    // (class 0: rows selected in registers)
    auto sample_cap = [&b](const Plan &p) {
        if (b.smode == kPivotSample && select_short_shape((uint32_t)p.S, (uint32_t)(p.r + 1))) return 0;
        int c = select_cap_for_k((uint32_t)(p.r + 1));
        if (p.S > c && p.S <= kSelectKeysCap) c = p.S <= 2048 ? 2048 : 4096;
        return c;
    };
    for (int cap : {0, 1024, 2048, 4096}) {
        SegLaunch L;
        L.cap = cap;
        for (const BatchPart &pt : b.parts) {
            const Plan &p = b.jobs[pt.job].p;
            if (sample_cap(p) != cap) continue;
            SelectSeg sg{};
            sg.dist = pt.Ds;
            sg.ld = p.S;
            sg.row0 = L.rows;
            sg.cols = (uint32_t)p.S;
            sg.k = (uint32_t)(p.r + 1);
            sg.out_val = pt.tv;
            sg.out_idx = pt.ti;
            L.cols = std::max(L.cols, sg.cols);
            L.k = std::max(L.k, sg.k);
            for (int64_t i = 0; i < pt.mb; ++i) L.row_seg.push_back((uint32_t)L.segs.size());
            L.segs.push_back(sg);
            L.rows += pt.mb;
        }
        if (L.rows) b.sample_sel.push_back(std::move(L));
    }
    SegLaunch K;
    K.cap = kSelectKeysCap;
    for (const BatchPart &pt : b.parts) {
        if (pt.direct) continue;
        const Plan &p = b.jobs[pt.job].p;
        SelectSeg sg{};
        sg.keys = pt.cand;
        sg.key_cnt = pt.cnt;
        sg.ld = p.cap;
        sg.row0 = K.rows;
        sg.cols = (uint32_t)p.cap;
        sg.k = (uint32_t)p.kk;
        sg.out_val = pt.sv;
        sg.out_idx = pt.si;
        K.cols = std::max(K.cols, sg.cols);
        K.k = std::max(K.k, sg.k);
        for (int64_t i = 0; i < pt.mb; ++i) K.row_seg.push_back((uint32_t)K.segs.size());
        K.segs.push_back(sg);
        K.rows += pt.mb;
    }
    b.keys_sel = std::move(K);
}

constexpr size_t kPrepSegs = 4;  // preparation segments of a job, at most

// Lays out the batch workspace (sizing pass with base == nullptr).  Every
// part keeps its own sample distances, selections and candidate lists, so
// each phase can run as one launch over all parts.
size_t carve_batch(Carve &c, BatchState &b, int num_cu, bool probe) {
    BatchShared &s = b.sh;
    // everything that a call starts from zero
    int64_t cnt_rows = 0;
    for (const BatchPart &pt : b.parts)
        if (!pt.direct) cnt_rows += pt.mb;
    const size_t njobs = b.jobs.size(), nparts = b.parts.size();
    s.nzeros = (int64_t)(njobs + 2 * nparts) + cnt_rows;
    s.zeros = c.take<uint32_t>((size_t)s.nzeros);
    s.cmax2 = s.zeros;
    s.nflag = s.zeros ? s.zeros + njobs : nullptr;
    s.nu = s.zeros ? s.nflag + nparts : nullptr;
    s.cnt_all = s.zeros ? s.nu + nparts : nullptr;
    s.cnt_rows = cnt_rows;
    for (size_t j = 0; j < b.jobs.size(); ++j) b.jobs[j].cmax2 = s.cmax2 ? s.cmax2 + j : nullptr;
    size_t qf = 0, df = 0, fv = 0, qfq = 0, fb = 0, selws = 0;
    for (BatchJob &js : b.jobs) {
        const Plan &p = js.p;
        js.cnorm = c.take<float>(js.n);
        js.qn2 = js.graph ? js.cnorm : c.take<float>(js.m);  // (a graph's queries are its corpus)
        if (p.prec != kPrecF32 || p.split) {
            js.Cq = c.take<char>((size_t)js.n * p.ldq);
            js.cs = c.take<float>(js.n);
            if (!js.graph) {
                js.Qq = c.take<char>((size_t)js.m * p.ldq);
                js.qs = c.take<float>(js.m);
            } else {
                js.Qq = js.Cq;
                js.qs = js.cs;
            }
        }
        js.Cs = js.C;
        js.csn = js.cnorm;
        js.Csq = js.Cq;
        js.css = js.cs;
        if (p.gathered && js.nparts) {
            js.csn = c.take<float>(p.S);
            if (p.prec != kPrecF32 || p.split) {
                js.Csq = c.take<char>((size_t)p.S * p.ldq);
                js.css = c.take<float>(p.S);
            } else {
                js.Cs = c.take<float>((size_t)p.S * p.d);
            }
        }
        qf = std::max(qf, (size_t)p.Fb * p.d);
        df = std::max(df, (size_t)p.Fb * js.n);
        fv = std::max(fv, (size_t)p.Fb * p.kk);
        if (!p.split) qfq = std::max(qfq, (size_t)p.Fb * p.ldq);
        fb = std::max(fb, (size_t)p.Fb);
        const int cap2 = select_cap_for_k(p.kk);
        selws = std::max(selws, select_ws_bytes(cap2, (uint32_t)js.n, select_grid(cap2, p.Fb, num_cu)));
    }
    int64_t cnt_off = 0;
    for (BatchPart &pt : b.parts) {
        const Plan &p = b.jobs[pt.job].p;
        pt.Ds = c.take<float>((size_t)pt.mb * p.S);
        pt.tv = c.take<float>((size_t)pt.mb * (p.r + 1));
        pt.ti = c.take<int32_t>((size_t)pt.mb * (p.r + 1));
        if (pt.direct) continue;
        pt.cnt = s.cnt_all ? s.cnt_all + cnt_off : nullptr;
        cnt_off += pt.mb;
        pt.cand = c.take<uint64_t>((size_t)pt.mb * p.cap);
        pt.flags = c.take<int32_t>(pt.mb);
        pt.sv = c.take<float>((size_t)pt.mb * p.kk);
        pt.si = c.take<int32_t>((size_t)pt.mb * p.kk);
    }
    for (BatchPart &pt : b.parts) {
        if (b.jobs[pt.job].p.prec != kPrecF32) continue;
        pt.ulist = c.take<int32_t>((size_t)pt.mb);
        pt.tfix = c.take<float>((size_t)pt.mb);
    }
    plan_selects(b);
    for (SegLaunch &L : b.sample_sel) {
        if (L.cap) selws = std::max(selws, select_ws_bytes(L.cap, L.cols, select_grid(L.cap, L.rows, num_cu)));
        L.dsegs = c.take<SelectSeg>(L.segs.size());
        L.drow_seg = c.take<uint32_t>((size_t)L.rows);
    }
    b.keys_sel.dsegs = c.take<SelectSeg>(std::max<size_t>(b.keys_sel.segs.size(), 1));
    b.keys_sel.drow_seg = c.take<uint32_t>((size_t)std::max<int64_t>(b.keys_sel.rows, 1));
    s.Qf = c.take<float>(qf);
    s.Df = c.take<float>(df);
    s.fv = c.take<float>(fv);
    s.fi = c.take<int32_t>(fv);
    s.Qfq = c.take<char>(qfq);
    s.qfs = c.take<float>(fb);
    s.selws_bytes = selws < 256 ? 256 : selws;
    s.selws = c.take<char>(s.selws_bytes);
    s.ninf = c.take<float>(1);
    s.table = c.take<DistArgs>(b.parts.size());
    s.stable = c.take<DistArgs>(b.parts.size());
    s.probe = probe ? c.take<DistArgs>(b.parts.size()) : nullptr;
    s.items = c.take<GemmItem>(std::max<size_t>(max_items(b), 1));
    std::vector<GemmItem> si;
    build_sample_items(b, false, si);
    s.sitems = c.take<GemmItem>(std::max<size_t>(si.size(), 1));
    b.nsitems = si.size();
    build_sample_items(b, true, si);
    s.psitems = c.take<GemmItem>(std::max<size_t>(si.size(), 1));
    b.npsitems = si.size();
    b.npitems = 0;
    for (const BatchPart &pt : b.parts)
        if (pt.pipe)
            b.npitems += (size_t)((pt.mb + kPipeTileDim - 1) / kPipeTileDim) *
                         (size_t)((b.jobs[pt.job].n + kPipeTileDim - 1) / kPipeTileDim);
    s.pitems = c.take<GemmItem>(std::max<size_t>(b.npitems, 1));
    s.queues = c.take<uint32_t>(8);
    const size_t np = kPrepSegs * b.jobs.size(), parts = b.parts.size();
    s.preps = c.take<PrepSeg>(np);
    s.preps_first = c.take<uint32_t>(2 * np);
    s.flags = c.take<FlagSeg>(parts);
    s.flags_first = c.take<uint32_t>(2 * parts);
    s.certs = c.take<CertifyArgs>(parts);
    s.certs_first = c.take<uint32_t>(2 * parts);
    s.reranks = c.take<RerankArgs>(parts);
    s.reranks_first = c.take<uint32_t>(2 * parts);
    return c.off;
}

DistArgs part_args(const BatchState &b, const BatchPart &pt) {
    const BatchJob &js = b.jobs[pt.job];
    const Plan &p = js.p;
    DistArgs a{};
    a.Q = js.Q + pt.i0 * js.d;
    a.m = pt.mb;
    a.C = js.C;
    a.n = js.n;
    a.d = js.d;
    a.cnorm = js.cnorm;
    a.self_offset = js.graph ? pt.i0 : -1;
    a.tau = pt.tv ? pt.tv + p.r : nullptr;  // the threshold is the last selected sample key
    a.tau_stride = p.r + 1;
    a.cnt = pt.cnt;
    a.cand = pt.cand;
    a.cap = p.cap;
    a.prec = p.split ? kPrecSplit : p.prec;
    a.Qq = js.Qq ? static_cast<const char *>(js.Qq) + pt.i0 * p.ldq : nullptr;
    a.Cq = js.Cq;
    a.ldq = p.ldq;
    a.qscale = js.qs ? js.qs + pt.i0 : nullptr;
    a.cscale = js.cs;
    return a;
}

// The sample product of a part: its rows against the job's threshold sample.
DistArgs sample_args(const BatchState &b, const BatchPart &pt) {
    const BatchJob &js = b.jobs[pt.job];
    const Plan &p = js.p;
    DistArgs sa = part_args(b, pt);
    sa.C = js.Cs;
    sa.n = p.S;
    sa.cnorm = js.csn;
    sa.self_offset = (js.graph && !p.gathered) ? pt.i0 : -1;
    sa.out = pt.Ds;
    sa.ldo = p.S;
    sa.tau = nullptr;
    sa.cnt = nullptr;
    sa.cand = nullptr;
    sa.Cq = js.Csq;
    sa.cscale = js.css;
    return sa;
}

SelectArgs seg_select_args(const BatchState &b, const SegLaunch &L) {
    SelectArgs a{};
    a.rows = L.rows;
    a.cols = L.cols;
    a.k = L.k;
    a.mode = b.smode;
    a.net = b.smode == kPivotLearned ? b.net : nullptr;
    a.segs = L.dsegs;
    a.row_seg = L.drow_seg;
    return a;
}

// Certificate of a part's kk candidates (FP32: uncertified rows are listed for
// the exact re-run; none is needed where they are all there are), and its exact
// re-rank.
const float *part_keys(const BatchPart &pt) { return pt.direct ? pt.tv : pt.sv; }
const int32_t *part_cidx(const BatchPart &pt) { return pt.direct ? pt.ti : pt.si; }
bool part_certified(const BatchState &b, const BatchPart &pt) {
    const Plan &p = b.jobs[pt.job].p;
    return p.kk < p.n_eff;
}

CertifyArgs certify_args(const BatchState &b, knn_handle_t h, size_t pi) {
    const BatchPart &pt = b.parts[pi];
    const BatchJob &js = b.jobs[pt.job];
    const Plan &p = js.p;
    return CertifyArgs{part_keys(pt), pt.mb, p.kk, js.k, js.qn2 + pt.i0, js.cmax2, p.rel, p.gamma,
                       stats_ptr(h) + kStatUncertified};
}

RerankArgs rerank_args(const BatchState &b, size_t pi) {
    const BatchPart &pt = b.parts[pi];
    const BatchJob &js = b.jobs[pt.job];
    const Plan &p = js.p;
    RerankArgs rr{js.Q + pt.i0 * js.d, pt.mb, js.C, js.n, js.d, part_cidx(pt), (uint32_t)p.kk, js.k,
                  js.out_dist + pt.i0 * js.k, js.out_idx + pt.i0 * js.k, js.graph ? pt.i0 : -1, js.oscale};
    if (part_certified(b, pt) && p.prec == kPrecF32) {
        rr.keys = part_keys(pt);
        rr.qnorm2 = js.qn2 + pt.i0;
        rr.cmax2_bits = js.cmax2;
        rr.rel = p.rel;
        rr.gamma = p.gamma;
        rr.ulist = pt.ulist;
        rr.nu = b.sh.nu + pi;
        rr.tfix = pt.tfix;
        rr.force = p.force_rerun;
        rr.rel_fix = pt.direct ? p.rel : p.gamma;  // (other parts: re-run from the FP32 product)
    }
    return rr;
}

// Norms, two-half or quantised operands, and the threshold sample of every job.
std::vector<PrepSeg> prep_segs(const BatchState &b) {
    std::vector<PrepSeg> v;
    for (int j : b.order) {
        const BatchJob &js = b.jobs[j];
        const Plan &p = js.p;
        if (js.nparts == 0) continue;
        const bool quant = p.prec != kPrecF32;
        auto add = [&](const float *X, int64_t n, int64_t src_n, const void *out, const float *scale, const float *norm,
                       unsigned int *max_bits) {
            const int kind = p.split ? kPrepSplit : (quant ? kPrepQuant : kPrepNorm);
            const bool operands = kind != kPrepNorm;
            v.push_back(PrepSeg{kind, X, n, src_n, js.d, p.prec, operands ? const_cast<void *>(out) : nullptr,
                                operands ? const_cast<float *>(scale) : nullptr, const_cast<float *>(norm), max_bits});
        };
        add(js.C, js.n, 0, js.Cq, js.cs, js.cnorm, js.cmax2);
        if (!js.graph) add(js.Q, js.m, 0, js.Qq, js.qs, js.qn2, nullptr);
        if (!p.gathered) continue;
        add(js.C, p.S, js.n, js.Csq, js.css, js.csn, nullptr);
        if (!quant && !p.split)
            v.push_back(PrepSeg{kPrepGather, js.C, p.S, js.n, js.d, p.prec, const_cast<float *>(js.Cs), nullptr,
                                nullptr, nullptr});
    }
    return v;
}

// ---- the phases, enqueued on a stream (captured or eager) ------------------
hipError_t enqueue_prep(const BatchState &b, int num_cu, hipStream_t s) {
    hipError_t e = hipSuccess;
    const BatchShared &sh = b.sh;
#define BTRY(call)                                 \
    do {                                           \
        if ((e = (call)) != hipSuccess) return e;  \
    } while (0)
    BTRY(launch_fill_u32(sh.zeros, sh.nzeros, 0u, s));
    for (const SegClass &c : b.preps) BTRY(launch_prep_group(c, sh.preps, sh.preps_first, s));
    // all sample products in one launch per form (FP32 parts with d % 4 != 0 on their own)
    BTRY(launch_dist_gemm_pipe_grouped(sh.stable, sh.psitems, (int64_t)b.npsitems, kPrecSplit, s, kEpiDense));
    BTRY(launch_dist_gemm_grouped(sh.stable, sh.sitems, (int64_t)b.nsitems, b.jobs[0].p.prec, kTileSmall, s,
                                  kEpiDense));
    for (const BatchPart &pt : b.parts)
        if (!pt.sgrouped && !pt.spipe) BTRY(launch_dist_gemm(sample_args(b, pt), kEpiDense, s));
    // all threshold selections, one launch per capacity class
    for (const SegLaunch &L : b.sample_sel) {
        SelectArgs sa = seg_select_args(b, L);
        if (L.cap == 0) BTRY(launch_select_short(sa, num_cu, s));
        else BTRY(launch_select(sa, L.cap, select_grid(L.cap, L.rows, num_cu), sh.selws, s));
    }
    return e;
}

hipError_t enqueue_product(const BatchState &b, const DistArgs *table, int tile, bool queue, int num_cu,
                           hipStream_t s) {
    hipError_t e = hipSuccess;
    if (table != b.sh.probe) {  // (the timed forms differ in the other parts alone)
        const int prec = b.jobs[0].p.prec == kPrecF32 ? kPrecSplit : b.jobs[0].p.prec;
        BTRY(launch_dist_gemm_pipe_grouped(table, b.sh.pitems, (int64_t)b.npitems, prec, s));
    }
    if (queue)
        BTRY(launch_dist_gemm_queue(table, b.sh.items, (int64_t)b.nitems, b.jobs[0].p.prec, tile, b.sh.queues, num_cu,
                                    s));
    else
        BTRY(launch_dist_gemm_grouped(table, b.sh.items, (int64_t)b.nitems, b.jobs[0].p.prec, tile, s));
    for (const BatchPart &pt : b.parts) {
        if (pt.grouped || pt.pipe || pt.direct) continue;
        DistArgs fa = part_args(b, pt);
        fa.tile = tile;
        if (table == b.sh.probe) {
            fa.tau = b.sh.ninf;
            fa.tau_stride = 0;
        }
        BTRY(launch_dist_gemm(fa, kEpiFilter, s));
    }
    return e;
}

hipError_t enqueue_flags(const BatchState &b, knn_handle_t h, hipStream_t s) {
    hipError_t e = hipSuccess;
    for (const SegClass &c : b.flags) BTRY(launch_flag_group(c, b.sh.flags, b.sh.flags_first, s));
    return hipMemcpyAsync(b.nflag_host, b.sh.nflag, b.parts.size() * sizeof(uint32_t), hipMemcpyDeviceToHost, s);
}

hipError_t enqueue_final(const BatchState &b, int num_cu, hipStream_t s) {
    hipError_t e = hipSuccess;
    // the kk smallest candidate keys of every filtered row, one launch
    if (b.keys_sel.rows) {
        SelectArgs ka = seg_select_args(b, b.keys_sel);
        BTRY(launch_select_keys(ka, num_cu, s));
    }
    for (const SegClass &c : b.certs) BTRY(launch_certify_group(c, b.sh.certs, b.sh.certs_first, s));
    for (const SegClass &c : b.reranks) BTRY(launch_rerank_group(c, b.sh.reranks, b.sh.reranks_first, s));
    // the uncertified-row counts, for the exact re-run that follows
    return hipMemcpyAsync(b.nflag_host + b.parts.size(), b.sh.nu, b.parts.size() * sizeof(uint32_t),
                          hipMemcpyDeviceToHost, s);
}

// After the flagged rows' candidate lists are re-done: the candidate selection,
// certificate and re-rank of one part again (its uncertified list restarts).
hipError_t refinal_part(const BatchState &b, knn_handle_t h, int num_cu, size_t pi, hipStream_t s) {
    hipError_t e = hipSuccess;
    const BatchPart &pt = b.parts[pi];
    const Plan &p = b.jobs[pt.job].p;
    BTRY(launch_fill_u32(b.sh.nu + pi, 1, 0u, s));
    SelectArgs ka{};
    ka.keys = pt.cand;
    ka.key_cnt = pt.cnt;
    ka.rows = pt.mb;
    ka.cols = (uint32_t)p.cap;
    ka.ld = p.cap;
    ka.k = (uint32_t)p.kk;
    ka.out_val = pt.sv;
    ka.out_idx = pt.si;
    ka.mode = b.smode;
    ka.net = b.smode == kPivotLearned ? b.net : nullptr;
    BTRY(launch_select_keys(ka, num_cu, s));
    if (part_certified(b, pt) && p.prec != kPrecF32) BTRY(launch_certify(certify_args(b, h, pi), s));
    BTRY(launch_rerank(rerank_args(b, pi), s));
    return hipMemcpyAsync(b.nflag_host + b.parts.size() + pi, b.sh.nu + pi, sizeof(uint32_t), hipMemcpyDeviceToHost,
                          s);
}

// Exact re-do of the flagged rows of every part (after the flag counts reached
// the host), as in knn_search.
hipError_t run_fallback(const BatchState &b, int num_cu, hipStream_t s, int64_t *total) {
    hipError_t e = hipSuccess;
    const BatchShared &sh = b.sh;
    for (size_t pi = 0; pi < b.parts.size(); ++pi) {
        const int64_t nf = b.nflag_host[pi];
        if (nf == 0) continue;
        *total += nf;
        const BatchPart &pt = b.parts[pi];
        const BatchJob &js = b.jobs[pt.job];
        const Plan &p = js.p;
        const float *Qb = js.Q + pt.i0 * js.d;
        for (int64_t f0 = 0; f0 < nf; f0 += p.Fb) {
            const int64_t fb = nf - f0 < p.Fb ? nf - f0 : p.Fb;
            BTRY(launch_gather_rows(Qb, pt.mb, js.d, pt.flags + f0, fb, sh.Qf, nullptr, nullptr, s));
            if (p.prec != kPrecF32) BTRY(launch_quantize(sh.Qf, fb, js.d, p.prec, sh.Qfq, sh.qfs, s));
            DistArgs da{};
            da.Q = sh.Qf;
            da.m = fb;
            da.C = js.C;
            da.n = js.n;
            da.d = js.d;
            da.cnorm = js.cnorm;
            da.self_offset = js.graph ? pt.i0 : -1;
            da.row_ids = pt.flags + f0;
            da.out = sh.Df;
            da.ldo = js.n;
            da.prec = p.prec;
            da.Qq = sh.Qfq;
            da.Cq = js.Cq;
            da.ldq = p.ldq;
            da.qscale = sh.qfs;
            da.cscale = js.cs;
            BTRY(launch_dist_gemm(da, kEpiDense, s));
            BTRY(select_dense(sh.Df, fb, js.n, js.n, p.kk, sh.fv, sh.fi, sh.selws, sh.selws_bytes, num_cu, b.smode, b.net, s));
            BTRY(launch_scatter_fallback(pt.flags + f0, fb, sh.fv, sh.fi, p.kk, pt.cand, pt.cnt, p.cap, s));
        }
    }
    return e;
}
// Exact re-run of the uncertified FP32 rows of every part (after their counts
// reached the host): from the part's sample distances when the sample is the
// whole corpus, else from rows materialised here.
hipError_t run_rerun(const BatchState &b, hipStream_t s, int64_t *total) {
    hipError_t e = hipSuccess;
    const BatchShared &sh = b.sh;
    const uint32_t *counts = b.nflag_host + b.parts.size();
    for (size_t pi = 0; pi < b.parts.size(); ++pi) {
        const int64_t nu = counts[pi];
        if (nu == 0) continue;
        *total += nu;
        const BatchPart &pt = b.parts[pi];
        const BatchJob &js = b.jobs[pt.job];
        const Plan &p = js.p;
        const float *Qb = js.Q + pt.i0 * js.d;
        FixupArgs fx{};
        fx.out_scale = js.oscale;
        fx.tfix = pt.tfix;
        fx.Q = Qb;
        fx.C = js.C;
        fx.n = js.n;
        fx.d = js.d;
        fx.k = js.k;
        fx.self_offset = js.graph ? pt.i0 : -1;
        fx.out_dist = js.out_dist + pt.i0 * js.k;
        fx.out_idx = js.out_idx + pt.i0 * js.k;
        if (pt.direct) {
            fx.D = pt.Ds;
            fx.ldd = p.S;
            fx.by_row = true;
            fx.rows = pt.ulist;
            fx.nrows = nu;
            BTRY(launch_fixup(fx, s));
            continue;
        }
        for (int64_t f0 = 0; f0 < nu; f0 += p.Fb) {
            const int64_t fb = nu - f0 < p.Fb ? nu - f0 : p.Fb;
            BTRY(launch_gather_rows(Qb, pt.mb, js.d, pt.ulist + f0, fb, sh.Qf, nullptr, nullptr, s));
            DistArgs da{};
            da.Q = sh.Qf;
            da.m = fb;
            da.C = js.C;
            da.n = js.n;
            da.d = js.d;
            da.cnorm = js.cnorm;
            da.self_offset = js.graph ? pt.i0 : -1;
            da.row_ids = pt.ulist + f0;
            da.out = sh.Df;
            da.ldo = js.n;
            BTRY(launch_dist_gemm(da, kEpiDense, s));
            fx.D = sh.Df;
            fx.ldd = js.n;
            fx.by_row = false;
            fx.rows = pt.ulist + f0;
            fx.nrows = fb;
            BTRY(launch_fixup(fx, s));
        }
    }
    return e;
}
#undef BTRY

// Captures `fn` enqueued on the state's capture stream into an executable graph.
hipError_t capture(BatchState &b, const std::function<hipError_t(hipStream_t)> &fn, hipGraphExec_t *out) {
    *out = nullptr;
    hipError_t e = hipStreamBeginCapture(b.cap_stream, hipStreamCaptureModeRelaxed);
    if (e != hipSuccess) return e;
    hipError_t fe = fn(b.cap_stream);
    hipGraph_t g = nullptr;
    e = hipStreamEndCapture(b.cap_stream, &g);
    if (fe != hipSuccess) e = fe;
    if (e == hipSuccess) e = hipGraphInstantiate(out, g, nullptr, nullptr, 0);
    if (g) hipGraphDestroy(g);
    if (e != hipSuccess) {
        *out = nullptr;
        (void)hipGetLastError();
    }
    return e;
}

std::vector<uint8_t> make_key(const knn_job_t *jobs, int32_t njobs, const knn_options_t &o, int smode,
                              const uint16_t *net, const void *ws) {
    std::vector<uint8_t> k(sizeof(knn_job_t) * (size_t)njobs + sizeof(o) + sizeof(smode) + 2 * sizeof(void *));
    uint8_t *p = k.data();
    std::memcpy(p, jobs, sizeof(knn_job_t) * (size_t)njobs);
    p += sizeof(knn_job_t) * (size_t)njobs;
    std::memcpy(p, &o, sizeof(o));
    p += sizeof(o);
    std::memcpy(p, &smode, sizeof(smode));
    p += sizeof(smode);
    std::memcpy(p, &net, sizeof(void *));
    p += sizeof(void *);
    std::memcpy(p, &ws, sizeof(void *));
    return k;
}

}  // namespace

knn_status_t run_batch(knn_handle_t h, const knn_job_t *jobs, int32_t njobs, hipStream_t stream,
                       const knn_options_t *opt_in) {
    knn_options_t o{};
    o.pivot = kPivotSample;
    if (opt_in) o = *opt_in;
    const int num_cu = handle_num_cu(h);
    const uint16_t *net = handle_net(h);
    int smode = o.pivot;
    if (smode == kPivotLearned && !net) smode = kPivotSample;

    hipError_t e;
#define KTRY(call)                                                                                       \
    do {                                                                                                 \
        if ((e = (call)) != hipSuccess)                                                                  \
            return fail_msg(h, KNN_ERROR_DEVICE, std::string(#call) + ": " + hipGetErrorString(e));     \
    } while (0)

    if (o.flags & KNN_FLAG_UNFUSED) {  // one job after the other, as knn_search
        for (int32_t j = 0; j < njobs; ++j) {
            const knn_job_t &jb = jobs[j];
            if (jb.m == 0) continue;
            const bool graph = jb.queries == nullptr;  // m > 0 here
            knn_status_t st = run_search(h, graph ? jb.corpus : jb.queries, jb.m, jb.corpus, jb.n, jb.d, jb.k, graph,
                                         jb.out_dist, jb.out_idx, stream, &o);
            if (st != KNN_SUCCESS) return st;
        }
        return KNN_SUCCESS;
    }

    // cosine / Pearson: every job on unit vectors (centred for Pearson), made
    // on each call before the captured steps run
    std::vector<knn_job_t> unit_jobs;
    if (o.metric != KNN_METRIC_SQEUCLIDEAN) {
        size_t total = 0;
        for (int32_t j = 0; j < njobs; ++j)
            if (jobs[j].m > 0) total += (size_t)(jobs[j].n + (jobs[j].queries ? jobs[j].m : 0)) * (size_t)jobs[j].d;
        void *u = nullptr;
        knn_status_t us = ensure_unit_ws(h, total * sizeof(float) + 256, stream, &u);
        if (us != KNN_SUCCESS) return us;
        float *U = static_cast<float *>(u);
        const bool centre = o.metric == KNN_METRIC_PEARSON;
        unit_jobs.assign(jobs, jobs + njobs);
        size_t off = 0;
        for (int32_t j = 0; j < njobs; ++j) {
            knn_job_t &jb = unit_jobs[(size_t)j];
            if (jb.m == 0) continue;
            KTRY(launch_unit_rows(jb.corpus, jb.n, jb.d, centre, U + off, stream));
            jb.corpus = U + off;
            off += (size_t)jb.n * jb.d;
            if (jb.queries) {
                KTRY(launch_unit_rows(jb.queries, jb.m, jb.d, centre, U + off, stream));
                jb.queries = U + off;
                off += (size_t)jb.m * jb.d;
            }
        }
        jobs = unit_jobs.data();
    }

    if (!h->batch) h->batch = new BatchState();
    BatchState &b = *h->batch;
    std::vector<uint8_t> key = make_key(jobs, njobs, o, smode, net, b.ws);
    const bool timed = (o.flags & KNN_FLAG_TIMING) != 0;
    const bool want_graph = (o.flags & KNN_FLAG_NO_GRAPH) == 0;

    if (key != b.key || b.ws == nullptr) {
        // ---- plan the batch ----
        KTRY(hipDeviceSynchronize());  // earlier batches may still use the graphs and workspace
        b.drop_graphs();
        b.key.clear();
        b.jobs.clear();
        b.parts.clear();
        b.smode = smode;
        b.net = net;
        b.force = (o.flags & KNN_FLAG_FORCE_FALLBACK) ? 1 : 0;
        b.timed = timed;
        const bool tune = autotune_enabled(&o);
        // two-half operands (as large as the points themselves) for the longest
        // jobs first, and whole distance rows of the jobs with short corpora, each
        // within its budget: the rest is the workspace's and the program's
        size_t split_left = 0, direct_left = 0;
        if (!std::getenv("KNN_BATCH_QUEUE")) {
            size_t free_bytes = 0, total_bytes = 0;
            KTRY(hipMemGetInfo(&free_bytes, &total_bytes));
            const BatchBudget most = batch_budget(free_bytes + b.ws_bytes);
            split_left = most.split;
            direct_left = most.rows;
        }
        for (int32_t j = 0; j < njobs; ++j) {
            const knn_job_t &jb = jobs[j];
            BatchJob js{};
            js.graph = jb.queries == nullptr && jb.m > 0;
            js.Q = js.graph ? jb.corpus : jb.queries;
            js.C = jb.corpus;
            js.m = jb.m;
            js.n = jb.n;
            js.d = jb.d;
            js.k = jb.k;
            js.out_dist = jb.out_dist;
            js.out_idx = jb.out_idx;
            js.p = make_plan(jb.m > 0 ? jb.m : 1, jb.n, jb.d, jb.k, js.graph, &o, kRowBlock);
            js.cost = 2.0 * (double)jb.m * (double)jb.n * jb.d;
            js.oscale = o.metric != KNN_METRIC_SQEUCLIDEAN ? 0.5f : 1.0f;
            b.jobs.push_back(js);
        }
        b.order.resize(b.jobs.size());
        for (size_t j = 0; j < b.jobs.size(); ++j) b.order[j] = (int)j;
        std::stable_sort(b.order.begin(), b.order.end(),
                         [&](int x, int y) { return b.jobs[x].cost > b.jobs[y].cost; });
        const bool lowprec_pipe = o.precision != KNN_PREC_FP32 && lowprec_pipe_on() && !std::getenv("KNN_BATCH_QUEUE");
        std::vector<Plan> plain;  // the plans before split operands
        for (const BatchJob &js : b.jobs) plain.push_back(js.p);
        bool any_split = false, any_direct = false;
        auto plan_parts = [&]() {
            b.parts.clear();
            any_split = any_direct = false;
            for (int j : b.order) {
                BatchJob &js = b.jobs[j];
                js.p = plain[j];
                if (js.m == 0) continue;
                const size_t rows = (size_t)js.m * (size_t)js.n * sizeof(float);
                if (js.p.gathered && js.n <= kSampleColsMax && rows <= direct_left && dense_serves(js.p, smode)) {
                    direct_left -= rows;
                    plan_direct(js.p);
                    any_direct = true;
                }
                if (!split_pays(js.p)) continue;
                const size_t need = (size_t)(js.n + (js.graph ? 0 : js.m) + js.p.S) * (size_t)split_row_bytes(js.d);
                if (need > split_left) continue;
                split_left -= need;
                use_split(js.p);
                any_split = true;
            }
            for (int32_t j = 0; j < njobs; ++j) {
                BatchJob &js = b.jobs[j];
                js.first_part = (int)b.parts.size();
                for (int64_t i0 = 0; i0 < js.m; i0 += js.p.Mb) {
                    BatchPart pt{};
                    pt.job = j;
                    pt.i0 = i0;
                    pt.mb = js.m - i0 < js.p.Mb ? js.m - i0 : js.p.Mb;
                    pt.direct = !js.p.gathered;
                    const bool group = !(js.p.prec == kPrecF32 && js.d % 4 != 0);
                    pt.spipe = js.p.split;
                    pt.sgrouped = !pt.spipe && group;
                    pt.pipe = !pt.direct && (js.p.split || (lowprec_pipe && pt.mb > 64 && js.p.ldq <= (1 << 22)));
                    pt.grouped = !pt.direct && !pt.pipe && group;
                    b.parts.push_back(pt);
                }
                js.nparts = (int)b.parts.size() - js.first_part;
            }
        };
        plan_parts();
        if (b.parts.empty()) return KNN_SUCCESS;

        for (;;) {
            Carve sizing{nullptr};
            const size_t bytes = carve_batch(sizing, b, num_cu, tune);
            if (bytes <= b.ws_bytes) break;
            if (b.ws) {
                hipFree(b.ws);
                b.ws = nullptr;
                b.ws_bytes = 0;
            }
            if (hipMalloc(&b.ws, bytes) == hipSuccess) {
                b.ws_bytes = bytes;
                break;
            }
            b.ws = nullptr;
            (void)hipGetLastError();
            if (!any_split && !any_direct)
                return fail_msg(h, KNN_ERROR_OUT_OF_MEMORY,
                                "knn_batch_search: workspace of " + std::to_string(bytes) + " bytes");
            split_left = direct_left = 0;  // again without them
            plan_parts();
        }
        Carve real{static_cast<char *>(b.ws)};
        carve_batch(real, b, num_cu, tune);
        if (b.parts.size() > b.nflag_host_cap) {
            if (b.nflag_host) hipHostFree(b.nflag_host);
            b.nflag_host = nullptr;
            b.nflag_host_cap = 0;
            if (hipHostMalloc(&b.nflag_host, 2 * b.parts.size() * sizeof(uint32_t), hipHostMallocDefault) !=
                hipSuccess) {
                b.nflag_host = nullptr;
                (void)hipGetLastError();
                return fail_msg(h, KNN_ERROR_OUT_OF_MEMORY, "knn_batch_search: pinned host buffer");
            }
            b.nflag_host_cap = b.parts.size();
        }
        if (!b.cap_stream) KTRY(hipStreamCreateWithFlags(&b.cap_stream, hipStreamNonBlocking));

        // ---- device tables ----
        std::vector<DistArgs> table(b.parts.size());
        for (size_t pi = 0; pi < b.parts.size(); ++pi) table[pi] = part_args(b, b.parts[pi]);
        KTRY(hipMemcpyAsync(b.sh.table, table.data(), table.size() * sizeof(DistArgs), hipMemcpyHostToDevice, stream));
        std::vector<DistArgs> stable(b.parts.size());
        for (size_t pi = 0; pi < b.parts.size(); ++pi) stable[pi] = sample_args(b, b.parts[pi]);
        KTRY(hipMemcpyAsync(b.sh.stable, stable.data(), stable.size() * sizeof(DistArgs), hipMemcpyHostToDevice,
                            stream));
        std::vector<GemmItem> sitems, psitems, pitems;
        build_sample_items(b, false, sitems);
        build_sample_items(b, true, psitems);
        build_items(b, kPipeForm, pitems);
        auto upload_items = [&](GemmItem *to, const std::vector<GemmItem> &v) -> hipError_t {
            if (v.empty()) return hipSuccess;
            return hipMemcpyAsync(to, v.data(), v.size() * sizeof(GemmItem), hipMemcpyHostToDevice, stream);
        };
        KTRY(upload_items(b.sh.sitems, sitems));
        KTRY(upload_items(b.sh.psitems, psitems));
        KTRY(upload_items(b.sh.pitems, pitems));
        std::vector<SegLaunch *> launches;
        for (SegLaunch &L : b.sample_sel) launches.push_back(&L);
        launches.push_back(&b.keys_sel);
        for (SegLaunch *L : launches) {
            if (!L->rows) continue;
            KTRY(hipMemcpyAsync(L->dsegs, L->segs.data(), L->segs.size() * sizeof(SelectSeg), hipMemcpyHostToDevice,
                                stream));
            KTRY(hipMemcpyAsync(L->drow_seg, L->row_seg.data(), L->row_seg.size() * sizeof(uint32_t),
                                hipMemcpyHostToDevice, stream));
        }
        std::vector<PrepSeg> preps = prep_segs(b);
        std::vector<FlagSeg> flags;
        std::vector<CertifyArgs> certs;
        std::vector<RerankArgs> reranks;
        for (size_t pi = 0; pi < b.parts.size(); ++pi) {
            const BatchPart &pt = b.parts[pi];
            const Plan &p = b.jobs[pt.job].p;
            if (!pt.direct)
                flags.push_back(FlagSeg{pt.cnt, pt.mb, (uint32_t)p.kk, (uint32_t)p.cap, b.force, b.sh.nflag + pi,
                                        pt.flags, stats_ptr(h) + kStatCandidates});
            // (FP32 parts are certified with their re-rank)
            if (part_certified(b, pt) && p.prec != kPrecF32) certs.push_back(certify_args(b, h, pi));
            reranks.push_back(rerank_args(b, pi));
        }
        std::vector<uint32_t> fpreps, fflags, fcerts, freranks;
        b.preps = group_prep(preps, fpreps);
        b.flags = group_flags(flags, fflags);
        b.certs = group_certify(certs, fcerts);
        b.reranks = group_rerank(reranks, freranks);
        auto upload_vec = [&](void *to, const void *from, size_t bytes) -> hipError_t {
            return bytes ? hipMemcpyAsync(to, from, bytes, hipMemcpyHostToDevice, stream) : hipSuccess;
        };
        KTRY(upload_vec(b.sh.preps, preps.data(), preps.size() * sizeof(PrepSeg)));
        KTRY(upload_vec(b.sh.flags, flags.data(), flags.size() * sizeof(FlagSeg)));
        KTRY(upload_vec(b.sh.certs, certs.data(), certs.size() * sizeof(CertifyArgs)));
        KTRY(upload_vec(b.sh.reranks, reranks.data(), reranks.size() * sizeof(RerankArgs)));
        KTRY(upload_vec(b.sh.preps_first, fpreps.data(), fpreps.size() * sizeof(uint32_t)));
        KTRY(upload_vec(b.sh.flags_first, fflags.data(), fflags.size() * sizeof(uint32_t)));
        KTRY(upload_vec(b.sh.certs_first, fcerts.data(), fcerts.size() * sizeof(uint32_t)));
        KTRY(upload_vec(b.sh.reranks_first, freranks.data(), freranks.size() * sizeof(uint32_t)));
        KTRY(hipStreamSynchronize(stream));  // the host vectors above are released at scope end
        KTRY(launch_fill_u32(reinterpret_cast<uint32_t *>(b.sh.ninf), 1, 0xFF800000u, stream));
        const int prec = b.jobs[0].p.prec;
        b.tile = kTileSmall1;
        b.queue = false;
        // overrides of the default form (tests, measurements): KNN_GEMM_TILE
        // small / wide / big / small1, KNN_BATCH_QUEUE 1 / 0 (the queue form has
        // no single-stage tile: small1 runs as small there)
        if (const char *te = std::getenv("KNN_GEMM_TILE")) {
            if (!std::strcmp(te, "small1")) b.tile = kTileSmall1;
            else if (!std::strcmp(te, "small")) b.tile = kTileSmall;
            else if (!std::strcmp(te, "wide")) b.tile = kTileWide;
            else if (!std::strcmp(te, "big") && prec != kPrecFP8) b.tile = kTileBig;
        }
        if (const char *qe = std::getenv("KNN_BATCH_QUEUE")) b.queue = qe[0] == '1';
        std::vector<GemmItem> items;
        int uploaded = -1;
        auto upload = [&](int tile) -> hipError_t {
            if (tile == uploaded) return hipSuccess;
            build_items(b, tile, items);
            b.nitems = items.size();
            hipError_t ue = hipSuccess;
            if (!items.empty())
                ue = hipMemcpyAsync(b.sh.items, items.data(), items.size() * sizeof(GemmItem), hipMemcpyHostToDevice,
                                    stream);
            if (ue == hipSuccess) ue = hipStreamSynchronize(stream);  // host vectors change on the next upload
            if (ue == hipSuccess) uploaded = tile;
            return ue;
        };
        // the parts whose product takes a tile shape: neither pipelined nor selected
        // from their sample (without one there is nothing to choose)
        auto tiled = [&](const BatchPart &pt) { return !pt.pipe && !pt.direct; };
        if (tune && std::any_of(b.parts.begin(), b.parts.end(), tiled)) {
            // key: device, precision, and the work-weighted dimension and corpus
            // size and the work of those parts ("tiled": entries without it counted
            // every job, timed or not)
            double w = 0, wd = 0, wn = 0;
            for (const BatchPart &pt : b.parts) {
                if (!tiled(pt)) continue;
                const BatchJob &js = b.jobs[pt.job];
                const double cost = 2.0 * (double)pt.mb * (double)js.n * js.d;
                w += cost;
                wd += cost * js.d;
                wn += cost * (double)js.n;
            }
            const std::string tkey = "grouped|" + h->arch + "|cu" + std::to_string(num_cu) + "|p" +
                                     std::to_string(prec) + "|d" + std::to_string(size_bucket((int64_t)(wd / w))) +
                                     "|n" + std::to_string(size_bucket((int64_t)(wn / w))) + "|f" +
                                     std::to_string(size_bucket((int64_t)(w / 1e6))) + "|tiled";
            int choice = autotune_lookup(tkey);
            if (choice < 0) {
                std::vector<DistArgs> probe = table;
                for (DistArgs &a : probe) {
                    a.tau = b.sh.ninf;
                    a.tau_stride = 0;
                }
                KTRY(hipMemcpyAsync(b.sh.probe, probe.data(), probe.size() * sizeof(DistArgs), hipMemcpyHostToDevice,
                                    stream));
                KTRY(hipStreamSynchronize(stream));
                // every tile shape, as one workgroup per item (c) and as a
                // resident grid over the per-XCD queues (c + kQueueChoice)
                // the default (single-stage 128 x 128, one workgroup per item)
                // first, kept unless another form is more than 3 % faster: the
                // probes keep nothing (threshold -inf), and the candidate writes
                // they leave out favour the default's more resident workgroups
                // per CU (512-job batch: probes tied, real calls 4 % faster)
                std::vector<int> cands = {kTileSmall1, kTileSmall, kTileWide};
                if (prec != kPrecFP8) cands.push_back(kTileBig);
                const size_t nshape = cands.size();
                for (size_t i = 1; i < nshape; ++i) cands.push_back(cands[i] + kQueueChoice);
                auto run = [&](int c) -> hipError_t {
                    const int tile = c % kQueueChoice;
                    hipError_t re = upload(tile);
                    if (re == hipSuccess) re = enqueue_product(b, b.sh.probe, tile, c >= kQueueChoice, num_cu, stream);
                    return re;
                };
                KTRY(autotune_pick(tkey, cands, run, stream, 2, &choice, 0.03f));
            }
            b.tile = choice % kQueueChoice;
            b.queue = choice >= kQueueChoice;
        }
        KTRY(upload(b.tile));

        // ---- graphs: prep (+ product + flags), then final ----
        b.eager = true;
        if (want_graph) {
            std::vector<hipGraphExec_t> gs;
            hipGraphExec_t g = nullptr;
            bool ok = true;
            // one graph for the whole call (two around the timed product); rows
            // flagged for the exact fallback come out of it with provisional
            // results, re-done eagerly afterwards
            if (timed) {
                ok = capture(b, [&](hipStream_t s) { return enqueue_prep(b, num_cu, s); }, &g) == hipSuccess;
                if (ok) gs.push_back(g);
                ok = ok && capture(b, [&](hipStream_t s) {
                               hipError_t ce = enqueue_flags(b, h, s);
                               if (ce == hipSuccess) ce = enqueue_final(b, num_cu, s);
                               return ce;
                           }, &g) == hipSuccess;
                if (ok) gs.push_back(g);
            } else {
                ok = capture(b, [&](hipStream_t s) {
                         hipError_t ce = enqueue_prep(b, num_cu, s);
                         if (ce == hipSuccess) ce = enqueue_product(b, b.sh.table, b.tile, b.queue, num_cu, s);
                         if (ce == hipSuccess) ce = enqueue_flags(b, h, s);
                         if (ce == hipSuccess) ce = enqueue_final(b, num_cu, s);
                         return ce;
                     }, &g) == hipSuccess;
                if (ok) gs.push_back(g);
            }
            if (ok) {
                b.graphs = gs;
                b.eager = false;
            } else {
                for (hipGraphExec_t x : gs) hipGraphExecDestroy(x);  // capture failed: eager steps
            }
        }
        b.key = make_key(jobs, njobs, o, smode, net, b.ws);
    }

    // ---- run ----
    int64_t rows = 0;
    for (const BatchJob &js : b.jobs) rows += js.m;
    ProductTimer timer;
    KTRY(timer.init(timed));
    double flops = 0;
    for (const BatchJob &js : b.jobs) flops += js.cost;
    if (b.eager) {
        KTRY(enqueue_prep(b, num_cu, stream));
        KTRY(timer.begin(stream, flops));
        KTRY(enqueue_product(b, b.sh.table, b.tile, b.queue, num_cu, stream));
        KTRY(timer.end(stream));
        KTRY(enqueue_flags(b, h, stream));
        KTRY(enqueue_final(b, num_cu, stream));
    } else if (timed) {
        KTRY(hipGraphLaunch(b.graphs[0], stream));
        KTRY(timer.begin(stream, flops));
        KTRY(enqueue_product(b, b.sh.table, b.tile, b.queue, num_cu, stream));
        KTRY(timer.end(stream));
        KTRY(hipGraphLaunch(b.graphs[1], stream));
    } else {
        KTRY(hipGraphLaunch(b.graphs[0], stream));
    }
    // the flag and uncertified-row counts reach the host here (one
    // synchronisation per call)
    KTRY(hipStreamSynchronize(stream));
    KTRY(timer.collect(h));
    int64_t fallback = 0;
    for (size_t pi = 0; pi < b.parts.size(); ++pi) fallback += b.nflag_host[pi];
    if (fallback > 0) {
        // rare: the flagged rows' candidate lists are re-done exactly, then the
        // selection, certificate and re-rank of the parts holding them run again
        int64_t done = 0;
        KTRY(run_fallback(b, num_cu, stream, &done));
        for (size_t pi = 0; pi < b.parts.size(); ++pi)
            if (b.nflag_host[pi] > 0) KTRY(refinal_part(b, h, num_cu, pi, stream));
        KTRY(hipStreamSynchronize(stream));
    }
    int64_t rerun = 0;
    if (b.jobs[0].p.prec == kPrecF32) KTRY(run_rerun(b, stream, &rerun));
#undef KTRY
    add_host_stats(h, rows, fallback);
    add_host_rerun(h, rerun);
    for (const BatchJob &js : b.jobs)
        if (js.p.stored) add_host_candidates(h, js.m * js.p.kk);
    return KNN_SUCCESS;
}

}  // namespace knn
