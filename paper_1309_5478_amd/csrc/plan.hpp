// Per-call plan and workspace layout of the search / graph path (shared by the
// single-call and the batched entry points).
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstdint>

#include "dist.hpp"
#include "internal.hpp"
#include "knn.h"

namespace knn {

void add_product_time(knn_handle_t h, double ms, double flops);

// Bump allocator over one workspace buffer (sizing pass with base == nullptr).
struct Carve {
    char *base;
    size_t off = 0;
    template <class T>
    T *take(size_t count) {
        off = (off + 255) & ~size_t(255);
        T *p = reinterpret_cast<T *>(base ? base + off : nullptr);
        off += count * sizeof(T);
        return p;
    }
};

constexpr int kSampleCols = 2048;
constexpr int kSampleColsMax = 16384;
constexpr int64_t kRowBlock = 32768;
// split operands of the corpus held at a time (a larger corpus passes in blocks
// of columns, split again for every block of rows: 8 bytes moved per element
// against 2 Mb flops)
constexpr size_t kSplitBytes = size_t(8) << 30;
constexpr size_t kDenseBytes = size_t(1) << 30;  // materialised distance block budget
// A batch holds the operands and the stored rows of all its jobs at once, and
// keeps them for its replays: at most this much of each, and a third and a sixth
// of what is free when it is planned (512 jobs with 101 GB of corpora want 105 and 4.3
// GiB, and have about 55 and 4.3 beside them).
constexpr size_t kBatchSplitBytes = size_t(64) << 30, kBatchRowBytes = size_t(8) << 30;

struct Plan {
    int64_t m, n, n_eff;
    int d, k, kk;
    int prec;          // kPrecF32 / kPrecBF16 / kPrecFP8
    int64_t ldq;       // bytes per quantised row
    float rel;         // relative dot-product error bound of the precision
    float gamma;       // relative error bound of an FP32 reduction over d terms
    bool graph, unfused;
    int force;
    int force_rerun;
    bool stored;       // keys stored and selected from where the corpus is larger than its sample: k' candidates a row
    bool few;          // a few queries: their distance rows stored in one pass over the corpus (with unfused)
    bool split;        // FP32 product on two-half operands (ldq: bytes per split row)
    int64_t Nb;        // corpus points whose operands are held at a time
    // fused
    int S;
    bool gathered;
    int r;
    int cap;
    int64_t Mb;
    int64_t Fb;
    // unfused
    int64_t Mu;
};

struct Bufs {
    float *cnorm = nullptr;
    float *qn2 = nullptr;
    unsigned int *cmax2 = nullptr;
    void *Cq = nullptr, *Qq = nullptr, *Csq = nullptr, *Qfq = nullptr;
    float *cs = nullptr, *qs = nullptr, *css = nullptr, *qfs = nullptr;
    float *Cs = nullptr, *csn = nullptr;
    float *Ds = nullptr, *tv = nullptr;
    int32_t *ti = nullptr;
    uint32_t *cnt = nullptr;
    uint64_t *cand = nullptr;
    int32_t *flags = nullptr;
    uint32_t *nflag = nullptr;
    float *sv = nullptr;
    int32_t *si = nullptr;
    float *Qf = nullptr, *Df = nullptr, *fv = nullptr;
    int32_t *fi = nullptr;
    float *Dm = nullptr;
    int32_t *ulist = nullptr;  // uncertified rows of the current block (FP32 re-run)
    uint32_t *nu = nullptr;
    float *tfix = nullptr;
    void *selws = nullptr;
    size_t selws_bytes = 0;
    float *ninf = nullptr;  // one -inf: threshold of the tile-timing launches
};

// Workspace of a dense selection that splits its rows (0: none of them does).
inline size_t dense_split_bytes(int64_t rows, int64_t cols, int k, int num_cu) {
    size_t need = 0;
    for (const bool sample : {false, true}) {
        const SplitPlan sp = select_split_plan(rows, (uint32_t)cols, (uint32_t)k, num_cu, false, sample);
        if (sp.parts > 1) need = std::max(need, select_split_ws_bytes(sp, rows, (uint32_t)k));
    }
    return need;
}

inline size_t carve(Carve &c, const Plan &p, Bufs &b, int num_cu) {
    b.cnorm = c.take<float>(p.n);
    b.qn2 = c.take<float>(p.m);
    if (p.prec != kPrecF32) {
        b.Cq = c.take<char>((size_t)p.n * p.ldq);
        b.cs = c.take<float>(p.n);
        if (!p.graph) {
            b.Qq = c.take<char>((size_t)p.m * p.ldq);
            b.qs = c.take<float>(p.m);
        }
        if (!p.unfused) {
            b.Csq = c.take<char>((size_t)p.S * p.ldq);
            b.css = c.take<float>(p.S);
            b.Qfq = c.take<char>((size_t)p.Fb * p.ldq);
            b.qfs = c.take<float>(p.Fb);
        }
    }
    if (p.split) {
        b.Cq = c.take<char>((size_t)p.Nb * p.ldq);
        b.cs = c.take<float>(p.Nb);
        if (!p.graph || p.Nb < p.n) {
            b.Qq = c.take<char>((size_t)p.Mb * p.ldq);
            b.qs = c.take<float>(p.Mb);
        }
        b.Csq = c.take<char>((size_t)p.S * p.ldq);
        b.css = c.take<float>(p.S);
    }
    size_t selws = 0;
    {
        const int64_t rows = p.unfused ? p.Mu : p.Mb;
        b.ulist = c.take<int32_t>((size_t)rows);
        b.tfix = c.take<float>((size_t)rows);
    }
    if (p.unfused) {
        b.Dm = c.take<float>((size_t)p.Mu * p.n);
        b.sv = c.take<float>((size_t)p.Mu * p.kk);
        b.si = c.take<int32_t>((size_t)p.Mu * p.kk);
        int cap = select_cap_for_k(p.kk);
        selws = select_ws_bytes(cap, (uint32_t)p.n, select_grid(cap, p.Mu, num_cu));
        selws = std::max(selws, dense_split_bytes(p.Mu, p.n, p.kk, num_cu));
    } else {
        if (p.gathered) {
            b.Cs = c.take<float>((size_t)p.S * p.d);
            b.csn = c.take<float>(p.S);
        }
        b.Ds = c.take<float>((size_t)p.Mb * p.S);
        b.tv = c.take<float>((size_t)p.Mb * (p.r + 1));
        b.ti = c.take<int32_t>((size_t)p.Mb * (p.r + 1));
        b.cnt = c.take<uint32_t>(p.Mb);
        b.cand = c.take<uint64_t>((size_t)p.Mb * p.cap);
        b.flags = c.take<int32_t>(p.Mb);
        b.sv = c.take<float>((size_t)p.Mb * p.kk);
        b.si = c.take<int32_t>((size_t)p.Mb * p.kk);
        b.Qf = c.take<float>((size_t)p.Fb * p.d);
        b.Df = c.take<float>((size_t)p.Fb * p.n);
        b.fv = c.take<float>((size_t)p.Fb * p.kk);
        b.fi = c.take<int32_t>((size_t)p.Fb * p.kk);
        int cap1 = select_cap_for_k(p.r + 1);
        size_t w1 = select_ws_bytes(cap1, (uint32_t)p.S, select_grid(cap1, p.Mb, num_cu));
        int cap2 = select_cap_for_k(p.kk);
        size_t w2 = select_ws_bytes(cap2, (uint32_t)p.n, select_grid(cap2, p.Fb, num_cu));
        // (fallback rows are few as a rule)
        selws = std::max(std::max(w1, w2), dense_split_bytes(p.Fb < 8 ? p.Fb : 8, p.n, p.kk, num_cu));
    }
    b.selws_bytes = selws < 256 ? 256 : selws;
    b.selws = c.take<char>(b.selws_bytes);
    b.ninf = c.take<float>(1);
    return c.off;
}

// Optional HIP-event timing of the main distance-product launches.
struct ProductTimer {
    bool on = false;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    double flops = 0;
    bool pending = false;
    ~ProductTimer() {
        if (e0) hipEventDestroy(e0);
        if (e1) hipEventDestroy(e1);
    }
    hipError_t init(bool enable) {
        on = enable;
        if (!on) return hipSuccess;
        hipError_t e = hipEventCreate(&e0);
        if (e == hipSuccess) e = hipEventCreate(&e1);
        return e;
    }
    hipError_t begin(hipStream_t s, double f) {
        if (!on) return hipSuccess;
        flops = f;
        pending = true;
        return hipEventRecord(e0, s);
    }
    hipError_t end(hipStream_t s) { return on ? hipEventRecord(e1, s) : hipSuccess; }
    // after the stream has been synchronised past end()
    hipError_t collect(knn_handle_t h) {
        if (!on || !pending) return hipSuccess;
        float ms = 0;
        hipError_t e = hipEventElapsedTime(&ms, e0, e1);
        if (e == hipSuccess) add_product_time(h, ms, flops);
        pending = false;
        return e;
    }
};

// The k smallest of every row, too few long rows for one workgroup each in
// parts where the workspace has room for them.
inline hipError_t select_dense(const float *D, int64_t rows, int64_t cols, int64_t ld, int k, float *ov, int32_t *oi,
                               void *ws, size_t ws_bytes, int num_cu, int mode, const uint16_t *net, hipStream_t stream) {
    SelectArgs a{};
    a.dist = D;
    a.rows = rows;
    a.cols = (uint32_t)cols;
    a.ld = ld;
    a.k = (uint32_t)k;
    a.out_val = ov;
    a.out_idx = oi;
    a.mode = mode;
    a.net = mode == kPivotLearned ? net : nullptr;
    const SplitPlan sp = select_split_plan(rows, (uint32_t)cols, (uint32_t)k, num_cu, false, mode == kPivotSample);
    if (sp.parts > 1 && select_split_ws_bytes(sp, rows, (uint32_t)k) <= ws_bytes)
        return launch_select_split(a, sp, ws, num_cu, stream);
    int cap = select_cap_for_k((uint32_t)k);
    return launch_select(a, cap, select_grid(cap, rows, num_cu), ws, stream);
}

// Whether two-half operands (gemm_pipe.hip) serve an FP32 plan's products: where
// they are at least as exact as the FP32 matrix instruction (d >= 64, measured
// there) and pay, from 128 rows on (making the operands moves 8 bytes per corpus
// element, about what 150 rows of the FP32 product take).  Only the filtered
// path: a corpus no larger than its sample is too small.  KNN_GEMM_SPLIT=0 turns
// it off, and so does a tile of the FP32 product asked for by KNN_GEMM_TILE.
inline bool split_pays(const Plan &p) {
    if (p.prec != kPrecF32 || p.d < 64 || p.m < 128 || split_row_bytes(p.d) > (1 << 22)) return false;
    if (const char *e = std::getenv("KNN_GEMM_SPLIT"))
        if (e[0] == '0') return false;
    return std::getenv("KNN_GEMM_TILE") == nullptr;
}
inline bool split_serves(const Plan &p) { return p.gathered && !p.unfused && split_pays(p); }
inline void use_split(Plan &p) {
    p.split = true;
    p.ldq = split_row_bytes(p.d);
    // Both operands are within 2^-23 of themselves, and low x low is left out: 2^-21.
    // The sums: one instruction adds 16 products to its accumulator with an error
    // of at most 2 u + u / 2 per product that is not zero, of the sum of all their
    // magnitudes (products are cut where they lie 25 bits below the largest term;
    // over 4 10^8 sums of one to 16 products, of every sign, spread and ratio to
    // the accumulator up to 2^30: at most 2.0 u of one product, 5.4 u of 16); three
    // products per element, three instructions per 16 elements.  (The product's
    // own error against FP64, on points made for it, one large element over small
    // ones at the cut: 0.17 of this bound at d = 65, 0.08 from d = 300 to 4096.)  That is less than
    // twice the FP32 instruction's gamma; the certificate (RerankArgs) asks for no
    // more than the gap of two keys of that one did: points of a mean far above
    // their spread keep theirs (32768 uniform points in [8, 9)^128: with 3 gamma and the
    // gap of two keys 32070 rows re-run, 7.4 ms, this way 6, 1.7 ms; in [4, 5)^1024 all
    // rows either way, 286 and 38 ms, and 65 with the FP32 instruction and that gap).
    p.rel = (float)(std::ldexp(1.0, -21) + std::ldexp(1.5 * p.d + 6.0 * ((p.d + 15) / 16), -24));
}

// Bytes of operands held at a time that the environment asks for (KNN_SPLIT_BYTES), or 0.
inline size_t split_bytes_asked() {
    const char *e = std::getenv("KNN_SPLIT_BYTES");
    const long long v = e ? std::atoll(e) : 0;
    return v > 0 ? (size_t)v : 0;
}
// What a batch may take for its jobs' operands and stored rows.
struct BatchBudget {
    size_t split, rows;
};
inline BatchBudget batch_budget(size_t free_bytes) {
    const size_t asked = split_bytes_asked(), split = std::min(free_bytes / 3, kBatchSplitBytes);
    return BatchBudget{asked ? std::min(asked, split) : split, std::min(free_bytes / 6, kBatchRowBytes)};
}

// The single call's choice: also once there is work for the large tiles
// (pipe_fills in gemm_pipe.hip).
inline void plan_split(Plan &p) {
    const int64_t bytes = split_row_bytes(p.d);
    if (!split_serves(p) || !pipe_fills(p.m < p.Mb ? p.m : p.Mb, p.n)) return;
    const size_t asked = split_bytes_asked();
    int64_t nb = (int64_t)((asked ? asked : kSplitBytes) / (size_t)bytes) / 256 * 256;
    if (nb < 256) nb = 256;
    p.Nb = nb < p.n ? nb : p.n;
    use_split(p);
}

// A few FP32 queries: their distance rows in one pass over the corpus (few.hip),
// selected as on the unfused path.  Up to 3 d rows, or 2^25 keys: more of them
// cost more than the corpus (the fused path / this one, n = 10^6, k = 10: d = 32,
// m = 96 356 / 327 us, m = 127 359 / 392; d = 24, m = 72 337 / 280; small corpora
// gain with any m).
inline void plan_few(Plan &p) {
    if (p.prec != kPrecF32 || p.graph || p.unfused || p.force || std::getenv("KNN_GEMM_TILE")) return;
    if (const char *e = std::getenv("KNN_FEW"))
        if (e[0] == '0') return;
    if (!p.gathered && p.m > 16) return;  // (2000 x 512: m = 16 94 / 58 us, m = 100 96 / 115)
    if (few_passes(p.m, p.d) == 0 || (p.m > 3 * (int64_t)p.d && p.m * p.n > (1 << 25))) return;
    if ((size_t)p.m * (size_t)p.n * sizeof(float) > kDenseBytes) return;
    p.few = p.unfused = true;
    p.stored = p.gathered;
    p.Mu = p.m;
}

// Corpora short enough that storing the distance rows and selecting from them
// costs less than the threshold sample, its selection, the candidate lists and a
// second product; as on the unfused path, the FP32 product on two-half operands.
// A stored key is written and read once, about 1.8 ps; what it replaces grows
// with the lists: up to 8192 + 40 kk points, and 20000 + 150 kk for FP32 rows too
// short for two-half operands, whose filter pass costs more (fused / this, us.
// 16384 queries, FP32 d = 128: kk = 128 n = 12000 684 / 644, 24000 833 / 1137; kk = 512
// 24000 1441 / 1358, 40000 1847 / 2032; kk = 1000 40000 2839 / 2357, 64000 2902 / 3263;
// BF16 d = 512: kk = 128 12000 1028 / 977, kk = 256 12000 1655 / 1419, 24000 1904 / 2084;
// FP32 d = 32: kk = 128 40000 1606 / 1439, 64000 2031 / 2285.  Graphs, FP32 d = 128:
// kk = 16 n = 4096 163 / 106, 8192 251 / 215, 16000 505 / 603; kk = 64 201 / 114, 290 /
// 233, 582 / 676; kk = 1024, n = 3000 1181 / 250).  The plain pivot rule reads long
// rows many times: 4096 points (kk = 32, n = 3000 223 / 170, 8192 378 / 448).  A
// corpus that is its own sample is stored anyway; it gains only the two-half
// product, from about 128 tiles on (20000 x 2000, d = 512 576 / 349; 2000 x 2000,
// d = 128 82 / 85).
inline bool dense_serves(const Plan &p, int smode) {
    if (p.unfused || p.force || std::getenv("KNN_GEMM_TILE")) return false;
    if (const char *e = std::getenv("KNN_DENSE"))
        if (e[0] == '0') return false;
    const int64_t most = smode == kPivotPlain             ? 4096
                         : p.prec == kPrecF32 && p.d < 64 ? std::min(20000 + 150 * p.kk, 65536)
                                                          : 8192 + 40 * p.kk;
    return p.n <= most;
}
inline void plan_dense(Plan &p, int smode) {
    if (!dense_serves(p, smode)) return;
    const bool split = split_pays(p) && pipe_fills(p.m, p.n);
    if (!p.gathered && (!split || ((p.m + 255) / 256) * ((p.n + 255) / 256) < 128)) return;
    if (split) use_split(p);  // (the operands of the whole corpus: Nb = n)
    const int64_t mu = (int64_t)(kDenseBytes / sizeof(float) / (size_t)p.n);
    p.Mu = mu < p.m ? mu : p.m;
    p.Mb = p.Mu;
    p.unfused = true;
    p.stored = p.gathered;
}

// The same in a batch, whose jobs keep their sample distances: the sample is the
// whole corpus.
inline void plan_direct(Plan &p) {
    p.S = (int)p.n;
    p.gathered = false;
    p.stored = true;
    p.r = p.kk - 1;
}

// The plan of one search / graph call: candidate oversampling, threshold sample,
// list capacity, row blocking.  Mb_limit caps the rows per block.
inline Plan make_plan(int64_t m, int64_t n, int d, int k, bool graph, const knn_options_t *opt, int64_t Mb_limit) {
    Plan p{};
    p.m = m;
    p.n = n;
    p.n_eff = graph ? n - 1 : n;
    p.d = d;
    p.k = k;
    p.graph = graph;
    p.Nb = n;
    int over = opt && opt->oversample > 0 ? opt->oversample : 4;
    int64_t kk = (int64_t)k * over;
    if (kk > kSelectMaxK) kk = kSelectMaxK;
    if (kk < k) kk = k;
    if (kk > p.n_eff) kk = p.n_eff;
    p.kk = (int)kk;
    p.unfused = opt && (opt->flags & KNN_FLAG_UNFUSED);
    p.force = (opt && (opt->flags & KNN_FLAG_FORCE_FALLBACK)) ? 1 : 0;
    p.force_rerun = (opt && (opt->flags & KNN_FLAG_FORCE_RERUN)) ? 1 : 0;
    p.prec = opt ? opt->precision : KNN_PREC_FP32;
    {
        const int dq = (d + kQuantPad - 1) / kQuantPad * kQuantPad;
        p.ldq = (int64_t)dq * (p.prec == kPrecBF16 ? 2 : 1);
        const double gamma = d * std::ldexp(1.0, -24) / (1.0 - d * std::ldexp(1.0, -24));
        const double u = p.prec == kPrecBF16 ? std::ldexp(1.0, -8) : (p.prec == kPrecFP8 ? std::ldexp(1.0, -4) : 0.0);
        p.rel = (float)(2 * u + u * u + gamma);
        p.gamma = (float)gamma;
    }
    if (p.unfused) {
        int64_t mu = (int64_t)(kDenseBytes / sizeof(float) / (size_t)n);
        p.Mu = mu < 1 ? 1 : (mu > m ? m : mu);
    } else {
        // sample columns: at least 2 n / kk (from 2048 up to 16384), and more while the
        // expected survivors of the threshold would exceed half the largest list
        // capacity, so that the candidate lists stay a few kk long and rarely overflow
        auto rank_for = [&](int64_t S, double &expected) -> int {
            if (n <= S) {
                expected = (double)p.kk;
                return p.kk - 1;  // the sample is the whole corpus (own index excluded)
            }
            const double mu = (double)S * p.kk / (double)p.n_eff;
            int64_t ri = (int64_t)std::ceil(mu + 3.0 * std::sqrt(mu) + 4.0);
            if (ri > S - 1) ri = S - 1;
            if (ri > kSelectMaxK - 1) ri = kSelectMaxK - 1;
            expected = (double)(ri + 1) * (double)p.n_eff / (double)S;
            return (int)ri;
        };
        int64_t S = kSampleCols;
        double expected = 0;
        for (;;) {
            rank_for(S, expected);
            const bool enough = S * p.kk >= 2 * n && 2.0 * expected <= kSelectKeysCap;
            if (enough || S >= kSampleColsMax || S >= n) break;
            S *= 2;
        }
        // then more sample columns while they cost less than the candidates
        // they save: with a small expected sample rank the margin above it lets
        // several kk through.  A kept candidate (its slot reservation and key
        // write in the product, its share of the candidate selection) costs
        // about 0.19 ns of the device with the tiles of gemm.hip (measured on
        // the 2^20 x 256 BF16 graph), 0.048 with the pipelined product; a
        // sample column costs, per row, its share of the sample product (2 d
        // flops) and a written and re-read distance, and above 8192 columns of
        // a selection that fewer rows share a CU for.  Pipelined, d = 256,
        // 262144 points, ms at 2048 / 4096 / 8192 / 16384 columns: FP8 kk = 256 53.0 /
        // 49.5 / 47.8 / 50.5, kk = 64 40.7 / 36.9 / 34.9 / 37.2, BF16 kk = 256 62.7 / 59.9 /
        // 59.4 / 62.3; 131072 x 1024, kk = 128: BF16 48.2 / 47.7 / 48.9 / 51.9, FP8 30.6 /
        // 30.0 / 30.7 / 33.5; FP32 131072 x 128, kk = 64 15.9 / 15.7 / 15.4 / 17.2.
        {
            const bool pipe = pipe_fills(m, n) && (p.prec != kPrecF32 || (d >= 64 && m >= 128));
            const double t_keep = pipe ? 4.8e-11 : 1.9e-10;
            const double flops = p.prec != kPrecF32 ? (pipe ? 8.0e14 : 6.0e14) : (pipe ? 4.2e14 : 1.25e14);
            while (2 * S <= kSampleColsMax && 2 * S < n) {
                const double t_col = 2.0 * d / flops + (pipe ? (S < 8192 ? 3.0e-13 : 1.3e-12) : 2.0e-12);
                double e2 = 0;
                rank_for(2 * S, e2);
                if (2.0 * e2 > kSelectKeysCap) break;
                if ((expected - e2) * t_keep <= (double)S * t_col) break;
                S *= 2;
                expected = e2;
            }
        }
        if (const char *e = std::getenv("KNN_SAMPLE_COLS")) {
            const long v = std::atol(e);
            if (v >= 64 && v <= 65536) S = v;
        }
        p.S = n < S ? (int)n : (int)S;
        p.gathered = n > p.S;
        p.r = rank_for(p.S, expected);
        // the survivor count varies with the sample's order statistic (relative
        // spread about 1 / sqrt(r + 1)): three times the expectation keeps
        // overflows (rows re-done exactly) rare
        int64_t cap = (int64_t)(3.0 * expected);
        if (cap < p.kk + 64) cap = p.kk + 64;
        cap = (cap + 63) / 64 * 64;
        if (cap > kSelectKeysCap) cap = kSelectKeysCap;
        p.cap = (int)cap;
        p.Mb = m < kRowBlock ? m : kRowBlock;
        if (p.Mb > Mb_limit) p.Mb = Mb_limit;
        int64_t fb = (int64_t)((size_t(256) << 20) / sizeof(float) / (size_t)n);
        p.Fb = fb < 1 ? 1 : (fb > p.Mb ? p.Mb : fb);
    }
    return p;
}

}  // namespace knn
