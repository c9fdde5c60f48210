// Host/device interface of the distance kernels (dist.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

namespace knn {

enum : int { kEpiDense = 0, kEpiFilter = 1 };
// (kPrecSplit: FP32 operands as two FP16 halves, see gemm_pipe.hip; a form of the
// operands inside the library, not a caller's precision)
enum : int { kPrecF32 = 0, kPrecBF16 = 1, kPrecFP8 = 2, kPrecSplit = 3 };
enum : int { kTileSmall = 0, kTileWide = 1, kTileBig = 2, kTileSmall1 = 3, kTilePipe = 4 };

// Quantised operands (BF16 / FP8): rows padded with zeros to a multiple of
// kQuantPad elements, so every 128-byte k-chunk load is in bounds.
constexpr int kQuantPad = 128;
// Split operands: rows of 128-byte chunks, each the high halves of 32 elements
// and then their low halves, zero-padded to a whole chunk.
inline int64_t split_row_bytes(int d) { return ((int64_t)d + 31) / 32 * 128; }

struct DistArgs {
    const float *Q;        // m x d queries
    int64_t m;
    const float *C;        // n x d corpus
    int64_t n;
    int d;
    const float *cnorm;    // n squared norms of the corpus rows
    const float *qnorm;    // kEpiDense only: if set, ||q_i||^2 is added (full squared distance)
    // self exclusion: when self_offset >= 0, query row i has global id
    // self_offset + (row_ids ? row_ids[i] : i) and corpus column j == that id is excluded
    int64_t self_offset;
    const int32_t *row_ids;
    // kEpiDense: d' into out (row stride ldo); excluded entries get +inf
    float *out;
    int64_t ldo;
    // kEpiFilter: keep d' <= tau[i * tau_stride]; append keys to cand[i * cap + ...]
    const float *tau;
    int64_t tau_stride;
    uint32_t *cnt;
    uint64_t *cand;
    int cap;
    // operand precision; for BF16 / FP8 / split operands the product reads Qq / Cq
    // (row stride ldq bytes) and, for FP8 and split ones, undoes the per-row
    // power-of-two scales qscale_i * cscale_j in the epilogue
    int prec;
    const void *Qq;
    const void *Cq;
    int64_t ldq;
    const float *qscale;
    const float *cscale;
    // tile shape (kTile*; kTilePipe: the pipelined product where it serves), or -1
    // for the default choice
    int tile = -1;
    // FILTER on the pipelined product only: corpus index of column 0 (the corpus
    // passes in blocks of columns)
    int64_t col_base = 0;
    // filled by the launcher
    uint32_t tiles_m, tiles_n;
};

struct RerankArgs {
    const float *Q;         // m x d
    int64_t m;
    const float *C;         // corpus, n x d
    int64_t n;
    int d;
    const int32_t *cidx;    // m x kk candidate corpus indices
    uint32_t kk;
    int k;
    float *out_dist;        // m x k
    int32_t *out_idx;       // m x k
    int64_t self_offset = -1;  // >= 0: row i's own corpus index self_offset + i is never returned
    float out_scale = 1.0f;    // returned distance = out_scale * the direct-form sum (a power of two)
    // Optional (FP32 products): the candidates' ascending reduced keys (m x kk)
    // and what bounds their error (as CertifyArgs).  Candidates whose key lies so
    // far above the k-th that neither the keys' nor the direct form's rounding
    // can bring them among the k smallest are not read.
    const float *keys = nullptr;
    const float *qnorm2 = nullptr;
    const unsigned int *cmax2_bits = nullptr;
    float rel = 0.f, gamma = 0.f;
    // With keys, optional: the certificate of every row, in the same launch.  E and
    // E' are CertifyArgs' bound with rel and with rel_fix (of the keys that a re-run
    // reads).  Every one of the k nearest has an exact key of at most
    //   U = min(key_k + E, D / (1 - gamma') - |q|^2 (1 - gamma)),
    // D the k-th direct-form distance among the candidates and gamma' that form's
    // error, and every point outside the candidates one of at least key_kk - E.  A
    // row with key_kk - E <= U is appended to ulist (count in *nu), with the bound U +
    // E' of what a re-run has to look at in tfix (NaN or infinite: everything).
    // The second bound of U needs E once where the gap of two keys needs it twice,
    // and decides where |q| is near max |c|: points far from the origin.
    int32_t *ulist = nullptr;
    uint32_t *nu = nullptr;
    float *tfix = nullptr;
    int force = 0;             // list every row
    float rel_fix = 0.f;
};

hipError_t launch_dist_gemm(const DistArgs &a, int epi, hipStream_t stream);

// ---- grouped product (batches) ---------------------------------------------
struct GemmItem {
    uint32_t job, tm, tn;
};
// Rows x columns of a tile shape (kTile*).
void gemm_tile_dims(int tile, int *bm, int *bn);
// One workgroup per item: jobs is a device array of DistArgs (tiles_m /
// tiles_n / tile unused), items a device array of nitems tiles of the shape
// `tile`, in dispatch order (item b runs on XCD b % 8).  FP32 jobs need
// d % 4 == 0.  The DENSE epilogue only with the small tile.
hipError_t launch_dist_gemm_grouped(const DistArgs *jobs, const GemmItem *items, int64_t nitems, int prec, int tile,
                                    hipStream_t stream, int epi = kEpiFilter);
// The same items (FILTER epilogue) taken by a resident grid from eight per-XCD
// atomic queues instead of one workgroup per item; `queues` is 8 uint32 of
// device memory (cleared by the launch).
hipError_t launch_dist_gemm_queue(const DistArgs *jobs, const GemmItem *items, int64_t nitems, int prec, int tile,
                                  uint32_t *queues, int num_cu, hipStream_t stream);
// The pipelined product over a list of 256 x 256 tiles of many products (split
// operands; BF16 and FP8 with the FILTER epilogue): as launch_dist_gemm_grouped,
// ldq at most 2^22 and no qnorm / row_ids.
constexpr int kPipeTileDim = 256;
hipError_t launch_dist_gemm_pipe_grouped(const DistArgs *jobs, const GemmItem *items, int64_t nitems, int prec,
                                         hipStream_t stream, int epi = kEpiFilter);
// The 256 x 256 tiles pay from about 24 of them on, for more than 64 rows
// (whole searches, 128 x 128 tiles / these; d = 256: BF16 256 x 3000 118 / 123 us,
// 128 x 6000 131 / 120, 100 x 40000 218 / 170, 1000 x 10000 170 / 153; FP8 256 x
// 3000 125 / 127, 256 x 6000 143 / 132, 1000 x 40000 273 / 210; halves, from 128
// rows on, 1000 x 10000 213 / 194, d = 1024 418 / 290; 128 x 40000, d = 256, 246 /
// 249).  Of at most 64 rows the 256-row tile wastes more than it gains once the
// corpus is long: 64 x 10^6, d = 1024, BF16 2753 / 2910.
inline bool pipe_fills(int64_t m, int64_t n) {
    return m > 64 && ((m + kPipeTileDim - 1) / kPipeTileDim) * ((n + kPipeTileDim - 1) / kPipeTileDim) >= 24;
}
// The pipelined product on 256 x 256 tiles (gemm_pipe.hip): whether it serves `a`
// (KNN_GEMM_PIPE=0 turns it off for BF16 and FP8), and its launch.
// launch_dist_gemm uses it where it applies.
bool gemm_pipe_applies(const DistArgs &a, int epi);
bool lowprec_pipe_on();  // (not turned off, and no tile of gemm.hip asked for by KNN_GEMM_TILE)
hipError_t launch_dist_gemm_pipe(const DistArgs &a, int epi, hipStream_t stream);
// The distance rows of a few FP32 queries (few.hip): out (m x n) = the reduced
// keys, with the queries' squared norms and, folded into max_bits (zero or a
// smaller value at launch), the largest corpus norm.  few_passes(m, d) must not
// be 0.
constexpr int kFewRows = 127;
constexpr int kFewPasses = 3;
constexpr size_t kFewLds = 156u << 10;
inline size_t few_lds_bytes(int tiles, int d) {  // of 16 queries each
    return (size_t)tiles * 16 * (((size_t)d + 15) / 16 * 16 + 4) * sizeof(float);
}
// Query tiles per pass over the corpus: as many as LDS holds.
inline int few_tiles(int64_t m, int d) {
    int tiles = m <= 16 ? 1 : (m <= 32 ? 2 : (m <= 64 ? 4 : 8));
    while (tiles > 1 && few_lds_bytes(tiles, d) > kFewLds) tiles /= 2;
    return tiles;
}
// Passes over the corpus, 0 where another path serves better (the fused path /
// this one, 200000 x 768: m = 33 in two passes 653 / 385 us, m = 64 663 / 410, m =
// 100 in four 664 / 749).
inline int few_passes(int64_t m, int d) {
    if (m < 1 || m > kFewRows || d > 8192 || few_lds_bytes(1, d) > kFewLds) return 0;
    const int rows = 16 * few_tiles(m, d), passes = ((int)m + rows - 1) / rows;
    return passes <= kFewPasses ? passes : 0;
}
hipError_t launch_dist_few(const float *Q, int64_t m, const float *C, int64_t n, int d, float *out, float *qnorm2,
                           unsigned int *max_bits, int num_cu, hipStream_t stream);
// The product with resident query rows for BF16 / FP8 rows of at most 256 bytes
// and the FILTER epilogue (gemm_rows.hip): whether it serves `a`
// (KNN_GEMM_ROWS=0 turns it off), and its launch.
bool gemm_rows_applies(const DistArgs &a, int epi);
hipError_t launch_dist_gemm_rows(const DistArgs &a, hipStream_t stream);
// Compute units of the current device.
int device_cus();
// Tile shape launch_dist_gemm uses for `a` (kTile*).
int gemm_tile_choice(const DistArgs &a);
// Squared norms of n rows of d floats into out; with max_bits (non-null, zero or
// a smaller value at launch) the largest norm's FP32 bits are folded in too.
hipError_t launch_sqnorm(const float *X, int64_t n, int d, float *out, unsigned int *max_bits, hipStream_t stream);
// The two-half operands of n rows of d floats (rows of split_row_bytes(d) bytes)
// with their scales 2^-e, and in the same read the squared norms (norm and
// max_bits as launch_sqnorm's, the same bits; norm may be null).  d >= 64.
// With src_n the n points are rows floor(i src_n / n) of src_n rows.
hipError_t launch_split(const float *X, int64_t n, int d, void *out, float *scale_out, float *norm,
                        unsigned int *max_bits, hipStream_t stream, int64_t src_n = 0);
hipError_t launch_gather_rows(const float *src, int64_t n, int d, const int32_t *idx, int64_t rows, float *dst,
                              const float *norms, float *dst_norms, hipStream_t stream);
// (total: the sum of the counts is added to it)
hipError_t launch_flag_rows(const uint32_t *cnt, int64_t m, uint32_t need, uint32_t cap, int force, uint32_t *nflag,
                            int32_t *flags, unsigned long long *total, hipStream_t stream);
hipError_t launch_scatter_fallback(const int32_t *rows, int64_t nrows, const float *val, const int32_t *idx, int kk,
                                   uint64_t *cand, uint32_t *cnt, int cap, hipStream_t stream);
hipError_t launch_rerank(const RerankArgs &a, hipStream_t stream);
// Quantises n x d FP32 rows to BF16 (prec 1) or OCP e4m3 with a per-row
// power-of-two scale (prec 2) into rows of dq = round_up(d, kQuantPad)
// elements; scale_out (FP8 only) receives 2^-e per row.
hipError_t launch_quantize(const float *X, int64_t n, int d, int prec, void *out, float *scale_out,
                           hipStream_t stream, float *norm = nullptr, unsigned int *max_bits = nullptr,
                           int64_t src_n = 0);
// Per-row certificate of a candidate list.  The reduced key of column j,
// ||c_j||^2 - 2 q_i.c_j, is computed with an error of at most
//   E_i = (gamma + 2u) max ||c||^2 + 2 (rel + 2u) ||q_i|| max ||c||
// (gamma: the FP32 norm reduction over d terms; rel: the relative error of the
// dot product in the operand precision; 2u: the final fused multiply-add).  A row
// is certified when the gap between its kk-th and k-th candidate keys exceeds
// 2 E_i: then every point outside the candidates has a larger exact key than the
// k-th candidate, so the exact top k lie among the candidates.  Uncertified rows
// of the reduced precisions are counted into *count.  (FP32 rows are certified
// with their re-rank, see RerankArgs.)
struct CertifyArgs {
    const float *sorted_keys;  // m x kk, ascending
    int64_t m;
    int kk, k;
    const float *qnorm2;       // m squared query norms
    const unsigned int *cmax2_bits;
    float rel, gamma;
    unsigned long long *count;
};
hipError_t launch_certify(const CertifyArgs &a, hipStream_t stream);

// Exact re-run of listed rows (uncertified FP32 rows) from their materialised
// reduced-key rows: every column whose key is at most the row's threshold tfix
// is re-ranked by its exact FP32 direct-form distance (the same arithmetic as
// the re-rank), and the k smallest (distance, index) pairs are written to the
// row's output.  Rows without a finite threshold re-rank every column.
struct FixupArgs {
    const float *D;          // reduced keys, row stride ldd: row f holds listed row rows[f], or
    int64_t ldd;             // with by_row, row i holds row id i (a materialised block)
    bool by_row;
    const int32_t *rows;     // nrows row ids within the block
    int64_t nrows;
    const float *tfix;       // thresholds by row id
    const float *Q;          // block queries, row-major (row id i at Q + i d)
    const float *C;          // corpus n x d
    int64_t n;
    int d, k;
    int64_t self_offset;     // >= 0: row i's own corpus index self_offset + i is excluded
    float *out_dist;         // block outputs, row id i at out + i k
    int32_t *out_idx;
    float out_scale = 1.0f;  // as RerankArgs::out_scale
};
hipError_t launch_fixup(const FixupArgs &a, hipStream_t stream);

// Unit vectors for the cosine (centre = false) and Pearson (centre = true)
// distances: each row of X minus its mean (Pearson), divided by its Euclidean
// norm, into out (n x d FP32).  A row without a direction (zero or non-finite
// norm after centring; a constant row for Pearson) becomes all NaN.
hipError_t launch_unit_rows(const float *X, int64_t n, int d, bool centre, float *out, hipStream_t stream);

// ---- the same steps over many matrices in one launch (batches) -----------------
enum : int { kPrepNorm = 0, kPrepSplit = 1, kPrepQuant = 2, kPrepGather = 3 };
// One matrix of a preparation step: its n rows, or (src_n > 0) rows
// floor(i src_n / n) of its src_n.  Norms (launch_sqnorm), two-half operands or
// quantised rows with norms (launch_split, launch_quantize), or copied rows.
struct PrepSeg {
    int kind;
    const float *X;
    int64_t n, src_n;
    int d, prec;
    void *out;
    float *scale, *norm;
    unsigned int *max_bits;
};
// One matrix of launch_flag_rows.
struct FlagSeg {
    const uint32_t *cnt;
    int64_t m;
    uint32_t need, cap;
    int force;
    uint32_t *nflag;
    int32_t *flags;
    unsigned long long *total;
};
// The segments of one launch: nseg from seg0 on, their first workgroups (and the
// end) from first0 on.
struct SegClass {
    int key;
    uint32_t seg0, nseg, first0, blocks;
};
// Classes of a list of segments (sorted by class in place) and the first
// workgroups: at most segments + classes entries.  Rows are taken as aligned as
// their pointers are.
std::vector<SegClass> group_prep(std::vector<PrepSeg> &segs, std::vector<uint32_t> &first);
std::vector<SegClass> group_rerank(std::vector<RerankArgs> &segs, std::vector<uint32_t> &first);
std::vector<SegClass> group_flags(std::vector<FlagSeg> &segs, std::vector<uint32_t> &first);
std::vector<SegClass> group_certify(std::vector<CertifyArgs> &segs, std::vector<uint32_t> &first);
// Their launches; segs and first are the lists in device memory.
hipError_t launch_prep_group(const SegClass &c, const PrepSeg *segs, const uint32_t *first, hipStream_t stream);
hipError_t launch_rerank_group(const SegClass &c, const RerankArgs *segs, const uint32_t *first, hipStream_t stream);
hipError_t launch_flag_group(const SegClass &c, const FlagSeg *segs, const uint32_t *first, hipStream_t stream);
hipError_t launch_certify_group(const SegClass &c, const CertifyArgs *segs, const uint32_t *first, hipStream_t stream);

}  // namespace knn
