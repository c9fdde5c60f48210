// Selection over rows of 1025 to 16384 columns, and over lists of at most 4096
// keys, held in registers.
//
// A row of up to 64 values per thread of a 256-thread workgroup is read once and
// stays in registers, so its first pivot can come from the whole row instead of
// a sample: the values fall into 256, 512 or 1024 disjoint groups (1, 2 or 4 per
// thread; at least about twice k), and the k-th smallest of the group minima
// bounds the k-th smallest value from above, since each of the k groups at or
// below it holds a value at or below it.  It is also tight: with G groups about
// -G ln(1 - k / G) values survive it (k = 33 of 16384: 35; k = 128 of 256 groups:
// 177), so no row is read twice, nothing spills, and one register sort of the
// survivors finishes.  (Methods, "GPU-based quick multi-select": the vote by
// ballot and mbcnt, the K-versus-L case with L >= K on the first pass.)
//
// Rows whose survivors do not fit (many equal values at the pivot, or fewer than
// k groups without NaN) lower the pivot by counting passes over the row on chip,
// and take the first columns of a value class that straddles the k-th place.
//
// Bound by the one read of the row, and below 8192 columns by the instructions
// of the sorts.  The sampled first pivot of select.hip costs a row of 4096 more
// than the row itself (a quarter of it read and sorted, then the stream): 4096
// rows of 4096, k = 64: 147 us there, 36 us here; 2048 rows of 16384, k = 64:
// 133 / 46 us; 32768 of 16384, k = 33: 614 / 510 us (4.2 TB/s); 64 rows of 4096,
// k = 10: 16.7 / 5.3 us.
#include "internal.hpp"
#include "keys.hpp"

namespace knn {

constexpr int kShortThreads = 256;
constexpr int kShortWaves = kShortThreads / kWave;
constexpr uint32_t kShortSeg = 512;  // survivors held per wave
constexpr uint32_t kShortKeys = kShortSeg * kShortWaves;
// (of a row: what leaves two workgroups with 64 KiB rows on a CU)
constexpr uint32_t kRowSeg = 504, kRowKeys = kRowSeg * kShortWaves;
static_assert(kRowKeys == kShortSortCols, "rows sorted whole");
static_assert(kShortMaxCols == 64 * kShortThreads && kShortMaxK == 2 * kShortThreads, "64 values per thread, 4 groups");

namespace {

typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));  // any element alignment

}  // namespace

// PER values per thread (16, 32 or 64).  The row is loaded by one run of
// independent loads per thread, whose values go into the group minima and into
// LDS; later passes over the row are short loops over LDS, not unrolled ones over
// registers: the first form kept the row in 64 registers per thread, and a call
// with few rows spent its time fetching the unrolled code (512 parts of 16384:
// 35 us, now 11).  The LDS of five, three or two workgroups fits a CU.
template <int PER>
__global__ __launch_bounds__(kShortThreads) void select_short_kernel(SelectArgs a) {
    constexpr uint32_t kBlock = 4 * kShortThreads;  // columns per load of the workgroup
    __shared__ __align__(16) float xs[PER * kShortThreads];  // the row; then the sort's exchange area
    __shared__ uint64_t keys[kRowKeys];                      // survivors, a segment per wave
    __shared__ uint32_t wcnt[kShortWaves];
    __shared__ uint32_t red[2][kShortWaves];
    static_assert(sizeof(xs) >= 8 * kShortThreads * sizeof(uint64_t), "exchange area");
    uint64_t *const xchg = reinterpret_cast<uint64_t *>(xs);
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const float qnan = __uint_as_float(0x7fc00000u);
    // row statistics (the same in every thread; the last thing that the workgroup writes)
    unsigned long long survivors = 0, passes = 0, cyc_pivot = 0, cyc_read = 0, cyc_keep = 0, cyc_sort = 0;
    uint32_t rows_done = 0, passes_max = 0;
    // (a reading waits for the wave's LDS accesses: 0.4 of 19 us with a row per workgroup)
    const bool timed = a.slots != nullptr;
    auto now = [timed]() -> long long { return timed ? clock64() : 0; };
    for (int64_t r = blockIdx.x; r < a.rows; r += gridDim.x) {
        const float *dist = a.dist;
        int64_t ld = a.ld, lr = r, orow = r;
        uint32_t N = a.cols, k = a.k, kout = a.k, col_off = 0;
        float *out_val = a.out_val;
        int32_t *out_idx = a.out_idx;
        if (a.split > 1) {  // part of a row (see SelectArgs)
            lr = r / a.split;
            col_off = (uint32_t)(r - lr * a.split) * a.cols;
            const uint32_t rest = a.row_cols - col_off;
            N = rest < a.cols ? rest : a.cols;
            k = k < N ? k : N;
        }
        if (a.segs) {
            const SelectSeg sg = uniform_load(a.segs + __builtin_amdgcn_readfirstlane(a.row_seg[r]));
            dist = sg.dist;
            ld = sg.ld;
            lr = r - sg.row0;
            orow = lr;
            N = sg.cols;
            k = sg.k;
            kout = k;
            out_val = sg.out_val;
            out_idx = sg.out_idx;
        }
        const float *row = dist + lr * ld + col_off;
        const long long t0 = now();

        // the row, 16 bytes per load whatever its alignment (load u of a thread:
        // columns 1024 u + 4 tid .. + 3), into LDS and the minima of four groups
        // per thread (columns g mod 4: a sorted row then has its smallest values
        // in different groups).  Every load is issued unconditionally,
        // those beyond the last whole block at the row's last 16 bytes (a part
        // of fewer than four columns has the part before it there) and unused;
        // the ragged block has its own guarded loads.
        const uint32_t whole = N / kBlock, blocks = (N + kBlock - 1) / kBlock;
        float g[4] = {qnan, qnan, qnan, qnan};  // (fminf is NaN only when both are)
        {
            f32x4 x[PER / 4];
#pragma unroll
            for (int u = 0; u < PER / 4; ++u) {
                const int64_t j = (uint32_t)u < whole ? (int64_t)(u * kBlock + 4 * tid) : (int64_t)N - 4;
                x[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_any *>(row + j));
            }
            f32x4 tail;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t j = kBlock * whole + 4 * tid + c;
                const float v = row[j < N ? j : N - 1];
                tail[c] = j < N ? v : qnan;
            }
#pragma unroll
            for (int u = 0; u < PER / 4; ++u)
                if ((uint32_t)u < whole) {
                    *reinterpret_cast<f32x4 *>(xs + u * kBlock + 4 * tid) = x[u];
#pragma unroll
                    for (int c = 0; c < 4; ++c) g[c] = fminf(g[c], x[u][c]);
                }
            if (whole < blocks) {
                *reinterpret_cast<f32x4 *>(xs + whole * kBlock + 4 * tid) = tail;
#pragma unroll
                for (int c = 0; c < 4; ++c) g[c] = fminf(g[c], tail[c]);
            }
        }
        // (each thread reads back only what it wrote)
        auto values = [&](uint32_t u) -> f32x4 { return *reinterpret_cast<const f32x4 *>(xs + u * kBlock + 4 * tid); };

        const long long t1 = now();
        // groups merged to two or one per thread when k leaves fewer enough
        uint32_t pord = kOrdNaN;
        // short enough to sort whole, and too short (a row's last part) or k too large for groups
        const bool all = N <= kRowKeys && (N < kShortMinCols || k > (uint32_t)kShortThreads / 2);
        if (!all) {
            const uint32_t rank = (k + kShortWaves - 1) / kShortWaves - 1;
            uint32_t p;
            if (k <= (uint32_t)kShortThreads / 2) {
                uint32_t m[1] = {ord32(fminf(fminf(g[0], g[1]), fminf(g[2], g[3])))};
                wave_sort_regs<1>(m);
                p = wave_key<1>(m, rank);
            } else if (k <= (uint32_t)kShortThreads) {
                uint32_t m[2] = {ord32(fminf(g[0], g[2])), ord32(fminf(g[1], g[3]))};
                wave_sort_regs<2>(m);
                p = wave_key<2>(m, rank);
            } else {
                uint32_t m[4] = {ord32(g[0]), ord32(g[1]), ord32(g[2]), ord32(g[3])};
                wave_sort_regs<4>(m);
                p = wave_key<4>(m, rank);
            }
            if (lane == 0) red[0][wave] = p;
            __syncthreads();
            pord = red[0][0];
#pragma unroll
            for (int w = 1; w < kShortWaves; ++w) pord = pord > red[0][w] ? pord : red[0][w];
        }

        const long long t2 = now();
        // survivors, in the wave's own segment; a wave with too many counts on
        uint32_t row_passes = 0;  // counting passes
        uint32_t c = 0, start[kShortWaves];
        bool fits = true;
        if (all) {
#pragma unroll 1
            for (uint32_t u = 0; u < blocks; ++u) {
                const f32x4 v = values(u);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t j = u * kBlock + 4 * tid + e;
                    if (j < N) keys[j] = make_key(v[e], j);
                }
            }
            c = N;
        } else if (pord != kOrdNaN) {
            const float pv = pord == kOrdZero ? 0.0f : ord_to_float(pord);
            uint32_t n = 0;  // (the same in every lane)
            uint64_t *const seg = keys + wave * kRowSeg;
#pragma unroll 2
            for (uint32_t u = 0; u < blocks; ++u) {
                const f32x4 v = values(u);
                uint64_t m[4], any = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    m[e] = __ballot(v[e] <= pv);  // (false for NaN)
                    any |= m[e];
                }
                if (any) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t p = n + lanes_below(m[e]);
                        if (v[e] <= pv && p < kRowSeg) seg[p] = key_of(ord32_not_nan(v[e]), u * kBlock + 4 * tid + e);
                        n += (uint32_t)__popcll(m[e]);
                    }
                }
            }
            if (lane == 0) wcnt[wave] = n;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < kShortWaves; ++w) {
                start[w] = c;
                c += wcnt[w];
                fits = fits && wcnt[w] <= kRowSeg;
            }
        } else {
            fits = false;
        }
        if (!fits) {
            // survivors appended across the waves, from keys[0], in three forms:
            // counting passes over the value classes between the row's smallest
            // and the pivot's (at least k values are at or below it) until one
            // has at least k values at or below it and few enough to hold; or,
            // where one class straddles (the usual case: the pivot's own value
            // repeated), every value below that class and its first columns
            uint32_t parity = 1;
            auto block_sum = [&](uint32_t v) -> uint32_t {  // v: one per wave, the same in its lanes
                if (lane == 0) red[parity][wave] = v;
                __syncthreads();
                uint32_t t = 0;
#pragma unroll
                for (int w = 0; w < kShortWaves; ++w) t += red[parity][w];
                parity ^= 1;  // (the next sum's writes never meet this one's reads)
                return t;
            };
            auto count_upto = [&](uint32_t t) -> uint32_t {
                uint32_t n = 0;
                ++row_passes;
#pragma unroll 1
                for (uint32_t u = 0; u < blocks; ++u) {
                    const f32x4 v = values(u);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        n += (uint32_t)__popcll(__ballot(ord32(v[e]) <= t && u * kBlock + 4 * tid + e < N));
                }
                return block_sum(n);
            };
            uint32_t hi = pord, lo = ord32(fminf(fminf(g[0], g[1]), fminf(g[2], g[3])));
#pragma unroll
            for (int st = 1; st < kWave; st <<= 1) {
                const uint32_t o = xor_lanes32(lo, st);
                lo = lo < o ? lo : o;
            }
            if (lane == 0) red[parity][wave] = lo;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < kShortWaves; ++w) lo = lo < red[parity][w] ? lo : red[parity][w];
            parity ^= 1;
            uint32_t below = hi > 0 ? count_upto(hi - 1) : 0;
            bool straddles = below < k;
            if (!straddles) {
                --hi;  // (below >= k values are at or below it)
                while (!straddles && below > kRowKeys) {
                    if (lo >= hi) {
                        below = hi > 0 ? count_upto(hi - 1) : 0;
                        straddles = true;
                        break;
                    }
                    const uint32_t mid = lo + (hi - lo) / 2, n = count_upto(mid);
                    if (n >= k) {
                        hi = mid;
                        below = n;
                    } else {
                        lo = mid + 1;
                    }
                }
            }
            const uint32_t upto = straddles ? hi - 1 : hi;  // every value class up to here (hi > 0 where it straddles)
            if (tid == 0) wcnt[0] = 0;
            __syncthreads();
#pragma unroll 1
            for (uint32_t u = 0; u < blocks; ++u) {
                const f32x4 v = values(u);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t j = u * kBlock + 4 * tid + e, o = ord32(v[e]);
                    const bool s = o <= upto && j < N;
                    const uint64_t m = __ballot(s);
                    if (m) {
                        uint32_t base = 0;
                        if (lane == 0) base = atomicAdd(&wcnt[0], (uint32_t)__popcll(m));
                        base = wave_bcast0(base);
                        if (s) keys[base + lanes_below(m)] = key_of(o, j);
                    }
                }
            }
            c = below;
            if (straddles) {
                // the first k - below columns of class hi, in column order
#pragma unroll 1
                for (uint32_t u = 0; u < blocks && c < k; ++u) {
                    const f32x4 v = values(u);
                    bool eq[4];
                    uint32_t rank = 0, total = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        eq[e] = ord32(v[e]) == hi && u * kBlock + 4 * tid + e < N;
                        const uint64_t m = __ballot(eq[e]);
                        rank += lanes_below(m);
                        total += (uint32_t)__popcll(m);
                    }
                    if (lane == 0) red[parity][wave] = total;
                    __syncthreads();
                    uint32_t at = c + rank;
#pragma unroll
                    for (int w = 0; w < kShortWaves; ++w) {
                        at += w < (int)wave ? red[parity][w] : 0u;
                        c += red[parity][w];
                    }
                    parity ^= 1;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (eq[e]) {
                            if (at < k) keys[at] = key_of(hi, u * kBlock + 4 * tid + e);
                            ++at;
                        }
                }
                c = k;
            }
        }
        if (all || !fits) {  // one run from keys[0]
            start[0] = 0;
#pragma unroll
            for (int w = 1; w < kShortWaves; ++w) start[w] = c;
        }
        __syncthreads();  // keys written, the row read
        survivors += c;
        ++rows_done;
        passes += row_passes;
        passes_max = passes_max > row_passes ? passes_max : row_passes;
        const long long t3 = now();

        // the segments' keys as one list, sorted in registers
        auto load = [&](uint32_t p) -> uint64_t {
            if (p >= c) return kKeyMax;
            uint32_t at = p;
#pragma unroll
            for (int w = 1; w < kShortWaves; ++w)
                if (p >= start[w]) at = w * kRowSeg + (p - start[w]);
            return keys[at];
        };
        auto emit = [&](uint32_t t, uint64_t key) {
            const int64_t o_at = orow * (int64_t)kout + t;
            if (a.out_keys) {
                a.out_keys[o_at] = key + col_off;
                return;
            }
            const uint32_t idx = key_idx(key), o = key_ord(key);
            // zero and NaN classes: the key holds the class, the input its bits
            out_val[o_at] = (o == kOrdZero || o == kOrdNaN) ? row[idx] : ord_to_float(o);
            if (out_idx) out_idx[o_at] = (int32_t)(idx + col_off);
        };
        if (a.out_keys)  // a part shorter than k: its missing slots hold the largest key
            for (uint32_t t = k + tid; t < kout; t += kShortThreads) a.out_keys[orow * (int64_t)kout + t] = kKeyMax;
        if (c <= (uint32_t)kWave) {
            if (wave == 0) {
                const uint64_t key = wave_sort64(load(lane));
                if (lane < k) emit(lane, key);
            }
        } else if (c <= 2u * kWave) {
            if (wave == 0) {
                uint64_t key[2] = {load(2 * lane), load(2 * lane + 1)};
                wave_sort_regs<2>(key);
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    if (2 * lane + j < k) emit(2 * lane + j, key[j]);
            }
        } else {
            if (c <= (uint32_t)kShortThreads) block_sort_regs_from<kShortThreads, 1, false>(xchg, load);
            else if (c <= 2u * kShortThreads) block_sort_regs_from<kShortThreads, 2, false>(xchg, load);
            else if (c <= 4u * kShortThreads) block_sort_regs_from<kShortThreads, 4, false>(xchg, load);
            else block_sort_regs_from<kShortThreads, 8, false>(xchg, load);
            for (uint32_t t = tid; t < k; t += kShortThreads) emit(t, xchg[t]);
        }
        __syncthreads();  // keys, row and counts are reused by the next row
        cyc_read += (unsigned long long)(t1 - t0);
        cyc_pivot += (unsigned long long)(t2 - t1);
        cyc_keep += (unsigned long long)(t3 - t2);
        cyc_sort += (unsigned long long)(now() - t3);
    }
    if (a.slots && tid < (uint32_t)kSelSlot) {
        unsigned long long v = 0;
        switch (tid) {
            case kSlotRows:
            case kSlotStreamPasses: v = rows_done; break;
            case kSlotPasses: v = passes; break;
            case kSlotPassesMax: v = passes_max; break;
            case kSlotFirstSurvivors: v = survivors; break;
            case kSlotCycles + 0: v = cyc_pivot; break;
            case kSlotCycles + 1: v = cyc_read; break;
            case kSlotCycles + 2: v = cyc_keep; break;
            case kSlotCycles + 3: v = cyc_sort; break;
        }
        a.slots[(size_t)blockIdx.x * kSelSlot + tid] = v;
    }
}

// Selection of the k smallest of each row's list of at most 4096 distinct keys
// (the candidates of a filtered product, or the lists of a row's parts), PER
// keys per thread: the same group minima, survivors and one sort, in 64 bits.
// A list shorter than k (a row whose candidates are re-done later) is padded
// with the largest key.  With k above half the groups the list is sorted whole,
// or, beyond 2048 keys, cut at its exact k-th key by bisection first.
//
// Against partition passes over the whole list in LDS (75 KB, two workgroups per
// CU): 32768 lists of about 513 keys, k = 128: 476 us there, 131 us here; 8 lists
// of 2048, k = 32: 12.3 us there, 5 us here.
template <int PER>
__global__ __launch_bounds__(kShortThreads, PER == 16 ? 4 : 6) void select_keys_kernel(SelectArgs a) {
    __shared__ uint64_t keys[kShortKeys];
    __shared__ uint64_t wpiv[kShortWaves];
    __shared__ uint32_t wcnt[kShortWaves];
    __shared__ uint32_t red[2][kShortWaves];
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    for (int64_t r = blockIdx.x; r < a.rows; r += gridDim.x) {
        const uint64_t *src = a.keys;
        const uint32_t *key_cnt = a.key_cnt;
        int64_t ld = a.ld, lr = r;
        uint32_t N = a.cols, k = a.k;
        float *out_val = a.out_val;
        int32_t *out_idx = a.out_idx;
        if (a.segs) {
            const SelectSeg sg = uniform_load(a.segs + __builtin_amdgcn_readfirstlane(a.row_seg[r]));
            src = sg.keys;
            key_cnt = sg.key_cnt;
            ld = sg.ld;
            lr = r - sg.row0;
            N = sg.cols;
            k = sg.k;
            out_val = sg.out_val;
            out_idx = sg.out_idx;
        }
        src += lr * ld;
        const uint32_t have = key_cnt ? key_cnt[lr] : N;
        const uint32_t n = have < N ? have : N;  // (at most 256 PER: see the launch)
        uint64_t x[PER];
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const uint32_t p = (uint32_t)e * kShortThreads + tid;
            x[e] = p < n ? __builtin_nontemporal_load(src + p) : kKeyMax;
        }
        uint64_t P = kKeyMax;  // survivors: keys below or at it
        const uint32_t used = (n + kShortThreads - 1) / kShortThreads;  // keys per thread
        auto lesser = [](uint64_t p, uint64_t q) { return p < q ? p : q; };
        uint64_t g[4] = {kKeyMax, kKeyMax, kKeyMax, kKeyMax};
#pragma unroll
        for (int e = 0; e < PER; ++e) g[e % 4] = lesser(g[e % 4], x[e]);
        const uint32_t rank = (k + kShortWaves - 1) / kShortWaves - 1;
        int groups = 0;  // per thread, or none: every key survives
        if (k <= (uint32_t)kShortThreads / 2 && used > 1) {
            uint64_t m[1] = {lesser(lesser(g[0], g[1]), lesser(g[2], g[3]))};
            wave_sort_regs<1>(m);
            P = wave_key<1>(m, rank);
            groups = 1;
        } else if (PER > 4 && k <= (uint32_t)kShortThreads && used > 4) {
            uint64_t m[2] = {lesser(g[0], g[2]), lesser(g[1], g[3])};
            wave_sort_regs<2>(m);
            P = wave_key<2>(m, rank);
            groups = 2;
        } else if (PER > 8 && k <= 2u * kShortThreads && used > 8) {
            wave_sort_regs<4>(g);
            P = wave_key<4>(g, rank);
            groups = 4;
        }
        if (groups) {
            if (lane == 0) wpiv[wave] = P;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < kShortWaves; ++w) P = P > wpiv[w] ? P : wpiv[w];
        }
        auto compact = [&]() -> uint32_t {  // this wave's survivors into its segment
            uint32_t c = 0;
            uint64_t *const seg = keys + wave * kShortSeg;
#pragma unroll
            for (int e = 0; e < PER; ++e) {
                const bool s = x[e] <= P && x[e] != kKeyMax;
                const uint64_t m = __ballot(s);
                if (m) {
                    const uint32_t p = c + lanes_below(m);
                    if (s && p < kShortSeg) seg[p] = x[e];
                    c += (uint32_t)__popcll(m);
                }
            }
            return c;
        };
        uint32_t c = 0, start[kShortWaves];
        for (int pass = 0;; ++pass) {
            const uint32_t mine = compact();
            if (lane == 0) wcnt[wave] = mine;
            __syncthreads();
            bool fits = true;
            c = 0;
#pragma unroll
            for (int w = 0; w < kShortWaves; ++w) {
                start[w] = c;
                c += wcnt[w];
                fits = fits && wcnt[w] <= kShortSeg;
            }
            __syncthreads();
            if (fits || pass) break;
            // too many for the segments: the exact k-th key, bit by bit (then at
            // most 1024 survive, but a wave may hold more than its segment: they
            // are dealt out again below)
            uint64_t K = 0;
            uint32_t parity = 0;
#pragma unroll 1
            for (int b = 63; b >= 0; --b) {
                const uint64_t t = K | ((1ull << b) - 1ull);
                uint32_t cnt = 0;
#pragma unroll
                for (int e = 0; e < PER; ++e) cnt += (uint32_t)__popcll(__ballot(x[e] <= t));
                if (lane == 0) red[parity][wave] = cnt;
                __syncthreads();
                uint32_t below = 0;
#pragma unroll
                for (int w = 0; w < kShortWaves; ++w) below += red[parity][w];
                parity ^= 1;
                if (below < k) K |= 1ull << b;
            }
            P = K;
            // one run from keys[0], at positions reserved across the waves
            __syncthreads();
            if (tid == 0) wcnt[0] = 0;
            __syncthreads();
#pragma unroll
            for (int e = 0; e < PER; ++e) {
                const bool s = x[e] <= P && x[e] != kKeyMax;
                const uint64_t m = __ballot(s);
                if (m) {
                    uint32_t base = 0;
                    if (lane == 0) base = atomicAdd(&wcnt[0], (uint32_t)__popcll(m));
                    base = wave_bcast0(base);
                    if (s) keys[base + lanes_below(m)] = x[e];
                }
            }
            __syncthreads();
            c = wcnt[0];
            start[0] = 0;
#pragma unroll
            for (int w = 1; w < kShortWaves; ++w) start[w] = c;
            break;
        }
        auto load = [&](uint32_t p) -> uint64_t {
            if (p >= c) return kKeyMax;
            uint32_t at = p;
#pragma unroll
            for (int w = 1; w < kShortWaves; ++w)
                if (p >= start[w]) at = w * kShortSeg + (p - start[w]);
            return keys[at];
        };
        auto emit = [&](uint32_t t, uint64_t key) {
            const int64_t o_at = lr * (int64_t)k + t;
            if (a.out_keys) {
                a.out_keys[o_at] = key;
                return;
            }
            uint32_t idx = key_idx(key);
            const uint32_t o = key_ord(key);
            float v = ord_to_float(o);
            if (key == kKeyMax) {  // a list shorter than k
                v = __uint_as_float(0x7fc00000u);
                idx = 0xFFFFFFFFu;
            } else if ((o == kOrdZero || o == kOrdNaN) && a.src) {
                v = a.src[lr * a.src_ld + idx];  // the key holds the class, the input its bits
            }
            out_val[o_at] = v;
            if (out_idx) out_idx[o_at] = (int32_t)idx;
        };
        if (c <= (uint32_t)kWave && k <= (uint32_t)kWave) {
            if (wave == 0) {
                const uint64_t key = wave_sort64(load(lane));
                if (lane < k) emit(lane, key);
            }
        } else if (c <= 2u * kWave && k <= 2u * kWave) {
            if (wave == 0) {
                uint64_t key[2] = {load(2 * lane), load(2 * lane + 1)};
                wave_sort_regs<2>(key);
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    if (2 * lane + j < k) emit(2 * lane + j, key[j]);
            }
        } else {
            const uint32_t len = c > k ? c : k;
            if (len <= (uint32_t)kShortThreads) block_sort_regs_from<kShortThreads, 1, true>(keys, load);
            else if (len <= 2u * kShortThreads) block_sort_regs_from<kShortThreads, 2, true>(keys, load);
            else if (len <= 4u * kShortThreads) block_sort_regs_from<kShortThreads, 4, true>(keys, load);
            else block_sort_regs_from<kShortThreads, 8, true>(keys, load);
            for (uint32_t t = tid; t < k; t += kShortThreads) emit(t, keys[t]);
        }
        __syncthreads();
    }
}

// ---- host side --------------------------------------------------------------
// Only for the sample rule, which leaves the first pivot to the library (the
// plain and learned rules name theirs).
// With thousands of rows what counts is the work per row, and there the streamed
// selection is ahead for many keys of the shortest and the longest rows
// (streamed / on chip, us: 2500 rows of 1500, k = 200 60 / 70; 5000 rows k = 300 9000
// columns 117 / 127, 16384 127 / 156; 16384 rows k = 128 14000 309 / 326, 16384 289 /
// 346, k = 200 1500 278 / 390, 9000 282 / 328; on chip ahead at 1200 rows, and from
// 4096 to 8192 columns everywhere).
bool select_short_applies(const SelectArgs &a) {
    if (a.mode != kPivotSample || a.keys || !select_short_shape(a.cols, a.k)) return false;
    if (a.split > 1) return true;
    if (a.k > 128 && a.cols <= kShortSortCols) return a.rows < 2000;
    if (a.k > 128 && a.cols > 8192) return a.rows < 4096;
    return !(a.k > 64 && a.cols > 13000 && a.rows >= 8192);
}

// Resident workgroups per CU of an instance.
template <class F>
static int resident(F kernel) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, kShortThreads, 0) != hipSuccess || n < 1) n = 1;
    return n < kSelSlotGroups ? n : kSelSlotGroups;
}

int select_short_grid(const SelectArgs &a, int num_cu) {
    static const int p16 = resident(select_short_kernel<16>), p32 = resident(select_short_kernel<32>),
                     p64 = resident(select_short_kernel<64>);
    const int per = a.cols <= 16u * kShortThreads ? p16 : (a.cols <= 32u * kShortThreads ? p32 : p64);
    const int64_t g = (int64_t)per * num_cu;
    return (int)(g < a.rows ? g : a.rows);
}

hipError_t launch_select_short(const SelectArgs &a, int num_cu, hipStream_t stream) {
    if (a.rows == 0) return hipSuccess;
    if (a.keys || a.cols > kShortMaxCols || a.k > kShortMaxK) return hipErrorInvalidValue;
    const dim3 g((unsigned)select_short_grid(a, num_cu)), b(kShortThreads);
    if (a.cols <= 16u * kShortThreads) hipLaunchKernelGGL(select_short_kernel<16>, g, b, 0, stream, a);
    else if (a.cols <= 32u * kShortThreads) hipLaunchKernelGGL(select_short_kernel<32>, g, b, 0, stream, a);
    else hipLaunchKernelGGL(select_short_kernel<64>, g, b, 0, stream, a);
    return hipGetLastError();
}

template <int PER>
static hipError_t launch_keys_t(const SelectArgs &a, int num_cu, hipStream_t stream) {
    static const int per = resident(select_keys_kernel<PER>);
    int64_t g = (int64_t)per * num_cu;
    if (g > a.rows) g = a.rows;
    hipLaunchKernelGGL(select_keys_kernel<PER>, dim3((unsigned)g), dim3(kShortThreads), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_select_keys(const SelectArgs &a, int num_cu, hipStream_t stream) {
    if (a.rows == 0) return hipSuccess;
    if (a.cols > (uint32_t)kSelectKeysCap || a.k > (uint32_t)kSelectMaxK) return hipErrorInvalidValue;
    // (an instance for the longest list the launch may hold; shorter lists leave
    // its later registers empty)
    if (a.cols <= 4u * kShortThreads) return launch_keys_t<4>(a, num_cu, stream);
    if (a.cols <= 8u * kShortThreads) return launch_keys_t<8>(a, num_cu, stream);
    return launch_keys_t<16>(a, num_cu, stream);
}

}  // namespace knn
