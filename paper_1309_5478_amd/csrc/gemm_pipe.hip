// Pipelined distance product on 256 x 256 tiles: BF16 and FP8 operands, and FP32
// operands split into two FP16 halves, with the threshold filter (the fused
// first pass of the quick multi-select) or the dense epilogue.
//
// FP32 as two halves.  x 2^e = h + l with h = FP16(x 2^e), l = FP16(x 2^e - h)
// and e per point (its largest magnitude scaled into [2^14, 2^15)): 11 + 11
// significand bits and l's sign hold x within one unit of FP32's last place (for
// three values in four exactly).  A dot product is then three FP16 products
// accumulated in FP32, hl + lh + hh, on matrix cores 16 times as fast as for
// FP32 operands; 2^-22 |x||y| of every product (the ll term) is left out.  That
// is less than what the FP32 matrix instruction loses: it rounds its sum at
// every second k, this one at every sixteenth (where it also cuts products 25
// bits below the largest term: the bound that certificates take of both is in
// plan.hpp, use_split).  Error of the dot product against
// FP64, rms over 512 x 512 pairs in units of 2^-24 |q||c|, FP32 instruction /
// two halves: uniform points 1.44 / 0.82 (d = 64), 5.4 / 3.3 (d = 1024); normal
// 0.30 / 0.24, 0.30 / 0.19; mixture 0.36 / 0.25, 0.79 / 0.49; unit vectors
// 0.36 / 0.26, 0.82 / 0.52; magnitudes spread over e^(3 N(0,1)) 0.28 / 0.24,
// 0.20 / 0.12.  Below d = 64 the halves lose (normal, d = 16: 0.31 / 0.36), and
// the FP32 instruction stays (search.hip).
//
// The kernel.  A persistent grid, one workgroup of eight waves per CU, each wave
// 128 rows x 64 columns (4 x 2 blocks of 32 x 32; 128 accumulator registers).
// Both operands are staged in LDS in chunks of 128 bytes of every row, two
// stages, by direct global-to-LDS loads (no registers, no LDS write
// instructions): the chunks of a workgroup's tiles form one stream, so while a
// chunk feeds the matrix cores the next one is in flight, and the next tile's
// first chunk during the last chunk and the epilogue.  16-byte piece c of row r
// lies at position c ^ ((r / 2) % 8): 16 consecutive rows read the same piece
// from all 64 banks once (with c ^ (r % 8) a sixth of all cycles were bank
// conflicts).  The large tile is what the matrix rate asks for: at 64 x 64 per
// wave the fragments alone take the LDS bandwidth (BF16: 128 B per cycle and CU
// at full rate, 96 here, 48 for the halves, which use each fragment twice).
//
// The epilogue forms d' = ||c||^2 - 2 q.c for two rows by two blocks at a time,
// votes per accumulator register and appends the kept keys to the wave's list
// in LDS (position from the ballot, nothing waited for).  The list is emptied
// to the rows, a lane per key so that the slot reservations (global atomics) are
// in flight together, when it is half full or the wave's rows change: a
// workgroup's tiles follow each other along a row tile, so most tiles pass
// without touching memory (four keys per lane at a time: 3.60 -> 3.44 ms below).  For short rows this path is the bound: the overflow
// branch, 128 times inline as first written, took 1.3 of 4.1 ms (FP8, 32768 x
// 262144, d = 256, 554 keys kept per row) in instruction fetch alone; with the
// test once per four registers, marked unlikely, 3.6 ms (2.6 with no key kept;
// gemm_rows.hip takes the largest of these).
// Nothing in front of a tile's first products waits for its thresholds, norms
// and scales (2.70 -> 2.55 ms with no key kept).
//
// Measured (32768 x 131072, d = 1024, about 450 keys kept per row): halves
// 19.3 ms = 451 TFLOP/s of FP32 work, 1352 on the matrix cores (FP32 instruction
// 69.0 ms, 128); on a mixture graph of 262144 points the cores are 69 % busy at
// the 1.72 GHz that the power limit leaves, without a bank conflict.  BF16 7.5 ms = 1133 TFLOP/s (128 x 128 tiles 12.0 ms, 731), FP8 3.7 ms
// = 2315 (871 at 128 x 128).  Whole k-NN graphs against a product that kept the
// corpus in registers and streamed the queries past it, which it replaced (k =
// 32; BF16 262144 x 256 56.9 -> 54.7 ms, 2^20 x 256 681 -> 660, 262144 x 64 38.5 ->
// 29.9; FP8 262144 x 256 48.1 -> 42.3).
#include <cstdlib>
#include <type_traits>

#include "dist.hpp"
#include "keys.hpp"

namespace knn {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

constexpr int kPipeWM = 2, kPipeWN = 4;                // waves: rows x columns
constexpr int kPipeBI = 4, kPipeBJ = 2;                // 32 x 32 blocks per wave
constexpr int kPipeWaves = kPipeWM * kPipeWN;
constexpr int kPipeThreads = 64 * kPipeWaves;
constexpr int kPipeTile = kPipeTileDim;               // rows and columns
static_assert(kPipeTile == 32 * kPipeBI * kPipeWM && kPipeTile == 32 * kPipeBJ * kPipeWN, "256 x 256");
constexpr int kPipeChunk = 128;                        // bytes of a row per stage
constexpr int kPipeStage = 2 * kPipeTile * kPipeChunk;
constexpr int kPipeLoads = 2 * kPipeTile / 8 / kPipeWaves;  // load instructions per wave and stage (8 rows each)
constexpr uint32_t kPipeList = 448;                    // listed keys per wave
constexpr uint32_t kListColBits = 25;
constexpr uint32_t kPipeGroup = 4;                     // row tiles walked together across the columns

// 64 lanes x 16 bytes from base + off (per lane) to LDS bytes lds .. + 1023.
// (The count of outstanding loads is kept by hand: see the waits below.)
__device__ __forceinline__ void load_to_lds(const unsigned char *base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base)
                 : "memory");
}

template <int PREC, class F>
__device__ __forceinline__ f32x16 mfma(F a, F b, f32x16 c) {
    if constexpr (PREC == kPrecSplit)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                      0, 0);
    else if constexpr (PREC == kPrecBF16)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                       0, 0, 0);
    else
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 127, 0, 127);
}

__device__ __forceinline__ i32x8 join(i32x4 x, i32x4 y) {
    return i32x8{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
}

template <int PREC>
constexpr int chunk_elems() {
    return PREC == kPrecSplit ? 32 : (PREC == kPrecBF16 ? 64 : 128);
}

}  // namespace

// One tile: the product it belongs to (scalar registers) and its origin.
struct PipeTile {
    const DistArgs *a;
    uint32_t row0, col0;
};

// The tiles of a workgroup.  One product (GROUPED false): its tiles are cut into
// eight contiguous ranges, one per XCD (workgroup b runs on XCD b % 8), each
// walked in groups of kPipeGroup row tiles across the column tiles, so that the
// workgroups of an XCD share operands in its L2.  Many products (GROUPED): items
// in dispatch order, workgroup b taking b, b + grid, .. (the grid is a multiple
// of eight, so an item stays on the XCD the order gives it).
template <int PREC, int EPI, bool GROUPED>
__global__ __launch_bounds__(kPipeThreads, 2) void dist_pipe_kernel(DistArgs one, const DistArgs *__restrict__ jobs,
                                                                    const GemmItem *__restrict__ items,
                                                                    uint32_t nitems) {
    constexpr int BI = kPipeBI, BJ = kPipeBJ;
    constexpr bool SC = PREC != kPrecBF16;  // per-point scales
    __shared__ __align__(1024) unsigned char stage[2 * kPipeStage];
    __shared__ uint2 list[EPI == kEpiFilter ? kPipeWaves : 1][EPI == kEpiFilter ? kPipeList : 1];
    __shared__ __align__(16) float stau[2][EPI == kEpiFilter ? kPipeTile : 4], sqs[2][SC ? kPipeTile : 4];
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint32_t wm = wave % kPipeWM, wn = wave / kPipeWM, h = lane / 32, l32 = lane % 32;

    uint32_t first, end, step;
    if (GROUPED) {
        first = blockIdx.x;
        end = nitems;
        step = gridDim.x;
    } else {
        const uint32_t T = one.tiles_m * one.tiles_n, per = (T + 7) / 8, x0 = (blockIdx.x % 8) * per;
        first = x0 + blockIdx.x / 8;
        end = x0 + per < T ? x0 + per : T;
        step = gridDim.x / 8;
    }
    if (first >= end) return;  // the whole workgroup leaves together
    auto tile_at = [&](uint32_t t) -> PipeTile {
        if (GROUPED) {
            const GemmItem w = items[t];
            return PipeTile{jobs + w.job, w.tm * kPipeTile, w.tn * kPipeTile};
        }
        const uint32_t group = t / (kPipeGroup * one.tiles_n), r0 = group * kPipeGroup;
        const uint32_t gs = one.tiles_m - r0 < kPipeGroup ? one.tiles_m - r0 : kPipeGroup;
        const uint32_t in = t - r0 * one.tiles_n;
        return PipeTile{&one, (r0 + in % gs) * kPipeTile, (in / gs) * kPipeTile};
    };

    // the load stream: instruction x of this wave fills rows 8 (wave kPipeLoads
    // + x) .. + 7 of the stage (256 query rows, then 256 corpus rows); rows
    // beyond the matrices read the last one (their results are never kept)
    uint32_t off[kPipeLoads];
    const unsigned char *Ab, *Bb;
    auto load_tile = [&](const PipeTile &pt) {
        const DistArgs &a = *pt.a;
        const uint32_t ldq = (uint32_t)a.ldq;
        Ab = static_cast<const unsigned char *>(a.Qq) + (int64_t)pt.row0 * ldq;
        Bb = static_cast<const unsigned char *>(a.Cq) + (int64_t)pt.col0 * ldq;
        const uint32_t alim = (uint32_t)a.m - pt.row0 - 1, blim = (uint32_t)a.n - pt.col0 - 1;
#pragma unroll
        for (int x = 0; x < kPipeLoads; ++x) {
            const uint32_t r8 = (wave * kPipeLoads + x) * 8;
            const uint32_t r = (r8 < kPipeTile ? r8 : r8 - kPipeTile) + lane / 8, lim = r8 < kPipeTile ? alim : blim;
            off[x] = (r < lim ? r : lim) * ldq + ((lane % 8) ^ (((r8 + lane / 8) >> 1) & 7)) * 16;
        }
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)stage;
    auto load_chunk = [&](int kc, uint32_t buf) {
#pragma unroll
        for (int x = 0; x < kPipeLoads; ++x) {
            const uint32_t r8 = (wave * kPipeLoads + x) * 8;
            load_to_lds((r8 < kPipeTile ? Ab : Bb) + (int64_t)kc * kPipeChunk, off[x],
                        lds0 + buf * kPipeStage + r8 * kPipeChunk);
        }
    };

    // one staged chunk: the fragments of block row i, columns j (lane half h
    // holds the upper or lower half of a k-step), then the products, k ascending
    const uint32_t sw = (l32 >> 1) & 7;
    const uint32_t arow = (wm * 32 * BI + l32) * kPipeChunk, brow = (kPipeTile + wn * 32 * BJ + l32) * kPipeChunk;
    f32x16 acc[BI][BJ];
    auto mma_chunk = [&](uint32_t buf) {
        const unsigned char *Ap = stage + buf * kPipeStage + arow, *Bp = stage + buf * kPipeStage + brow;
        auto fa = [&](int i, int piece) -> i32x4 {
            return *reinterpret_cast<const i32x4 *>(Ap + i * 32 * kPipeChunk + ((piece ^ sw) * 16));
        };
        auto fb = [&](int j, int piece) -> i32x4 {
            return *reinterpret_cast<const i32x4 *>(Bp + j * 32 * kPipeChunk + ((piece ^ sw) * 16));
        };
        if constexpr (PREC == kPrecSplit) {
            // a chunk row: the high halves of 32 elements, then their low halves
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                i32x4 ah[BI], al[BI], bh[BJ], bl[BJ];
#pragma unroll
                for (int j = 0; j < BJ; ++j) bh[j] = fb(j, 2 * s + h), bl[j] = fb(j, 4 + 2 * s + h);
#pragma unroll
                for (int i = 0; i < BI; ++i) ah[i] = fa(i, 2 * s + h), al[i] = fa(i, 4 + 2 * s + h);
#pragma unroll
                for (int i = 0; i < BI; ++i)
#pragma unroll
                    for (int j = 0; j < BJ; ++j) {
                        acc[i][j] = mfma<PREC>(ah[i], bl[j], acc[i][j]);
                        acc[i][j] = mfma<PREC>(al[i], bh[j], acc[i][j]);
                        acc[i][j] = mfma<PREC>(ah[i], bh[j], acc[i][j]);
                    }
            }
        } else if constexpr (PREC == kPrecBF16) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                i32x4 af[BI], bf[BJ];
#pragma unroll
                for (int j = 0; j < BJ; ++j) bf[j] = fb(j, 2 * s + h);
#pragma unroll
                for (int i = 0; i < BI; ++i) af[i] = fa(i, 2 * s + h);
#pragma unroll
                for (int i = 0; i < BI; ++i)
#pragma unroll
                    for (int j = 0; j < BJ; ++j) acc[i][j] = mfma<PREC>(af[i], bf[j], acc[i][j]);
            }
        } else {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                i32x8 af[BI], bf[BJ];
#pragma unroll
                for (int j = 0; j < BJ; ++j) bf[j] = join(fb(j, 4 * s + 2 * h), fb(j, 4 * s + 2 * h + 1));
#pragma unroll
                for (int i = 0; i < BI; ++i) af[i] = join(fa(i, 4 * s + 2 * h), fa(i, 4 * s + 2 * h + 1));
#pragma unroll
                for (int i = 0; i < BI; ++i)
#pragma unroll
                    for (int j = 0; j < BJ; ++j) acc[i][j] = mfma<PREC>(af[i], bf[j], acc[i][j]);
            }
        }
    };

    PipeTile next = tile_at(first);
    load_tile(next);
    load_chunk(0, 0);
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    uint32_t buf = 0, par = 0;
    uint32_t kept = 0, list_col0 = 0;  // listed keys of this wave (the same in every lane), origin of their columns
    for (uint32_t t = first; t < end; t += step, par ^= 1) {
        const uint32_t row0 = next.row0, col0 = next.col0;
        const DistArgs &a = *next.a;
        const int nk = (a.d + chunk_elems<PREC>() - 1) / chunk_elems<PREC>();
        const bool more = t + step < end;
        if (more) next = tile_at(t + step);
        // This tile's thresholds, scales and norms are requested now (rows and
        // columns beyond the matrices: the last one's) and not touched before
        // the first chunk's products are done, so that nothing waits for them.
        float tv = 0.f, qv = 1.f;
        const uint32_t grow = row0 + tid;
        if (tid < (uint32_t)kPipeTile) {
            const int64_t gi = grow < a.m ? grow : a.m - 1;
            if (EPI == kEpiFilter) tv = a.tau[gi * a.tau_stride];
            if (SC) qv = a.qscale[gi];
        }
        float cn[BJ], cs[BJ];
#pragma unroll
        for (int j = 0; j < BJ; ++j) {
            const uint32_t gj = col0 + wn * 32 * BJ + j * 32 + l32;
            const int64_t cj = gj < a.n ? gj : a.n - 1;
            cn[j] = a.cnorm[cj];
            cs[j] = SC ? a.cscale[cj] : 1.0f;
        }
#pragma unroll
        for (int i = 0; i < BI; ++i)
#pragma unroll
            for (int j = 0; j < BJ; ++j) acc[i][j] = f32x16{0.f};
        for (int kc = 0; kc < nk; ++kc) {
            // every wave has left the other buffer (the barrier below)
            if (kc + 1 < nk) {
                load_chunk(kc + 1, buf ^ 1);
            } else if (more) {
                load_tile(next);
                load_chunk(0, buf ^ 1);
            }
            mma_chunk(buf);
            // this wave's loads have landed; with the first chunk the thresholds
            // and scales go to LDS (the copy of this tile's parity: another wave
            // may still be in the previous tile's epilogue).  A NaN threshold
            // keeps nothing (rows beyond the matrix), nor does a NaN norm
            // (columns beyond it).
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (kc == 0 && tid < (uint32_t)kPipeTile) {
                if (EPI == kEpiFilter) stau[par][tid] = grow < a.m ? tv : __uint_as_float(0x7fc00000u);
                if (SC) sqs[par][tid] = qv;
            }
            // and its LDS accesses are done, and after the barrier every wave's
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            buf ^= 1;
        }

        // element (i, j), register r: row 32 i + 8 (r / 4) + 4 h + r % 4, column 32 j + l32 of the wave's block
        const uint32_t gr0 = row0 + wm * 32 * BI, gc0 = col0 + wn * 32 * BJ;
        // (opaque to the compiler here: the epilogue's offsets are then formed in
        // place, not kept in registers through the K loop)
        uint32_t hv = h, lv = l32;
        asm volatile("" : "+v"(hv), "+v"(lv));
#pragma unroll
        for (int j = 0; j < BJ; ++j) {
            asm volatile("" : "+v"(cn[j]), "+v"(cs[j]));
            if (col0 + wn * 32 * BJ + j * 32 + lv >= a.n) cn[j] = __uint_as_float(0x7fc00000u);
            cs[j] *= -2.0f;
        }
        const float *qp = &sqs[par][SC ? wm * 32 * BI + 4 * hv : 0];
        if constexpr (EPI == kEpiDense) {
#pragma unroll
            for (int i = 0; i < BI; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    f32x4 q4 = {1.f, 1.f, 1.f, 1.f};
                    if (SC) q4 = *reinterpret_cast<const f32x4 *>(qp + i * 32 + 8 * q);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t gi = gr0 + i * 32 + 8 * q + 4 * hv + e;
                        const int64_t own = a.self_offset >= 0 ? a.self_offset + gi : (int64_t)-1;
#pragma unroll
                        for (int j = 0; j < BJ; ++j) {
                            const uint32_t gj = gc0 + j * 32 + lv;
                            const float dot = SC ? acc[i][j][4 * q + e] * q4[e] : acc[i][j][4 * q + e];
                            const float dp = fmaf(cs[j], dot, cn[j]);
                            if (gi < a.m && gj < a.n)
                                a.out[(int64_t)gi * a.ldo + gj] = (int64_t)gj == own ? __uint_as_float(0x7f800000u) : dp;
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
        } else {
            // listed: the distance's bits, and the row in the wave's block (7
            // bits) over the column from list_col0 on (25 bits)
            if (kept == 0) list_col0 = gc0;
            uint2 *const mine = list[wave];
            auto drain = [&]() {
                __builtin_amdgcn_wave_barrier();
                // four keys per lane at a time: their slots are asked for together
                for (uint32_t p0 = 0; p0 < kept; p0 += 4 * kWave) {
                    uint32_t slot[4], row[4], col[4];
                    float v[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const uint32_t p = p0 + x * kWave + lane;
                        slot[x] = 0xffffffffu;
                        if (p < kept) {
                            const uint2 e = mine[p];
                            v[x] = __uint_as_float(e.x);
                            row[x] = gr0 + (e.y >> kListColBits);
                            col[x] = (uint32_t)a.col_base + list_col0 + (e.y & ((1u << kListColBits) - 1));
                            if (a.self_offset < 0 || (int64_t)col[x] != a.self_offset + row[x])  // (not its own point)
                                slot[x] = atomicAdd(&a.cnt[row[x]], 1u);
                        }
                    }
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        if (slot[x] < (uint32_t)a.cap)
                            a.cand[(size_t)row[x] * a.cap + slot[x]] = key_of(ord32_not_nan(v[x]), col[x]);
                }
                __builtin_amdgcn_wave_barrier();
                kept = 0;
            };
            const uint32_t rc0 = (4 * hv << kListColBits) + (gc0 - list_col0 + lv);
            const float *tp = &stau[par][wm * 32 * BI + 4 * hv];
#pragma unroll
            for (int i = 0; i < BI; ++i) {
                f32x4 t4[4], q4[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    t4[q] = *reinterpret_cast<const f32x4 *>(tp + i * 32 + 8 * q);
                    if (SC) q4[q] = *reinterpret_cast<const f32x4 *>(qp + i * 32 + 8 * q);
                }
#pragma unroll
                for (int g = 0; g < 8; ++g) {  // two rows by BJ blocks at a time
                    const int q = g / 2;
                    uint64_t m[2][BJ], any = 0;
                    float dp[2][BJ];
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int j = 0; j < BJ; ++j) {
                            const int e = 2 * (g % 2) + u;
                            const float dot = SC ? acc[i][j][4 * q + e] * q4[q][e] : acc[i][j][4 * q + e];
                            dp[u][j] = fmaf(cs[j], dot, cn[j]);
                            m[u][j] = __ballot(dp[u][j] <= t4[q][e]);
                            any |= m[u][j];
                        }
                    if (any) {
                        if (__builtin_expect(kept > kPipeList - 2 * BJ * kWave, 0)) {
                            drain();
                            // (the list's origin stays: rc0 counts from it)
                        }
#pragma unroll
                        for (int u = 0; u < 2; ++u)
#pragma unroll
                            for (int j = 0; j < BJ; ++j)
                                if (m[u][j]) {
                                    if (__builtin_amdgcn_inverse_ballot_w64(m[u][j]))
                                        mine[kept + lanes_below(m[u][j])] =
                                            uint2{__float_as_uint(dp[u][j]),
                                                  rc0 + ((uint32_t)(i * 32 + 8 * q + 2 * (g % 2) + u) << kListColBits) +
                                                      j * 32};
                                    kept += (uint32_t)__popcll(m[u][j]);
                                }
                    }
                    // (hoisting the other groups' work would hold them all in
                    // registers)
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            // the list stays open while the tiles stay in these rows
            if (!more || next.row0 != row0 || next.a != &a || next.col0 < col0 ||
                next.col0 - list_col0 >= (1u << kListColBits) - kPipeTile || kept > kPipeList / 2)
                drain();
        }
    }
}

// ---- host side --------------------------------------------------------------
int device_cus() {
    // (the library targets one device type, so one value per process)
    static const int cus = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 8)
            n = 256;
        return n;
    }();
    return cus;
}

bool lowprec_pipe_on() {
    const char *e = std::getenv("KNN_GEMM_PIPE");
    return !(e && e[0] == '0') && !std::getenv("KNN_GEMM_TILE");
}

bool gemm_pipe_applies(const DistArgs &a, int epi) {
    if (a.prec == kPrecSplit) return true;  // (there is no other kernel for split operands)
    // (dense: the tile's 256 KiB of results leave the cores idle while they are
    // written, and the 128 x 128 tiles, several to a CU, overlap that: 32768 x
    // 8192, d = 1024, BF16: 697 us here, 496 there)
    if (epi != kEpiFilter || (a.prec != kPrecBF16 && a.prec != kPrecFP8)) return false;
    if (a.qnorm || a.row_ids || (a.tile >= 0 && a.tile != kTilePipe) || a.ldq > (1 << 22)) return false;
    return lowprec_pipe_on() && pipe_fills(a.m, a.n);
}

template <int PREC>
static hipError_t launch_pipe_t(const DistArgs &a0, int epi, hipStream_t stream) {
    DistArgs a = a0;
    a.tiles_m = (uint32_t)((a.m + kPipeTile - 1) / kPipeTile);
    a.tiles_n = (uint32_t)((a.n + kPipeTile - 1) / kPipeTile);
    const uint64_t tiles = (uint64_t)a.tiles_m * a.tiles_n;
    // tile numbers up to the end of the last XCD's range, plus one step, in 32 bits
    if (tiles > 0x7fffffffull || a.ldq > (1 << 22) || a.qnorm || a.row_ids) return hipErrorInvalidValue;
    if (!a.Qq || !a.Cq || (PREC != kPrecBF16 && (!a.qscale || !a.cscale))) return hipErrorInvalidValue;
    const uint64_t fit = (tiles + 7) / 8 * 8, cus = (uint64_t)device_cus() / 8 * 8;
    const dim3 g((unsigned)(fit < cus ? fit : cus)), b(kPipeThreads);
    if (epi == kEpiDense) {
        if constexpr (PREC == kPrecSplit)
            hipLaunchKernelGGL((dist_pipe_kernel<PREC, kEpiDense, false>), g, b, 0, stream, a, nullptr, nullptr, 0u);
        else
            return hipErrorInvalidValue;
    } else {
        hipLaunchKernelGGL((dist_pipe_kernel<PREC, kEpiFilter, false>), g, b, 0, stream, a, nullptr, nullptr, 0u);
    }
    return hipGetLastError();
}

hipError_t launch_dist_gemm_pipe(const DistArgs &a, int epi, hipStream_t stream) {
    if (a.m == 0 || a.n == 0) return hipSuccess;
    switch (a.prec) {
        case kPrecSplit: return launch_pipe_t<kPrecSplit>(a, epi, stream);
        case kPrecBF16: return launch_pipe_t<kPrecBF16>(a, epi, stream);
        case kPrecFP8: return launch_pipe_t<kPrecFP8>(a, epi, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_dist_gemm_pipe_grouped(const DistArgs *jobs, const GemmItem *items, int64_t nitems, int prec,
                                         hipStream_t stream, int epi) {
    if (nitems == 0) return hipSuccess;
    if (nitems > 0x7fffffff) return hipErrorInvalidValue;
    const int64_t fit = (nitems + 7) / 8 * 8, cus = (int64_t)device_cus() / 8 * 8;
    const dim3 g((unsigned)(fit < cus ? fit : cus)), b(kPipeThreads);
    const DistArgs none{};
    const uint32_t n = (uint32_t)nitems;
#define KNN_PIPE_GROUPED(PREC, EPI) \
    hipLaunchKernelGGL((dist_pipe_kernel<PREC, EPI, true>), g, b, 0, stream, none, jobs, items, n)
    if (epi == kEpiDense) {
        if (prec != kPrecSplit) return hipErrorInvalidValue;
        KNN_PIPE_GROUPED(kPrecSplit, kEpiDense);
    } else {
        switch (prec) {
            case kPrecSplit: KNN_PIPE_GROUPED(kPrecSplit, kEpiFilter); break;
            case kPrecBF16: KNN_PIPE_GROUPED(kPrecBF16, kEpiFilter); break;
            case kPrecFP8: KNN_PIPE_GROUPED(kPrecFP8, kEpiFilter); break;
            default: return hipErrorInvalidValue;
        }
    }
#undef KNN_PIPE_GROUPED
    return hipGetLastError();
}

}  // namespace knn
