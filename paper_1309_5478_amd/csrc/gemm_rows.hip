// Distance product with resident query rows: BF16 and FP8 operands of at most
// 256 bytes a row (d <= 128 and d <= 256), with the threshold filter.
//
// Such rows have so short a product that the filter decides: on the 256 x 256
// tiles (gemm_pipe.hip) all waves of a SIMD are in their products together and
// in their filters together, so the matrix cores idle half of the time.  Here a
// wave keeps its 64 query rows and their thresholds in registers and the corpus
// passes in steps of 64 columns through a ring of four LDS stages (direct
// global-to-LDS loads, three steps ahead; 16-byte piece c of a row at c ^ row,
// no bank conflicts), one barrier a step.  Of the two waves of a SIMD one filters
// step t after its product, the other, `late`, before its product of step t + 1,
// on the other side of the barrier: the products of one run under the filter of
// the other.  The row scales of FP8 are an operand of its matrix instruction
// (exponents, exact: scaled partial sums stay normal numbers for e in [-100, 100]),
// the column scales a factor of the final fused multiply-add; the key bits are
// those of the tiles.
//
// Kept keys go to the wave's list as there, and all waves empty their lists
// after the same step (one asks, a step ahead: a wave alone at the atomics would
// hold up the others at the barrier, 2.79 -> 2.69 ms).  An XCD's workgroups take row
// tiles of one eighth of the columns, so a step's corpus rows are read into its
// L2 once for all of them.
//
// Measured, 32768 x 262144, about 550 (BF16 470) keys kept per row, 256 x 256 tiles /
// this: FP8 d = 256 3.43 / 2.69 ms (1.6 PFLOP/s; 1.73 with no key kept), d = 128 2.78 /
// 2.32, BF16 d = 128 2.55.
#include <cstdlib>

#include "dist.hpp"
#include "keys.hpp"

namespace knn {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

constexpr int kRowsWaves = 8, kRowsThreads = 64 * kRowsWaves;
constexpr int kRowsBI = 2, kRowsBJ = 2;                   // 32 x 32 blocks per wave
constexpr int kRowsWave = 32 * kRowsBI;                   // query rows of a wave
constexpr int kRowsTile = kRowsWave * kRowsWaves;         // and of a workgroup
constexpr int kRowsCols = 32 * kRowsBJ;                   // corpus columns of a step
constexpr int kRowsRing = 4;                              // staged steps
constexpr uint32_t kRowsList = 640;                       // listed keys per wave
constexpr uint32_t kRowsColBits = 26;

// 64 lanes x 16 (or 4) bytes from base + off (per lane) to LDS bytes lds ...
__device__ __forceinline__ void rows_load16(const unsigned char *base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base)
                 : "memory");
}
__device__ __forceinline__ void rows_load4(const void *base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(off), "s"(base)
                 : "memory");
}

__device__ __forceinline__ i32x8 rows_join(i32x4 x, i32x4 y) {
    return i32x8{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
}

}  // namespace

// units: of an XCD's column range, sub parts by row tiles (row tile first).
template <int PREC, int LD>  // LD: the bytes of a row that are used
__global__ __launch_bounds__(kRowsThreads, 2) void dist_rows_kernel(DistArgs a, uint32_t row_tiles, uint32_t sub) {
    constexpr int BI = kRowsBI, BJ = kRowsBJ;
    constexpr bool SC = PREC == kPrecFP8;
    constexpr int PIECES = LD / 16;                 // of a row
    constexpr int KS = PREC == kPrecFP8 ? LD / 64 : LD / 32;  // k-steps
    constexpr int STAGE = kRowsCols * LD;
    constexpr int LOADS = STAGE / 1024 / kRowsWaves;  // 16-byte load instructions per wave and step
    constexpr int ROWS = 1024 / LD;                 // corpus rows per load instruction
    __shared__ __align__(1024) unsigned char stage[kRowsRing * STAGE];
    __shared__ __align__(256) float scn[kRowsRing][kRowsCols], scs[kRowsRing][SC ? kRowsCols : 1];
    __shared__ uint2 list[kRowsWaves][kRowsList];
    __shared__ uint32_t empty_at[2];  // the step after which every wave empties its list, by parity
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint32_t h = lane / 32, l32 = lane % 32;
    const bool late = wave >= kRowsWaves / 2;  // the waves whose epilogue follows the barrier

    const uint32_t T = (uint32_t)((a.n + kRowsCols - 1) / kRowsCols), xcd = blockIdx.x % 8;
    const uint32_t x0 = (uint32_t)((uint64_t)T * xcd / 8), x1 = (uint32_t)((uint64_t)T * (xcd + 1) / 8);
    const uint32_t ldq = (uint32_t)a.ldq;
    const unsigned char *const Q = static_cast<const unsigned char *>(a.Qq), *const C = static_cast<const unsigned char *>(a.Cq);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)stage;
    const uint32_t ldn0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float *)&scn[0][0];
    const uint32_t lds1 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float *)&scs[0][0];
    auto swz = [](uint32_t r) -> uint32_t { return LD == 256 ? (r & 15) : ((r >> 1) & 7); };

    for (uint32_t u = blockIdx.x / 8; u < row_tiles * sub; u += gridDim.x / 8) {
        const uint32_t part = u / row_tiles, row0 = (u % row_tiles) * kRowsTile + wave * kRowsWave;
        const uint32_t t0 = x0 + (uint32_t)((uint64_t)(x1 - x0) * part / sub);
        const uint32_t t1 = x0 + (uint32_t)((uint64_t)(x1 - x0) * (part + 1) / sub);
        if (t0 >= t1) continue;  // (the same for the whole workgroup)
        const uint32_t col_first = t0 * kRowsCols;

        // this wave's rows (beyond the matrix: the last one, kept by no threshold)
        i32x4 af[BI][PIECES / 2];
        int sa = 0;
        float tv[BI][16];
#pragma unroll
        for (int i = 0; i < BI; ++i) {
            const int64_t r = row0 + 32 * i + l32, rr = r < a.m ? r : a.m - 1;
            const unsigned char *q = Q + rr * ldq;
#pragma unroll
            for (int p = 0; p < PIECES / 2; ++p) {
                const int piece = PREC == kPrecFP8 ? 4 * (p / 2) + p % 2 + 2 * (int)h : 2 * p + (int)h;
                af[i][p] = *reinterpret_cast<const i32x4 *>(q + 16 * piece);
            }
            if (SC) sa |= (int)((__float_as_uint(a.qscale[rr]) >> 23) & 255u) << (8 * i);
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                const int64_t g = row0 + 32 * i + 8 * (x / 4) + 4 * h + x % 4;
                const float t = a.tau[(g < a.m ? g : a.m - 1) * a.tau_stride];
                tv[i][x] = g < a.m ? t : __uint_as_float(0x7fc00000u);
            }
        }

        // (waited for here: inside the loop the compiler's wait would be for the
        // steps under way as well)
        asm volatile("" : "+v"(sa));
#pragma unroll
        for (int i = 0; i < BI; ++i) {
#pragma unroll
            for (int p = 0; p < PIECES / 2; ++p) asm volatile("" : "+v"(af[i][p]));
#pragma unroll
            for (int x = 0; x < 16; ++x) asm volatile("" : "+v"(tv[i][x]));
        }

        auto load_step = [&](uint32_t t) {
            const uint32_t slot = t % kRowsRing, c0 = t * kRowsCols;
            const uint32_t lim = (uint32_t)a.n - c0 - 1;
            const unsigned char *base = C + (int64_t)c0 * ldq;
#pragma unroll
            for (int x = 0; x < LOADS; ++x) {
                const uint32_t r0 = (wave * LOADS + x) * ROWS, r = r0 + lane / PIECES;
                rows_load16(base, (r < lim ? r : lim) * ldq + ((lane % PIECES) ^ swz(r)) * 16,
                            lds0 + slot * STAGE + r0 * LD);
            }
            if (wave == 0) rows_load4(a.cnorm + c0, (lane < lim ? lane : lim) * 4, ldn0 + slot * kRowsCols * 4);
            if (SC && wave == 1) rows_load4(a.cscale + c0, (lane < lim ? lane : lim) * 4, lds1 + slot * kRowsCols * 4);
        };

        f32x16 acc[BI][BJ];
        float cn[BJ], cs[BJ];
        auto product = [&](uint32_t t) {
            const uint32_t slot = t % kRowsRing;
            const unsigned char *Bp = stage + slot * STAGE + l32 * LD;
#pragma unroll
            for (int j = 0; j < BJ; ++j) {
                cn[j] = scn[slot][j * 32 + l32];
                cs[j] = SC ? scs[slot][j * 32 + l32] : 1.0f;
            }
#pragma unroll
            for (int i = 0; i < BI; ++i)
#pragma unroll
                for (int j = 0; j < BJ; ++j) acc[i][j] = f32x16{0.f};
            auto fb = [&](int j, int piece) -> i32x4 {
                return *reinterpret_cast<const i32x4 *>(Bp + j * 32 * LD + ((uint32_t)piece ^ swz(l32)) * 16);
            };
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if constexpr (PREC == kPrecFP8) {
                    i32x8 b[BJ];
#pragma unroll
                    for (int j = 0; j < BJ; ++j) b[j] = rows_join(fb(j, 4 * s + 2 * h), fb(j, 4 * s + 2 * h + 1));
#pragma unroll
                    for (int j = 0; j < BJ; ++j) {
                        acc[0][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                            rows_join(af[0][2 * s], af[0][2 * s + 1]), b[j], acc[0][j], 0, 0, 0, sa, 0, 127);
                        acc[1][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                            rows_join(af[1][2 * s], af[1][2 * s + 1]), b[j], acc[1][j], 0, 0, 1, sa, 0, 127);
                    }
                } else {
                    i32x4 b[BJ];
#pragma unroll
                    for (int j = 0; j < BJ; ++j) b[j] = fb(j, 2 * s + h);
#pragma unroll
                    for (int i = 0; i < BI; ++i)
#pragma unroll
                        for (int j = 0; j < BJ; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                __builtin_bit_cast(bf16x8, af[i][s]), __builtin_bit_cast(bf16x8, b[j]), acc[i][j], 0,
                                0, 0);
                }
            }
        };

        uint2 *const mine = list[wave];
        uint32_t kept = 0;  // (the same in every lane)
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
                        row[x] = row0 + (e.y >> kRowsColBits);
                        col[x] = (uint32_t)a.col_base + col_first + (e.y & ((1u << kRowsColBits) - 1));
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
        auto filter = [&](uint32_t t, uint32_t now) {
            const uint32_t rc0 = (4 * h << kRowsColBits) + ((t - t0) * kRowsCols + l32);
#pragma unroll
            for (int j = 0; j < BJ; ++j) {
                if (t * kRowsCols + j * 32 + l32 >= a.n) cn[j] = __uint_as_float(0x7fc00000u);
                cs[j] *= -2.0f;
            }
#pragma unroll
            for (int i = 0; i < BI; ++i)
#pragma unroll
                for (int g = 0; g < 8; ++g) {  // two rows by BJ blocks at a time
                    uint64_t m[2][BJ], any = 0;
                    float dp[2][BJ];
#pragma unroll
                    for (int w = 0; w < 2; ++w)
#pragma unroll
                        for (int j = 0; j < BJ; ++j) {
                            dp[w][j] = fmaf(cs[j], acc[i][j][2 * g + w], cn[j]);
                            m[w][j] = __ballot(dp[w][j] <= tv[i][2 * g + w]);
                            any |= m[w][j];
                        }
                    if (any) {
                        if (__builtin_expect(kept > kRowsList - 2 * BJ * kWave, 0)) drain();
#pragma unroll
                        for (int w = 0; w < 2; ++w)
#pragma unroll
                            for (int j = 0; j < BJ; ++j)
                                if (m[w][j]) {
                                    if (__builtin_amdgcn_inverse_ballot_w64(m[w][j]))
                                        mine[kept + lanes_below(m[w][j])] =
                                            uint2{__float_as_uint(dp[w][j]),
                                                  rc0 + ((uint32_t)(i * 32 + 8 * (g / 2) + 2 * (g % 2) + w)
                                                         << kRowsColBits) + j * 32};
                                    kept += (uint32_t)__popcll(m[w][j]);
                                }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            if (kept > kRowsList / 4 && lane == 0) empty_at[(now + 1) & 1] = now + 1;
        };

        if (tid < 2) empty_at[tid] = 0xffffffffu;
        // every wave has left the ring (and its loads have landed)
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        for (uint32_t t = t0; t < t0 + kRowsRing - 1 && t < t1; ++t) load_step(t);
        for (uint32_t t = t0; t < t1; ++t) {
            // this wave's loads of step t have landed (those of the two after it
            // may be outstanding), and after the barrier every wave's; every wave
            // has left step t - 1's slot
            if (t + 2 < t1) {
                if (wave < (SC ? 2 : 1)) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * (LOADS + 1)) : "memory");
                else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * LOADS) : "memory");
            } else {
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            }
            if (t + kRowsRing - 1 < t1) load_step(t + kRowsRing - 1);
            const bool empty = empty_at[t & 1] == t;
            if (late && t > t0) filter(t - 1, t);
            product(t);
            if (!late) filter(t, t);
            if (empty) drain();
        }
        if (late) filter(t1 - 1, t1);
        drain();
    }
}

// ---- host side --------------------------------------------------------------
static int rows_bytes(const DistArgs &a) { return ((a.prec == kPrecBF16 ? 2 * a.d : a.d) + 127) / 128 * 128; }

bool gemm_rows_applies(const DistArgs &a, int epi) {
    if (epi != kEpiFilter || (a.prec != kPrecBF16 && a.prec != kPrecFP8)) return false;
    if (a.qnorm || a.row_ids || (a.tile >= 0 && a.tile != kTilePipe) || rows_bytes(a) > 256) return false;
    if (!lowprec_pipe_on() || a.n > (int64_t(1) << 29)) return false;
    if (const char *e = std::getenv("KNN_GEMM_ROWS")) return e[0] == '1';
    // (below, the row tiles of 512 are too few for the workgroups or a part's
    // beginning costs what the steps save; whole searches, 256 x 256 tiles /
    // this, us: FP8 d = 256 m = n = 16000 611 / 576, 20000 x 1000 queries 168 / 185,
    // 300000 x 1100 585 / 569, 300000 x 16384 2850 / 2405; BF16 d = 64 30000^2 916 /
    // 930, 300000 x 16384 1948 / 1829, 131072^2 7943 / 7449)
    return a.m >= 4096 && a.m * a.n >= (int64_t(1) << 31);
}

template <int PREC, int LD>
static hipError_t launch_rows_t(const DistArgs &a, hipStream_t stream) {
    const int64_t R = (a.m + kRowsTile - 1) / kRowsTile, T8 = ((a.n + kRowsCols - 1) / kRowsCols + 7) / 8;
    const int64_t W = device_cus() / 8;
    // parts of an XCD's columns: what leaves its W workgroups most evenly loaded
    // (a part costs about six steps to begin)
    int64_t sub = 1, best = INT64_MAX;
    for (int64_t s = 1; s <= 64 && s * 8 <= T8; ++s) {
        const int64_t cost = (R * s + W - 1) / W * ((T8 + s - 1) / s + 6);
        if (cost < best) best = cost, sub = s;
    }
    if (R * sub > 0x7fffffff) return hipErrorInvalidValue;
    const int64_t per = R * sub < W ? R * sub : W;
    hipLaunchKernelGGL((dist_rows_kernel<PREC, LD>), dim3((unsigned)(8 * per)), dim3(kRowsThreads), 0, stream, a,
                       (uint32_t)R, (uint32_t)sub);
    return hipGetLastError();
}

hipError_t launch_dist_gemm_rows(const DistArgs &a, hipStream_t stream) {
    if (a.m == 0 || a.n == 0) return hipSuccess;
    if (!a.Qq || !a.Cq || (a.prec == kPrecFP8 && (!a.qscale || !a.cscale))) return hipErrorInvalidValue;
    if (rows_bytes(a) > a.ldq || rows_bytes(a) > 256 || a.n > (int64_t(1) << 29)) return hipErrorInvalidValue;
    const bool one = rows_bytes(a) == 128;
    if (a.prec == kPrecFP8)
        return one ? launch_rows_t<kPrecFP8, 128>(a, stream) : launch_rows_t<kPrecFP8, 256>(a, stream);
    if (a.prec != kPrecBF16) return hipErrorInvalidValue;
    return one ? launch_rows_t<kPrecBF16, 128>(a, stream) : launch_rows_t<kPrecBF16, 256>(a, stream);
}

}  // namespace knn
