// Distance kernels around the matrix-core product (Methods, "Distance
// calculation"): squared norms, unit vectors for the cosine and Pearson
// distances, reduced-precision operands, candidate bookkeeping, the
// certificate, and the exact direct-form re-rank of the surviving candidates
// (and of uncertified rows).  The product itself is in gemm.hip.
#include <algorithm>
#include <vector>

#include <cstdlib>
#include <cstring>
#include "dist.hpp"
#include "keys.hpp"

namespace knn {

// ---- unit vectors (cosine and Pearson distances) ------------------------------
// Methods, "Distance calculation": the cosine similarity of x and y is
// x.y / (|x| |y|), and Pearson's correlation is the cosine similarity of the
// vectors minus their means.  With u = x / |x| and v = y / |y|,
// 1 - cos = |u - v|^2 / 2, so both distances are half the squared Euclidean
// distance of unit vectors, and the Euclidean path ranks them unchanged.  One
// wave per row: lane-strided sums in a fixed order reduced by a lane tree; the
// norm is taken of the row scaled by its largest magnitude (no overflow or
// underflow in the squares), and every element is divided once.

// V > 0: rows of at most 64 V elements, held in registers, 64 / G of them to a
// wave (G lanes each; V = 1 below 64): one read and one write of memory.  V = 0:
// longer rows, read again for every step.  The sums run over the same elements in
// the same order either way.  Memory-bound: cosine searches, with a row read four
// times / once: 5003 x 150001 x 300 1795 / 1601 us, 16 x 10^6 x 128 697 / 489, 16 x
// 10^6 x 16 324 / 140 (half of that from four rows to a wave).
template <int V, int G>
__global__ __launch_bounds__(256) void unit_rows_kernel(const float *__restrict__ X, int64_t n, int d, int centre,
                                                        float *__restrict__ out) {
    const uint32_t lane = lane_id() % G;
    const int64_t i = ((int64_t)blockIdx.x * (256 / kWave) + threadIdx.x / kWave) * (kWave / G) + lane_id() / G;
    if (G == kWave && i >= n) return;
    const bool in = i < n;
    const float *x = X + (in ? i : n - 1) * d;
    float *o = out + i * d;
    float held[V > 0 ? V : 1];
    if (V > 0) {
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const int t = (int)lane + u * G;
            held[u] = t < d ? x[t] : 0.f;
        }
    }
    // f(element, its register) over this lane's elements, in order
    auto each = [&](auto f) {
        if constexpr (V > 0) {
#pragma unroll
            for (int u = 0; u < V; ++u)
                if ((int)lane + u * G < d) f((int)lane + u * G, held[u]);
        } else {
            for (int t = (int)lane; t < d; t += G) {
                float v = x[t];
                f(t, v);
            }
        }
    };
    auto tree = [&](float v, auto op) {
#pragma unroll
        for (int off = G / 2; off > 0; off >>= 1) v = op(v, shfl_xor_any(v, off));
        return v;
    };
    auto add = [](float p, float q) { return p + q; };
    auto low = [](float p, float q) { return fminf(p, q); };
    auto high = [](float p, float q) { return fmaxf(p, q); };
    float mu = 0.f;
    bool flat = false;
    if (centre) {
        float s = 0.f, lo = __uint_as_float(0x7f800000u), hi = -lo;
        each([&](int, float &v) {
            s += v;
            lo = fminf(lo, v);
            hi = fmaxf(hi, v);
        });
        mu = tree(s, add) / (float)d;
        // a constant row is exactly zero once centred, whatever the rounding of its mean
        flat = tree(lo, low) == tree(hi, high);
    }
    float amax = 0.f, nans = 0.f;
    each([&](int, float &v) {
        v = v - mu;
        nans = v != v ? 1.f : nans;
        amax = fmaxf(amax, fabsf(v));
    });
    amax = tree(amax, high);
    nans = tree(nans, high);
    const bool ok = !flat && nans == 0.f && amax > 0.f && amax <= 3.4028235e38f;
    float ss = 0.f;
    if (ok)
        each([&](int, float &v) {
            v = (V > 0 ? v : v - mu) / amax;
            ss = fmaf(v, v, ss);
        });
    const float nrm = sqrtf(tree(ss, add));
    const float qnan = __uint_as_float(0x7fc00000u);
    if (in)
        each([&](int t, float &v) { o[t] = ok ? (V > 0 ? v : (v - mu) / amax) / nrm : qnan; });
}

template <int V, int G>
static void launch_unit_t(const float *X, int64_t n, int d, bool centre, float *out, hipStream_t stream) {
    const int64_t per = 4 * (kWave / G);
    hipLaunchKernelGGL((unit_rows_kernel<V, G>), dim3((unsigned)((n + per - 1) / per)), dim3(256), 0, stream, X, n, d,
                       centre ? 1 : 0, out);
}

hipError_t launch_unit_rows(const float *X, int64_t n, int d, bool centre, float *out, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    if ((n + 3) / 4 > 0x7fffffffll) return hipErrorInvalidValue;
    if (d <= 16) launch_unit_t<1, 16>(X, n, d, centre, out, stream);
    else if (d <= 32) launch_unit_t<1, 32>(X, n, d, centre, out, stream);
    else if (d <= 64) launch_unit_t<1, 64>(X, n, d, centre, out, stream);
    else if (d <= 128) launch_unit_t<2, 64>(X, n, d, centre, out, stream);
    else if (d <= 256) launch_unit_t<4, 64>(X, n, d, centre, out, stream);
    else if (d <= 512) launch_unit_t<8, 64>(X, n, d, centre, out, stream);
    else if (d <= 1024) launch_unit_t<16, 64>(X, n, d, centre, out, stream);
    else launch_unit_t<0, 64>(X, n, d, centre, out, stream);
    return hipGetLastError();
}

// ---- squared norms ----------------------------------------------------------
// G lanes per point (the power of two covering the point's 16-byte chunks, or
// its elements without 16-byte loads; at most 64), 64 / G points per wave,
// grid-stride over points.  Each lane accumulates its strided elements in
// order, then a fixed xor-shuffle tree over the G lanes.  With max_bits, the
// largest norm (as FP32 bits; norms are non-negative) is folded into *max_bits
// with one atomic per workgroup.
// (src_n: the points are the n of src_n rows that source_row gives.)
__device__ __forceinline__ int64_t source_row(int64_t i, int64_t n, int64_t src_n) {
    return src_n ? (i * src_n) / n : i;
}

template <int G, bool VEC>
__device__ __forceinline__ void sqnorm_body(const float *__restrict__ X, int64_t n, int64_t src_n, int d,
                                            float *__restrict__ out, unsigned int *__restrict__ max_bits,
                                            uint32_t block, uint32_t blocks) {
    constexpr int PPW = kWave / G;
    __shared__ float wmax[256 / kWave];
    const uint32_t lane = lane_id(), sub = lane % G, grp = lane / G, wave = threadIdx.x / kWave;
    const int64_t stride = (int64_t)blocks * (256 / kWave) * PPW;
    float mx = 0.f;
    // two points per group per step (independent loads in flight)
    for (int64_t base = ((int64_t)block * (256 / kWave) + wave) * PPW; base < n; base += 2 * stride) {
        float acc[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int64_t i = base + u * stride + grp;
            float s = 0.f;
            if (i < n) {
                const float *x = X + source_row(i, n, src_n) * d;
                if (VEC) {
                    for (int t = (int)sub * 4; t < d; t += G * 4) {
                        const f32x4 v = *reinterpret_cast<const f32x4 *>(x + t);
                        s = fmaf(v[0], v[0], s);
                        s = fmaf(v[1], v[1], s);
                        s = fmaf(v[2], v[2], s);
                        s = fmaf(v[3], v[3], s);
                    }
                } else {
                    for (int t = (int)sub; t < d; t += G) s = fmaf(x[t], x[t], s);
                }
            }
            acc[u] = s;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int off = G / 2; off > 0; off >>= 1) acc[u] += shfl_xor_any(acc[u], off);
            const int64_t i = base + u * stride + grp;
            if (i < n && sub == 0) out[i] = acc[u];
            mx = fmaxf(mx, acc[u]);
        }
    }
    if (max_bits) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, shfl_xor_any(mx, off));
        if (lane == 0) wmax[wave] = mx;
        __syncthreads();
        if (threadIdx.x == 0) {
            float m = wmax[0];
            for (int w = 1; w < 256 / kWave; ++w) m = fmaxf(m, wmax[w]);
            atomicMax(max_bits, __float_as_uint(m));
        }
    }
}

template <int G, bool VEC>
__global__ __launch_bounds__(256) void sqnorm_kernel(const float *__restrict__ X, int64_t n, int d,
                                                     float *__restrict__ out, unsigned int *__restrict__ max_bits) {
    sqnorm_body<G, VEC>(X, n, 0, d, out, max_bits, blockIdx.x, gridDim.x);
}

// ---- FP32 operands as two FP16 halves ----------------------------------------
// The point scaled by 2^e, its largest finite magnitude into [2^14, 2^15) (e in
// [-113, 126]; 0 for a zero point; at e = 126, magnitudes below 2^-111, two halves
// still hold what an FP32 element holds), each element as h = FP16(x 2^e) and l =
// FP16(x 2^e - h), both to nearest even; the subtraction is exact.  A
// non-finite element keeps its infinity or NaN in h with l = 0.  The squared
// norms come from the same read, in sqnorm_kernel's order.  Memory-bound: 4 d
// bytes read (the second pass over a row finds it in L1) and 4 d written per
// point, against the d^2-fold work of the product it feeds.
template <int G, bool VEC>
__device__ __forceinline__ void split_body(const float *__restrict__ X, int64_t n, int64_t src_n, int d,
                                           unsigned char *__restrict__ out, int64_t ldo, float *__restrict__ scale_out,
                                           float *__restrict__ norm, unsigned int *__restrict__ max_bits,
                                           uint32_t block, uint32_t blocks) {
    constexpr int PPW = kWave / G;
    __shared__ float wmax[256 / kWave];
    const uint32_t lane = lane_id(), sub = lane % G, grp = lane / G, wave = threadIdx.x / kWave;
    const int64_t stride = (int64_t)blocks * (256 / kWave) * PPW;
    const int dp = (d + 31) / 32 * 32;
    float mx = 0.f;
    for (int64_t base = ((int64_t)block * (256 / kWave) + wave) * PPW; base < n; base += stride) {
        const int64_t i = base + grp;
        const bool in = i < n;
        const float *x = X + source_row(in ? i : n - 1, n, src_n) * d;
        float s = 0.f, am = 0.f;
        auto see = [&](float v) {
            s = fmaf(v, v, s);
            const float a = fabsf(v);
            if (a <= 3.4028235e38f) am = fmaxf(am, a);  // finite magnitudes only
        };
        if (VEC) {
            for (int t = (int)sub * 4; t < d; t += G * 4) {
                const f32x4 v = *reinterpret_cast<const f32x4 *>(x + t);
#pragma unroll
                for (int c = 0; c < 4; ++c) see(v[c]);
            }
        } else {
            for (int t = (int)sub; t < d; t += G) see(x[t]);
        }
#pragma unroll
        for (int off = G / 2; off > 0; off >>= 1) {
            s += shfl_xor_any(s, off);
            am = fmaxf(am, shfl_xor_any(am, off));
        }
        int e = 0;
        if (am > 0.f) {
            int E;
            (void)frexpf(am, &E);  // am = f 2^E, f in [0.5, 1)
            e = 15 - E;
            e = e < -113 ? -113 : (e > 126 ? 126 : e);
        }
        const float up = ldexpf(1.0f, e);
        if (in && sub == 0) {
            scale_out[i] = ldexpf(1.0f, -e);
            if (norm) norm[i] = s;
        }
        if (in) mx = fmaxf(mx, s);
        unsigned char *o = out + (in ? i : n - 1) * ldo;
        auto halves = [&](float v, _Float16 &hi, _Float16 &lo) {
            const float y = v * up;
            hi = (_Float16)y;
            const float r = y - (float)hi;
            lo = r == r ? (_Float16)r : (_Float16)0.f;  // (inf - inf and NaN: no low half)
        };
        typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
        if (VEC) {
            for (int t = (int)sub * 4; t < dp; t += G * 4) {
                f32x4 v = {0.f, 0.f, 0.f, 0.f};
                if (t < d) v = *reinterpret_cast<const f32x4 *>(x + t);
                f16x4 hi, lo;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    _Float16 a, b;
                    halves(v[c], a, b);
                    hi[c] = a;
                    lo[c] = b;
                }
                unsigned char *p = o + (t / 32) * 128 + (t % 32) * 2;
                if (in) {
                    *reinterpret_cast<f16x4 *>(p) = hi;
                    *reinterpret_cast<f16x4 *>(p + 64) = lo;
                }
            }
        } else {
            for (int t = (int)sub; t < dp; t += G) {
                _Float16 a, b;
                halves(t < d ? x[t] : 0.f, a, b);
                unsigned char *p = o + (t / 32) * 128 + (t % 32) * 2;
                if (in) {
                    *reinterpret_cast<_Float16 *>(p) = a;
                    *reinterpret_cast<_Float16 *>(p + 64) = b;
                }
            }
        }
    }
    if (max_bits) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, shfl_xor_any(mx, off));
        if (lane == 0) wmax[wave] = mx;
        __syncthreads();
        if (threadIdx.x == 0) {
            float m = wmax[0];
            for (int w = 1; w < 256 / kWave; ++w) m = fmaxf(m, wmax[w]);
            atomicMax(max_bits, __float_as_uint(m));
        }
    }
}

template <int G, bool VEC>
__global__ __launch_bounds__(256) void split_rows_kernel(const float *__restrict__ X, int64_t n, int64_t src_n, int d,
                                                         unsigned char *__restrict__ out, int64_t ldo,
                                                         float *__restrict__ scale_out, float *__restrict__ norm,
                                                         unsigned int *__restrict__ max_bits) {
    split_body<G, VEC>(X, n, src_n, d, out, ldo, scale_out, norm, max_bits, blockIdx.x, gridDim.x);
}

// Lanes per point or candidate for a row length d: the power of two covering
// its 16-byte chunks (or its elements), at most a wave.
static int lanes_for(int d, bool vec) {
    const int units = vec ? (d + 3) / 4 : d;
    int g = 1;
    while (g < units && g < kWave) g <<= 1;
    return g;
}

// ---- gather rows (and their norms) -----------------------------------------
// dst row t = src row idx[t] (idx null: row floor(t * n / rows)).
__global__ __launch_bounds__(256) void gather_rows_kernel(const float *__restrict__ src, int64_t n, int d,
                                                          const int32_t *__restrict__ idx, int64_t rows,
                                                          float *__restrict__ dst, const float *__restrict__ norms,
                                                          float *__restrict__ dst_norms) {
    const int64_t t = (int64_t)blockIdx.x * 4 + threadIdx.x / kWave;
    if (t >= rows) return;
    const int64_t s = idx ? (int64_t)idx[t] : (t * n) / rows;
    const uint32_t lane = lane_id();
    for (int c = lane; c < d; c += kWave) dst[t * d + c] = src[s * d + c];
    if (norms && lane == 0) dst_norms[t] = norms[s];
}

// ---- candidate bookkeeping ----------------------------------------------------
// Rows whose candidate count is below `need` or above `cap` are listed for the
// exact fallback.
// The counts are summed on the way.
__device__ __forceinline__ void flag_body(const FlagSeg &a, int64_t i) {
    const uint32_t c = i < a.m ? a.cnt[i] : 0u;
    if (i < a.m && (a.force || c < a.need || c > a.cap)) {
        uint32_t p = atomicAdd(a.nflag, 1u);
        a.flags[p] = (int32_t)i;
    }
    // (256 counts of at most 2^31 - 1: in 64 bits from the waves on)
    unsigned long long t = c;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off);
    if (lane_id() == 0 && t) atomicAdd(a.total, t);
}
__global__ __launch_bounds__(256) void flag_rows_kernel(FlagSeg a) {
    flag_body(a, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// Replaces the candidate lists of the flagged rows by the exact selection made
// on their materialised distance rows.
__global__ __launch_bounds__(256) void scatter_fallback_kernel(const int32_t *__restrict__ rows, int64_t nrows,
                                                               const float *__restrict__ val,
                                                               const int32_t *__restrict__ idx, int kk,
                                                               uint64_t *__restrict__ cand, uint32_t *__restrict__ cnt,
                                                               int cap) {
    const int64_t f = blockIdx.x;
    if (f >= nrows) return;
    const int64_t i = rows[f];
    for (int t = threadIdx.x; t < kk; t += blockDim.x)
        cand[i * cap + t] = make_key(val[f * kk + t], (uint32_t)idx[f * kk + t]);
    if (threadIdx.x == 0) cnt[i] = (uint32_t)kk;
}

// ---- exact re-rank ----------------------------------------------------------
// One workgroup per query: the exact FP32 squared distance sum_t (q_t - c_t)^2
// to each of the row's kk candidates, then a bitonic sort of the (distance,
// index) keys; the first k are written (missing entries: +inf, index -1).
// G lanes per candidate (the power of two covering d's 16-byte chunks, at
// most a wave), so a wave works on 64 / G candidates at once, two per lane
// group per step to keep more loads in flight; each lane accumulates its
// strided elements in order, then a fixed xor-shuffle tree over the G lanes.
//
// Bound by the gather of the candidates' rows.  With FP32 keys most of the kk =
// 4 k candidates cannot be among the k smallest: a key is within E of its exact
// value (E: see CertifyArgs) and a direct-form sum within gamma (|q| + max|c|)^2
// of the exact distance, so a candidate whose key exceeds the k-th by more than
// twice both bounds has a larger direct-form distance than the k first, and its
// row is not read (32768 rows, d = 1024, k' = 128, k = 32: 2.52 -> 0.83 ms;
// about 36 candidates of 128 are left).
constexpr int kRerankThreads = 256;
constexpr int kRerankMax = 1024;

constexpr float kKeyU2 = 2.0f * 5.9604645e-8f;  // 2^-23: the final fused multiply-add of a key

template <int G, bool VEC>
__device__ __forceinline__ float rerank_dist(const float *__restrict__ q, const float *__restrict__ y, int d,
                                             uint32_t sub) {
    float s = 0.f;
    if (VEC) {
        for (int t = (int)sub * 4; t < d; t += G * 4) {
            const f32x4 qv = *reinterpret_cast<const f32x4 *>(q + t);
            const f32x4 yv = *reinterpret_cast<const f32x4 *>(y + t);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float df = qv[e] - yv[e];
                s = fmaf(df, df, s);
            }
        }
    } else {
        for (int t = (int)sub; t < d; t += G) {
            const float df = q[t] - y[t];
            s = fmaf(df, df, s);
        }
    }
    return s;
}

// The certificate of row i (RerankArgs), whose k-th candidate by distance is
// `kth`.  In FP64: nothing is added to the bounds for their own evaluation.
__device__ __forceinline__ void rerank_certify(const RerankArgs &a, int64_t i, uint64_t kth) {
    const double u2 = kKeyU2, g = a.gamma, gd = g + 2.0 * u2;
    const double q2 = a.qnorm2[i], c2 = __uint_as_float(*a.cmax2_bits), qc = sqrt(q2 * c2);
    // (1.001: norms and products of them that are themselves rounded)
    const double nrm = (g + u2) * c2, E = 1.001 * (nrm + 2.0 * (a.rel + u2) * qc);
    const double Ef = 1.001 * (nrm + 2.0 * (a.rel_fix + u2) * qc);
    const float *key = a.keys + i * a.kk;
    double U = (double)key[a.k - 1] + E;
    const double byd = (double)ord_to_float(key_ord(kth)) / (1.0 - gd) - q2 * (1.0 - g);
    if (byd < U) U = byd;  // (false for NaN)
    if (!a.force && (double)key[a.kk - 1] - E > U) return;
    const double t = U + Ef;
    float tf = (float)t;
    if ((double)tf < t) tf = nextafterf(tf, __uint_as_float(0x7f800000u));
    a.tfix[i] = tf;
    a.ulist[atomicAdd(a.nu, 1u)] = (int32_t)i;
}

template <int G, bool VEC>
__device__ __forceinline__ void rerank_body(const RerankArgs &a, int64_t i) {
    constexpr uint32_t PPW = kWave / G;                       // candidates per wave per pass
    constexpr uint32_t STEP = (kRerankThreads / kWave) * PPW;  // per workgroup per pass
    __shared__ uint64_t keys[kRerankMax];
    if (i >= a.m) return;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave, sub = lane % G, grp = lane / G;
    const float *q = a.Q + i * a.d;
    const int32_t *ci = a.cidx + i * a.kk;
    uint32_t kk = a.kk;
    if (a.keys) {
        const float *key = a.keys + i * a.kk;
        const float c2 = __uint_as_float(*a.cmax2_bits), q2 = a.qnorm2[i], cm = sqrtf(c2), qm = sqrtf(q2);
        const float E = (a.gamma + kKeyU2) * c2 + 2.0f * (a.rel + kKeyU2) * qm * cm;
        // (1.001: slack for the FP32 evaluation; 4 u: the differences, products
        // and the last sums of the direct form)
        const float ak = key[a.k - 1], T = ak + 2.002f * (E + (a.gamma + 2.0f * kKeyU2) * (qm + cm) * (qm + cm));
        if (fabsf(T) <= 3.4028235e38f) {  // a bound exists (false for NaN): the keys up to T, in order
            kk = 0;
            for (uint32_t t0 = 0; t0 < a.kk; t0 += kRerankThreads) {
                const uint32_t t = t0 + tid;
                const int c = __syncthreads_count(t < a.kk && key[t] <= T);
                kk += (uint32_t)c;
                if (c < kRerankThreads) break;
            }
        }
    }
    const int64_t own = a.self_offset >= 0 ? a.self_offset + i : (int64_t)-1;
    for (uint32_t c0 = wave * PPW + grp; c0 < kk; c0 += 2 * STEP) {
        const uint32_t c1 = c0 + STEP;
        const uint32_t j0 = (uint32_t)ci[c0];
        const uint32_t j1 = c1 < kk ? (uint32_t)ci[c1] : 0xFFFFFFFFu;
        // missing candidates (never for valid lists) and the query's own index
        // (a candidate only when its row has no other finite key) are dropped
        const bool ok0 = (int64_t)j0 < a.n && (int64_t)j0 != own, ok1 = (int64_t)j1 < a.n && (int64_t)j1 != own;
        float s0 = ok0 ? rerank_dist<G, VEC>(q, a.C + (int64_t)j0 * a.d, a.d, sub) : 0.f;
        float s1 = ok1 ? rerank_dist<G, VEC>(q, a.C + (int64_t)j1 * a.d, a.d, sub) : 0.f;
#pragma unroll
        for (int off = G / 2; off > 0; off >>= 1) {
            s0 += shfl_xor_any(s0, off);
            s1 += shfl_xor_any(s1, off);
        }
        if (sub == 0) {
            keys[c0] = ok0 ? make_key(s0, j0) : kKeyMax;
            if (c1 < kk) keys[c1] = ok1 ? make_key(s1, j1) : kKeyMax;
        }
    }
    __syncthreads();
    block_sort<kRerankThreads>(keys, kk);
    if (a.ulist && tid == 0) rerank_certify(a, i, a.k <= (int)kk ? keys[a.k - 1] : kKeyMax);
    for (uint32_t t = tid; t < (uint32_t)a.k; t += kRerankThreads) {
        const uint64_t key = t < kk ? keys[t] : kKeyMax;
        if (key == kKeyMax) {
            a.out_dist[i * a.k + t] = __uint_as_float(0x7f800000u);
            a.out_idx[i * a.k + t] = -1;
        } else {
            a.out_dist[i * a.k + t] = a.out_scale * ord_to_float(key_ord(key));
            a.out_idx[i * a.k + t] = (int32_t)key_idx(key);
        }
    }
}

template <int G, bool VEC>
__global__ __launch_bounds__(kRerankThreads) void rerank_kernel(RerankArgs a) {
    rerank_body<G, VEC>(a, blockIdx.x);
}

// ---- reduced-precision operands ---------------------------------------------
// OCP e4m3 (1 sign, 4 exponent bits with bias 7, 3 mantissa bits, no infinity),
// round to nearest even, saturating at +-448 (also for infinities); a NaN
// becomes the NaN code S.1111.111.
__device__ __forceinline__ uint8_t f32_to_e4m3(float x) {
    const uint8_t sign = (uint8_t)((__float_as_uint(x) >> 24) & 0x80u);
    const float a = fabsf(x);
    if (a != a) return sign | 0x7Fu;
    if (!(a < 448.0f)) return sign | 0x7Eu;
    if (a < 0.015625f) {                               // below 2^-6: subnormals, step 2^-9
        return sign | (uint8_t)rintf(a * 512.0f);      // 8 (= 2^-6) encodes the smallest normal
    }
    int e = (int)((__float_as_uint(a) >> 23) & 0xFFu) - 127;  // floor(log2 a), in [-6, 8]
    float r = rintf(ldexpf(a, 3 - e));                 // mantissa with the hidden bit, in [8, 16]
    if (r >= 16.0f) {
        r = 8.0f;
        e += 1;
    }
    if (e > 8 || (e == 8 && r > 14.0f)) return sign | 0x7Eu;
    return sign | (uint8_t)(((e + 7) << 3) | ((int)r - 8));
}

// BF16 by round to nearest even on the low 16 bits; a NaN stays a quiet NaN
// (the rounding carry could otherwise turn a NaN with only low payload bits
// into an infinity).
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if (f != f) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// FP8: e = the largest integer with amax * 2^e <= 448, amax the largest finite
// magnitude of the point (e = 0 without a finite non-zero element; e limited to
// [-100, 100]), elements x * 2^e rounded to e4m3, scale 2^-e.  The squared norms
// come from the same read, in sqnorm_kernel's order and lane grouping.
// Memory-bound (FP8's second pass over a row finds it in L1).  whole: out is
// aligned to 8 bytes (a caller's own buffer may not be).
template <int G, bool VEC>
__device__ __forceinline__ void quantize_body(const float *__restrict__ X, int64_t n, int64_t src_n, int d, int prec,
                                              void *__restrict__ out, float *__restrict__ scale_out,
                                              float *__restrict__ norm, unsigned int *__restrict__ max_bits,
                                              uint32_t block, uint32_t blocks, bool whole) {
    constexpr int PPW = kWave / G, W = VEC ? 4 : 1;
    __shared__ float wmax[256 / kWave];
    const uint32_t lane = lane_id(), sub = lane % G, grp = lane / G, wave = threadIdx.x / kWave;
    const int64_t stride = (int64_t)blocks * (256 / kWave) * PPW;
    const int dq = (d + kQuantPad - 1) / kQuantPad * kQuantPad;
    const bool fp8 = prec == kPrecFP8;
    float mx = 0.f;
    for (int64_t base = ((int64_t)block * (256 / kWave) + wave) * PPW; base < n; base += stride) {
        const int64_t i = base + grp;
        const bool in = i < n;
        const float *x = X + source_row(in ? i : n - 1, n, src_n) * d;
        // f(t, V elements from t on, zeros beyond the row) over this lane's part, V =
        // W for the sums; operands are written four at a time either way
        auto each = [&](auto width, int end, auto f) {
            constexpr int V = decltype(width)::value;
            for (int t = (int)sub * V; t < end; t += G * V) {
                f32x4 v = {0.f, 0.f, 0.f, 0.f};
                if constexpr (VEC) {
                    if (t < d) v = *reinterpret_cast<const f32x4 *>(x + t);
                } else if constexpr (V == 1) {
                    if (t < d) v[0] = x[t];
                } else {
                    typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
                    if (t + 4 <= d) {
                        v = *reinterpret_cast<const f32x4_any *>(x + t);
                    } else {
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (t + c < d) v[c] = x[t + c];
                    }
                }
                f(t, v);
            }
        };
        const std::integral_constant<int, W> wide{};
        const std::integral_constant<int, 4> four{};
        float s = 0.f, amax = 0.f;
        auto see = [&](const f32x4 &v) {
#pragma unroll
            for (int c = 0; c < W; ++c) {
                s = fmaf(v[c], v[c], s);
                const float m = fabsf(v[c]);
                if (m <= 3.4028235e38f) amax = fmaxf(amax, m);  // finite magnitudes only
            }
        };
        unsigned char *const o = static_cast<unsigned char *>(out) + (in ? i : n - 1) * dq * (fp8 ? 1 : 2);
        if (!VEC || fp8) each(wide, d, [&](int, const f32x4 &v) { see(v); });
        if (!fp8)
            each(four, dq, [&](int t, const f32x4 &v) {
                if (VEC && t < d) see(v);  // (one pass)
                typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
                u16x4 q;
#pragma unroll
                for (int c = 0; c < 4; ++c) q[c] = f32_to_bf16_rne(v[c]);
                if (!in) return;
                if (whole) {
                    *reinterpret_cast<u16x4 *>(o + 2 * t) = q;
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) reinterpret_cast<uint16_t *>(o)[t + c] = q[c];
                }
            });
#pragma unroll
        for (int off = G / 2; off > 0; off >>= 1) {
            s += shfl_xor_any(s, off);
            amax = fmaxf(amax, shfl_xor_any(amax, off));
        }
        if (in && norm && sub == 0) norm[i] = s;
        if (in) mx = fmaxf(mx, s);
        if (!fp8) continue;
        int e = 0;
        if (amax > 0.f) {
            // amax = f 2^E with f in [0.5, 1): amax 2^e <= 448 = 0.875 * 2^9 exactly
            // when e <= 9 - E, less one when f > 0.875
            int E;
            const float f = frexpf(amax, &E);
            e = 9 - E - (f > 0.875f ? 1 : 0);
            e = e < -100 ? -100 : (e > 100 ? 100 : e);
        }
        each(four, dq, [&](int t, const f32x4 &v) {
            uint32_t q = 0;
            if (t < d) {  // (the padding of a short row is most of it)
#pragma unroll
                for (int c = 0; c < 4; ++c) q |= (uint32_t)f32_to_e4m3(ldexpf(v[c], e)) << (8 * c);
            }
            if (!in) return;
            if (whole) {
                *reinterpret_cast<uint32_t *>(o + t) = q;
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) o[t + c] = (unsigned char)(q >> (8 * c));
            }
        });
        if (in && sub == 0) scale_out[i] = ldexpf(1.0f, -e);
    }
    if (max_bits) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, shfl_xor_any(mx, off));
        if (lane == 0) wmax[wave] = mx;
        __syncthreads();
        if (threadIdx.x == 0) {
            float m = wmax[0];
            for (int w = 1; w < 256 / kWave; ++w) m = fmaxf(m, wmax[w]);
            // (most workgroups find a larger one there: no atomic)
            if (__float_as_uint(m) > __hip_atomic_load(max_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                atomicMax(max_bits, __float_as_uint(m));
        }
    }
}
template <int G, bool VEC>
__global__ __launch_bounds__(256) void quantize_kernel(const float *__restrict__ X, int64_t n, int64_t src_n, int d,
                                                       int prec, void *__restrict__ out, float *__restrict__ scale_out,
                                                       float *__restrict__ norm, unsigned int *__restrict__ max_bits,
                                                       bool whole) {
    quantize_body<G, VEC>(X, n, src_n, d, prec, out, scale_out, norm, max_bits, blockIdx.x, gridDim.x, whole);
}

// Per-row candidate certificate (see launch_certify in dist.hpp for the bound).
__device__ __forceinline__ void certify_body(const CertifyArgs &a, int64_t i) {
    bool bad = false;
    if (i < a.m) {
        const float ak = a.sorted_keys[i * a.kk + a.k - 1];
        const float gap = a.sorted_keys[i * a.kk + a.kk - 1] - ak;
        const float c2 = __uint_as_float(*a.cmax2_bits), cm = sqrtf(c2), qm = sqrtf(a.qnorm2[i]);
        // 1.001: slack for the FP32 evaluation of the bound itself
        const float E = 1.001f * ((a.gamma + kKeyU2) * c2 + 2.0f * (a.rel + kKeyU2) * qm * cm);
        bad = !(gap > 2.0f * E);
    }
    const uint64_t b = __ballot(bad);
    if (lane_id() == 0 && b) atomicAdd(a.count, (unsigned long long)__popcll(b));
}

__global__ __launch_bounds__(256) void certify_kernel(CertifyArgs a) {
    certify_body(a, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

// ---- exact re-run of uncertified rows ------------------------------------------
// One workgroup per listed row.  The row's reduced keys are scanned in tiles of
// 1024; columns at or below the threshold are compacted into LDS (ballot +
// population count, one LDS reservation per wave) and, once 1024 or more are
// pending, re-ranked by exact distance, sorted and merged into the running
// 1024 smallest (distance, index) keys: the elementwise minimum of the
// ascending running list and the reversed lower half of the sorted batch holds
// exactly the 1024 smallest of both, as a bitonic sequence, which ten
// half-cleaning steps sort.
constexpr int kFixThreads = 256;
constexpr int kFixTop = 1024;
constexpr int kFixBatch = 2048;

template <int G, bool VEC>
__global__ __launch_bounds__(kFixThreads) void exact_rows_kernel(FixupArgs a) {
    constexpr uint32_t PPW = kWave / G;
    constexpr uint32_t STEP = (kFixThreads / kWave) * PPW;
    __shared__ uint64_t top[kFixTop];
    __shared__ uint64_t batch[kFixBatch];
    __shared__ uint32_t cidx[kFixBatch];
    __shared__ uint32_t cnt;
    const int64_t f = blockIdx.x;
    if (f >= a.nrows) return;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave, sub = lane % G, grp = lane / G;
    const int64_t i = a.rows[f];
    const float *drow = a.D + (a.by_row ? i : f) * a.ldd;
    const float T = a.tfix[i];
    const bool bounded = fabsf(T) <= 3.4028235e38f;  // finite (false for NaN)
    const float *q = a.Q + i * a.d;
    const int64_t own = a.self_offset >= 0 ? a.self_offset + i : (int64_t)-1;
    for (uint32_t t = tid; t < (uint32_t)kFixTop; t += kFixThreads) top[t] = kKeyMax;
    if (tid == 0) cnt = 0;
    __syncthreads();

    auto flush = [&](uint32_t c) {
        for (uint32_t c0 = wave * PPW + grp; c0 < c; c0 += STEP) {
            const uint32_t j = cidx[c0];
            float s = rerank_dist<G, VEC>(q, a.C + (int64_t)j * a.d, a.d, sub);
#pragma unroll
            for (int off = G / 2; off > 0; off >>= 1) s += shfl_xor_any(s, off);
            if (sub == 0) batch[c0] = (int64_t)j == own ? kKeyMax : make_key(s, j);
        }
        for (uint32_t t = c + tid; t < (uint32_t)kFixTop; t += kFixThreads) batch[t] = kKeyMax;
        __syncthreads();
        block_sort<kFixThreads, 8>(batch, c < (uint32_t)kFixTop ? (uint32_t)kFixTop : c);
        for (uint32_t t = tid; t < (uint32_t)kFixTop; t += kFixThreads) {
            const uint64_t x = top[t], y = batch[kFixTop - 1 - t];
            top[t] = x < y ? x : y;
        }
        __syncthreads();
        for (uint32_t st = kFixTop / 2; st > 0; st >>= 1) {
            for (uint32_t t = tid; t < (uint32_t)kFixTop / 2; t += kFixThreads) {
                const uint32_t lo = (t / st) * 2 * st + t % st, hi = lo + st;
                const uint64_t x = top[lo], y = top[hi];
                if (y < x) {
                    top[lo] = y;
                    top[hi] = x;
                }
            }
            __syncthreads();
        }
    };

    constexpr uint32_t kTileCols = 4 * kFixThreads;
    for (int64_t j0 = 0; j0 < a.n; j0 += kTileCols) {
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) {
            const int64_t j = j0 + u * kFixThreads + tid;
            const bool valid = j < a.n;
            const float v = valid ? drow[j] : 0.f;
            const bool pass = valid && (!bounded || v <= T);
            const uint64_t m = __ballot(pass);
            if (m) {
                uint32_t base = 0;
                if (lane == 0) base = atomicAdd(&cnt, (uint32_t)__popcll(m));
                base = wave_bcast0(base);
                if (pass) cidx[base + lanes_below(m)] = (uint32_t)j;
            }
        }
        __syncthreads();
        const uint32_t c = cnt;
        __syncthreads();
        if (c > 0 && (c >= (uint32_t)kFixTop || j0 + kTileCols >= a.n)) {
            flush(c);
            if (tid == 0) cnt = 0;
            __syncthreads();
        }
    }
    for (uint32_t t = tid; t < (uint32_t)a.k; t += kFixThreads) {
        const uint64_t key = top[t];
        const int64_t o = i * a.k + t;
        if (key == kKeyMax) {
            a.out_dist[o] = __uint_as_float(0x7f800000u);
            a.out_idx[o] = -1;
        } else {
            a.out_dist[o] = a.out_scale * ord_to_float(key_ord(key));
            a.out_idx[o] = (int32_t)key_idx(key);
        }
    }
}

// Workgroups for n points of G lanes each.
static int64_t sqnorm_blocks(int64_t n, int G) {
    const int64_t b = (n * G + 8 * kWave - 1) / (8 * kWave);
    return b > 4096 ? 4096 : b;
}
static int64_t split_blocks(int64_t n, int G) {
    const int64_t b = (n * G + 4 * kWave - 1) / (4 * kWave);
    return b > 8192 ? 8192 : b;
}

// (rows without 16-byte loads are longer chains of loads, sums and stores: more of
// them at a time.  Whole searches, at most 8192 / 65536 workgroups: 50 x 214506 x
// 39 BF16 247 / 213 us, 747 x 274103 x 27 267 / 214; with 16-byte loads 16 x 10^6 x
// 128 FP8 425 / 464)
static int64_t quantize_blocks(int64_t n, int G, bool vec) {
    const int64_t b = (n * G + 4 * kWave - 1) / (4 * kWave), most = vec ? 8192 : 65536;
    return b > most ? most : b;
}

template <int G>
static void launch_sqnorm_g(const float *X, int64_t n, int d, float *out, unsigned int *max_bits, bool vec,
                            hipStream_t stream) {
    const int64_t blocks = sqnorm_blocks(n, G);
    if (vec)
        hipLaunchKernelGGL((sqnorm_kernel<G, true>), dim3((unsigned)blocks), dim3(256), 0, stream, X, n, d, out,
                           max_bits);
    else
        hipLaunchKernelGGL((sqnorm_kernel<G, false>), dim3((unsigned)blocks), dim3(256), 0, stream, X, n, d, out,
                           max_bits);
}

hipError_t launch_sqnorm(const float *X, int64_t n, int d, float *out, unsigned int *max_bits, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const bool vec = d % 4 == 0 && (reinterpret_cast<uintptr_t>(X) & 15u) == 0;
    switch (lanes_for(d, vec)) {
        case 1: launch_sqnorm_g<1>(X, n, d, out, max_bits, vec, stream); break;
        case 2: launch_sqnorm_g<2>(X, n, d, out, max_bits, vec, stream); break;
        case 4: launch_sqnorm_g<4>(X, n, d, out, max_bits, vec, stream); break;
        case 8: launch_sqnorm_g<8>(X, n, d, out, max_bits, vec, stream); break;
        case 16: launch_sqnorm_g<16>(X, n, d, out, max_bits, vec, stream); break;
        case 32: launch_sqnorm_g<32>(X, n, d, out, max_bits, vec, stream); break;
        default: launch_sqnorm_g<64>(X, n, d, out, max_bits, vec, stream); break;
    }
    return hipGetLastError();
}

template <int G>
static void launch_split_g(const float *X, int64_t n, int64_t src_n, int d, void *out, float *sc, float *norm,
                           unsigned int *max_bits, bool vec, hipStream_t stream) {
    const int64_t blocks = split_blocks(n, G);
    unsigned char *o = static_cast<unsigned char *>(out);
    const int64_t ldo = split_row_bytes(d);
    if (vec)
        hipLaunchKernelGGL((split_rows_kernel<G, true>), dim3((unsigned)blocks), dim3(256), 0, stream, X, n, src_n,
                           d, o, ldo, sc, norm, max_bits);
    else
        hipLaunchKernelGGL((split_rows_kernel<G, false>), dim3((unsigned)blocks), dim3(256), 0, stream, X, n, src_n,
                           d, o, ldo, sc, norm, max_bits);
}

hipError_t launch_split(const float *X, int64_t n, int d, void *out, float *scale_out, float *norm,
                        unsigned int *max_bits, hipStream_t stream, int64_t src_n) {
    if (n == 0) return hipSuccess;
    const bool vec = d % 4 == 0 && (reinterpret_cast<uintptr_t>(X) & 15u) == 0;
    // (the lane grouping of launch_sqnorm, so that the norms are the same bits)
    switch (lanes_for(d, vec)) {
        case 16: launch_split_g<16>(X, n, src_n, d, out, scale_out, norm, max_bits, vec, stream); break;
        case 32: launch_split_g<32>(X, n, src_n, d, out, scale_out, norm, max_bits, vec, stream); break;
        case 64: launch_split_g<64>(X, n, src_n, d, out, scale_out, norm, max_bits, vec, stream); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_gather_rows(const float *src, int64_t n, int d, const int32_t *idx, int64_t rows, float *dst,
                              const float *norms, float *dst_norms, hipStream_t stream) {
    if (rows == 0) return hipSuccess;
    hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, stream, src, n, d, idx,
                       rows, dst, norms, dst_norms);
    return hipGetLastError();
}

hipError_t launch_flag_rows(const uint32_t *cnt, int64_t m, uint32_t need, uint32_t cap, int force, uint32_t *nflag,
                            int32_t *flags, unsigned long long *total, hipStream_t stream) {
    if (m == 0) return hipSuccess;
    hipLaunchKernelGGL(flag_rows_kernel, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, stream,
                       FlagSeg{cnt, m, need, cap, force, nflag, flags, total});
    return hipGetLastError();
}

hipError_t launch_scatter_fallback(const int32_t *rows, int64_t nrows, const float *val, const int32_t *idx, int kk,
                                   uint64_t *cand, uint32_t *cnt, int cap, hipStream_t stream) {
    if (nrows == 0) return hipSuccess;
    hipLaunchKernelGGL(scatter_fallback_kernel, dim3((unsigned)nrows), dim3(256), 0, stream, rows, nrows, val, idx, kk,
                       cand, cnt, cap);
    return hipGetLastError();
}

template <int G>
static void launch_quantize_g(const float *X, int64_t n, int64_t src_n, int d, int prec, void *out, float *sc,
                              float *norm, unsigned int *max_bits, bool vec, hipStream_t stream) {
    const dim3 g((unsigned)quantize_blocks(n, G, vec)), b(256);
    const bool whole = (reinterpret_cast<uintptr_t>(out) & 7u) == 0;
    if (vec)
        hipLaunchKernelGGL((quantize_kernel<G, true>), g, b, 0, stream, X, n, src_n, d, prec, out, sc, norm, max_bits,
                           whole);
    else
        hipLaunchKernelGGL((quantize_kernel<G, false>), g, b, 0, stream, X, n, src_n, d, prec, out, sc, norm, max_bits,
                           whole);
}

hipError_t launch_quantize(const float *X, int64_t n, int d, int prec, void *out, float *scale_out,
                           hipStream_t stream, float *norm, unsigned int *max_bits, int64_t src_n) {
    if (n == 0) return hipSuccess;
    const bool vec = d % 4 == 0 && (reinterpret_cast<uintptr_t>(X) & 15u) == 0;
    switch (lanes_for(d, vec)) {
        case 1: launch_quantize_g<1>(X, n, src_n, d, prec, out, scale_out, norm, max_bits, vec, stream); break;
        case 2: launch_quantize_g<2>(X, n, src_n, d, prec, out, scale_out, norm, max_bits, vec, stream); break;
        case 4: launch_quantize_g<4>(X, n, src_n, d, prec, out, scale_out, norm, max_bits, vec, stream); break;
        case 8: launch_quantize_g<8>(X, n, src_n, d, prec, out, scale_out, norm, max_bits, vec, stream); break;
        case 16: launch_quantize_g<16>(X, n, src_n, d, prec, out, scale_out, norm, max_bits, vec, stream); break;
        case 32: launch_quantize_g<32>(X, n, src_n, d, prec, out, scale_out, norm, max_bits, vec, stream); break;
        default: launch_quantize_g<64>(X, n, src_n, d, prec, out, scale_out, norm, max_bits, vec, stream); break;
    }
    return hipGetLastError();
}

hipError_t launch_certify(const CertifyArgs &a, hipStream_t stream) {
    if (a.m == 0) return hipSuccess;
    hipLaunchKernelGGL(certify_kernel, dim3((unsigned)((a.m + 255) / 256)), dim3(256), 0, stream, a);
    return hipGetLastError();
}

template <int G>
static void launch_fixup_g(const FixupArgs &a, bool vec, hipStream_t stream) {
    if (vec)
        hipLaunchKernelGGL((exact_rows_kernel<G, true>), dim3((unsigned)a.nrows), dim3(kFixThreads), 0, stream, a);
    else
        hipLaunchKernelGGL((exact_rows_kernel<G, false>), dim3((unsigned)a.nrows), dim3(kFixThreads), 0, stream, a);
}

hipError_t launch_fixup(const FixupArgs &a, hipStream_t stream) {
    if (a.nrows == 0) return hipSuccess;
    if (a.k < 1 || a.k > kFixTop || a.nrows > 0x7fffffff) return hipErrorInvalidValue;
    // the same lane grouping as the re-rank, so a pair's distance has the same bits
    const bool vec = a.d % 4 == 0 && (reinterpret_cast<uintptr_t>(a.Q) & 15u) == 0 &&
                     (reinterpret_cast<uintptr_t>(a.C) & 15u) == 0;
    switch (lanes_for(a.d, vec)) {
        case 1: launch_fixup_g<1>(a, vec, stream); break;
        case 2: launch_fixup_g<2>(a, vec, stream); break;
        case 4: launch_fixup_g<4>(a, vec, stream); break;
        case 8: launch_fixup_g<8>(a, vec, stream); break;
        case 16: launch_fixup_g<16>(a, vec, stream); break;
        case 32: launch_fixup_g<32>(a, vec, stream); break;
        default: launch_fixup_g<64>(a, vec, stream); break;
    }
    return hipGetLastError();
}

template <int G>
static void launch_rerank_g(const RerankArgs &a, bool vec, hipStream_t stream) {
    if (vec)
        hipLaunchKernelGGL((rerank_kernel<G, true>), dim3((unsigned)a.m), dim3(kRerankThreads), 0, stream, a);
    else
        hipLaunchKernelGGL((rerank_kernel<G, false>), dim3((unsigned)a.m), dim3(kRerankThreads), 0, stream, a);
}

hipError_t launch_rerank(const RerankArgs &a, hipStream_t stream) {
    if (a.m == 0) return hipSuccess;
    if (a.kk > kRerankMax) return hipErrorInvalidValue;
    const bool vec = a.d % 4 == 0 && (reinterpret_cast<uintptr_t>(a.Q) & 15u) == 0 &&
                     (reinterpret_cast<uintptr_t>(a.C) & 15u) == 0;
    switch (lanes_for(a.d, vec)) {
        case 1: launch_rerank_g<1>(a, vec, stream); break;
        case 2: launch_rerank_g<2>(a, vec, stream); break;
        case 4: launch_rerank_g<4>(a, vec, stream); break;
        case 8: launch_rerank_g<8>(a, vec, stream); break;
        case 16: launch_rerank_g<16>(a, vec, stream); break;
        case 32: launch_rerank_g<32>(a, vec, stream); break;
        default: launch_rerank_g<64>(a, vec, stream); break;
    }
    return hipGetLastError();
}

// ---- the same steps over many matrices in one launch ---------------------------
// A batch has hundreds of matrices, most of them a few microseconds of work: a
// launch each costs more than the work (96 jobs: 1100 launches, 0.4 to 0.5 ms of
// every 4.5 us step, and the small ones leave most CUs idle).  One launch per
// kernel instance instead: workgroup b finds its segment by a search over the
// segments' first workgroups (uniform: scalar loads).
__device__ __forceinline__ uint32_t segment_of(const uint32_t *__restrict__ first, uint32_t nseg, uint32_t b) {
    uint32_t lo = 0, hi = nseg;  // first[lo] <= b < first[hi]
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) / 2;
        if (first[mid] <= b) lo = mid;
        else hi = mid;
    }
    return lo;
}

template <int G, bool VEC>
__global__ __launch_bounds__(256) void sqnorm_group_kernel(const PrepSeg *__restrict__ segs,
                                                           const uint32_t *__restrict__ first, uint32_t nseg) {
    const uint32_t s = segment_of(first, nseg, blockIdx.x);
    const PrepSeg &a = segs[s];
    sqnorm_body<G, VEC>(a.X, a.n, a.src_n, a.d, a.norm, a.max_bits, blockIdx.x - first[s], first[s + 1] - first[s]);
}

template <int G, bool VEC>
__global__ __launch_bounds__(256) void split_group_kernel(const PrepSeg *__restrict__ segs,
                                                          const uint32_t *__restrict__ first, uint32_t nseg) {
    const uint32_t s = segment_of(first, nseg, blockIdx.x);
    const PrepSeg &a = segs[s];
    split_body<G, VEC>(a.X, a.n, a.src_n, a.d, static_cast<unsigned char *>(a.out), (int64_t)((a.d + 31) / 32) * 128,
                       a.scale, a.norm, a.max_bits, blockIdx.x - first[s], first[s + 1] - first[s]);
}

template <int G, bool VEC>
__global__ __launch_bounds__(256) void quantize_group_kernel(const PrepSeg *__restrict__ segs,
                                                             const uint32_t *__restrict__ first, uint32_t nseg) {
    const uint32_t s = segment_of(first, nseg, blockIdx.x);
    const PrepSeg &a = segs[s];
    quantize_body<G, VEC>(a.X, a.n, a.src_n, a.d, a.prec, a.out, a.scale, a.norm, a.max_bits, blockIdx.x - first[s],
                          first[s + 1] - first[s], true);
}

__global__ __launch_bounds__(256) void gather_group_kernel(const PrepSeg *__restrict__ segs,
                                                           const uint32_t *__restrict__ first, uint32_t nseg) {
    const uint32_t s = segment_of(first, nseg, blockIdx.x);
    const PrepSeg &a = segs[s];
    const int64_t i = (int64_t)(blockIdx.x - first[s]) * 4 + threadIdx.x / kWave;
    if (i >= a.n) return;
    const float *x = a.X + source_row(i, a.n, a.src_n) * a.d;
    float *o = static_cast<float *>(a.out) + i * a.d;
    for (int c = (int)lane_id(); c < a.d; c += kWave) o[c] = x[c];
}

__global__ __launch_bounds__(256) void flag_group_kernel(const FlagSeg *__restrict__ segs,
                                                         const uint32_t *__restrict__ first, uint32_t nseg) {
    const uint32_t s = segment_of(first, nseg, blockIdx.x);
    flag_body(segs[s], (int64_t)(blockIdx.x - first[s]) * 256 + threadIdx.x);
}

__global__ __launch_bounds__(256) void certify_group_kernel(const CertifyArgs *__restrict__ segs,
                                                            const uint32_t *__restrict__ first, uint32_t nseg) {
    const uint32_t s = segment_of(first, nseg, blockIdx.x);
    certify_body(segs[s], (int64_t)(blockIdx.x - first[s]) * 256 + threadIdx.x);
}

template <int G, bool VEC>
__global__ __launch_bounds__(kRerankThreads) void rerank_group_kernel(const RerankArgs *__restrict__ segs,
                                                                      const uint32_t *__restrict__ first,
                                                                      uint32_t nseg) {
    const uint32_t s = segment_of(first, nseg, blockIdx.x);
    rerank_body<G, VEC>(segs[s], blockIdx.x - first[s]);
}

namespace {

// Sorts the segments by class, and lists the classes and the segments' first
// workgroups (each class's from 0, with its end; at most 2^30 workgroups a class).
template <class Seg, class ClassOf, class BlocksOf>
std::vector<SegClass> group_segments(std::vector<Seg> &segs, std::vector<uint32_t> &first, ClassOf class_of,
                                     BlocksOf blocks_of) {
    std::stable_sort(segs.begin(), segs.end(), [&](const Seg &x, const Seg &y) { return class_of(x) < class_of(y); });
    std::vector<SegClass> out;
    first.clear();
    int64_t total = 0;
    for (size_t i = 0; i < segs.size(); ++i) {
        const int c = class_of(segs[i]);
        const int64_t nb = blocks_of(segs[i]);
        if (out.empty() || out.back().key != c || total + nb > (1 << 30)) {
            if (!out.empty()) first.push_back((uint32_t)total);
            out.push_back(SegClass{c, (uint32_t)i, 0, (uint32_t)first.size(), 0});
            total = 0;
        }
        first.push_back((uint32_t)total);
        total += nb;
        out.back().nseg += 1;
        out.back().blocks = (uint32_t)total;
    }
    if (!out.empty()) first.push_back((uint32_t)total);
    return out;
}

bool vec_rows(const float *X, int d) { return d % 4 == 0 && (reinterpret_cast<uintptr_t>(X) & 15u) == 0; }

// A class: the step, the lanes per row (or one class for all) and 16-byte loads.
int prep_class(const PrepSeg &a) {
    if (a.kind == kPrepGather) return a.kind * 256;
    const bool vec = vec_rows(a.X, a.d);
    return a.kind * 256 + lanes_for(a.d, vec) * 2 + vec;
}

}  // namespace

std::vector<SegClass> group_prep(std::vector<PrepSeg> &segs, std::vector<uint32_t> &first) {
    return group_segments(segs, first, prep_class, [](const PrepSeg &a) -> int64_t {
        const int G = prep_class(a) % 256 / 2;
        if (a.kind == kPrepNorm) return sqnorm_blocks(a.n, G);
        if (a.kind == kPrepSplit) return split_blocks(a.n, G);
        if (a.kind == kPrepQuant) return quantize_blocks(a.n, G, prep_class(a) % 2 != 0);
        return (a.n + 3) / 4;
    });
}

std::vector<SegClass> group_rerank(std::vector<RerankArgs> &segs, std::vector<uint32_t> &first) {
    return group_segments(
        segs, first,
        [](const RerankArgs &a) {
            const bool vec = vec_rows(a.Q, a.d) && vec_rows(a.C, a.d);
            return lanes_for(a.d, vec) * 2 + (int)vec;
        },
        [](const RerankArgs &a) { return a.m; });
}

std::vector<SegClass> group_flags(std::vector<FlagSeg> &segs, std::vector<uint32_t> &first) {
    return group_segments(
        segs, first, [](const FlagSeg &) { return 0; }, [](const FlagSeg &a) { return (a.m + 255) / 256; });
}

std::vector<SegClass> group_certify(std::vector<CertifyArgs> &segs, std::vector<uint32_t> &first) {
    return group_segments(
        segs, first, [](const CertifyArgs &) { return 0; }, [](const CertifyArgs &a) { return (a.m + 255) / 256; });
}

// One instance per (lanes, 16-byte loads).
#define KNN_LANES_CASE(KERNEL, G)                                                                              \
    case 2 * G: hipLaunchKernelGGL((KERNEL<G, false>), g, b, 0, stream, s, f, c.nseg); break;                   \
    case 2 * G + 1: hipLaunchKernelGGL((KERNEL<G, true>), g, b, 0, stream, s, f, c.nseg); break;

hipError_t launch_prep_group(const SegClass &c, const PrepSeg *segs, const uint32_t *first, hipStream_t stream) {
    if (c.blocks == 0) return hipSuccess;
    const dim3 g(c.blocks), b(256);
    const PrepSeg *s = segs + c.seg0;
    const uint32_t *f = first + c.first0;
    const int kind = c.key / 256, inst = c.key % 256;
    if (kind == kPrepQuant) {
        switch (inst) {
            KNN_LANES_CASE(quantize_group_kernel, 1)
            KNN_LANES_CASE(quantize_group_kernel, 2)
            KNN_LANES_CASE(quantize_group_kernel, 4)
            KNN_LANES_CASE(quantize_group_kernel, 8)
            KNN_LANES_CASE(quantize_group_kernel, 16)
            KNN_LANES_CASE(quantize_group_kernel, 32)
            KNN_LANES_CASE(quantize_group_kernel, 64)
            default: return hipErrorInvalidValue;
        }
    } else if (kind == kPrepGather) {
        hipLaunchKernelGGL(gather_group_kernel, g, b, 0, stream, s, f, c.nseg);
    } else if (kind == kPrepSplit) {
        switch (inst) {
            KNN_LANES_CASE(split_group_kernel, 16)
            KNN_LANES_CASE(split_group_kernel, 32)
            KNN_LANES_CASE(split_group_kernel, 64)
            default: return hipErrorInvalidValue;
        }
    } else {
        switch (inst) {
            KNN_LANES_CASE(sqnorm_group_kernel, 1)
            KNN_LANES_CASE(sqnorm_group_kernel, 2)
            KNN_LANES_CASE(sqnorm_group_kernel, 4)
            KNN_LANES_CASE(sqnorm_group_kernel, 8)
            KNN_LANES_CASE(sqnorm_group_kernel, 16)
            KNN_LANES_CASE(sqnorm_group_kernel, 32)
            KNN_LANES_CASE(sqnorm_group_kernel, 64)
            default: return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

hipError_t launch_rerank_group(const SegClass &c, const RerankArgs *segs, const uint32_t *first, hipStream_t stream) {
    if (c.blocks == 0) return hipSuccess;
    const dim3 g(c.blocks), b(kRerankThreads);
    const RerankArgs *s = segs + c.seg0;
    const uint32_t *f = first + c.first0;
    switch (c.key) {
        KNN_LANES_CASE(rerank_group_kernel, 1)
        KNN_LANES_CASE(rerank_group_kernel, 2)
        KNN_LANES_CASE(rerank_group_kernel, 4)
        KNN_LANES_CASE(rerank_group_kernel, 8)
        KNN_LANES_CASE(rerank_group_kernel, 16)
        KNN_LANES_CASE(rerank_group_kernel, 32)
        KNN_LANES_CASE(rerank_group_kernel, 64)
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
#undef KNN_LANES_CASE

hipError_t launch_flag_group(const SegClass &c, const FlagSeg *segs, const uint32_t *first, hipStream_t stream) {
    if (c.blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(flag_group_kernel, dim3(c.blocks), dim3(256), 0, stream, segs + c.seg0, first + c.first0, c.nseg);
    return hipGetLastError();
}

hipError_t launch_certify_group(const SegClass &c, const CertifyArgs *segs, const uint32_t *first,
                                hipStream_t stream) {
    if (c.blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(certify_group_kernel, dim3(c.blocks), dim3(256), 0, stream, segs + c.seg0, first + c.first0,
                       c.nseg);
    return hipGetLastError();
}

}  // namespace knn
