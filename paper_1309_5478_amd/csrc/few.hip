// Distance rows of a few queries: d'(i, j) = ||c_j||^2 - 2 q_i.c_j for up to 127
// FP32 query rows against the whole corpus, stored densely, with the corpus norms
// (their largest for the certificate), in one pass over the corpus.
//
// With so few queries a search is one read of the corpus: 2 m flops per 4 bytes
// are below the balance of the FP32 matrix instruction (about 25 flops per byte)
// up to m = 50, and what the fused path does around its product (norms in a pass
// of their own, gathered sample, thresholds, a 128-row tile that is mostly
// padding) costs several reads more.  Storing the m x n keys costs 4 m bytes per
// corpus row of 4 d, and the selection one more read of them.
//
// A wave takes 16 corpus rows at a time: lane l holds, of row l % 16, elements
// 16 t + 4 (l / 16) + 0..3 for t = 0..7, straight from memory in 16-byte loads, two
// chunks of 128 elements in flight; the sum runs over them in that order, and
// queries lie in LDS in the same order (row stride 4 mod 16 words: the 16 rows
// of a read fall on different banks).  16 x 16 x 4 products: corpus fragments
// are used for all query tiles, and the results come with one corpus row per
// lane, as its norm does.
//
// Measured, whole searches with k = 10, fused path / this one: 16 x 10^6 x 128
// 542 / 197 us (product alone 328 + 57 for the norms), 64 x 10^6 x 128 560 / 307,
// 1 x 10^6 x 300 1046 / 295 (4.1 TB/s), 16 x 200000 x 768 641 / 211, 16 x 5000 x 128
// 132 / 66.
#include "dist.hpp"
#include "keys.hpp"

namespace knn {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // (rows of any length)

constexpr int kFewChunk = 128;                // elements of a row per step
constexpr int kFewLoads = kFewChunk / 16;     // loads per lane and step
constexpr int kFewMaxWaves = 16;
constexpr int few_waves(int mt) { return mt <= 2 ? 16 : 8; }  // per CU: what the registers leave

}  // namespace

// MT: 16-query tiles.
template <int MT>
__global__ __launch_bounds__(few_waves(MT) * kWave) void dist_few_kernel(const float *__restrict__ Q, int m,
                                                                       const float *__restrict__ C, int64_t n, int d,
                                                                       float *__restrict__ out,
                                                                       float *__restrict__ qnorm2,
                                                                       unsigned int *__restrict__ max_bits) {
    extern __shared__ __align__(16) float sq[];  // MT * 16 rows of the padded length
    __shared__ float wmax[kFewMaxWaves];
    const int ld = (d + 15) / 16 * 16 + 4;
    const uint32_t lane = lane_id(), wave = threadIdx.x / kWave, waves = blockDim.x / kWave;
    const uint32_t l16 = lane % 16, g = lane / 16;
    for (int r = (int)wave; r < MT * 16; r += (int)waves)
        for (int c = (int)lane; c < ld; c += kWave) sq[r * ld + c] = r < m && c < d ? Q[(int64_t)r * d + c] : 0.f;
    __syncthreads();
    if (blockIdx.x == 0)  // squared query norms, for the certificate
        for (int r = (int)wave; r < m; r += (int)waves) {
            float s = 0.f;
            for (int c = (int)lane; c < d; c += kWave) s = fmaf(sq[r * ld + c], sq[r * ld + c], s);
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) s += shfl_xor_any(s, off);
            if (lane == 0) qnorm2[r] = s;
        }

    const int64_t tiles = (n + 15) / 16, step = (int64_t)gridDim.x * waves;
    const int nk = (d + kFewChunk - 1) / kFewChunk;
    const float *const qa = sq + l16 * ld + 4 * g;
    // this lane's part of chunk kc of its row (zeros beyond the row's end)
    auto load = [&](f32x4 (&v)[kFewLoads], const float *row, int kc) {
        const int k0 = kc * kFewChunk + 4 * (int)g;
        if ((kc + 1) * kFewChunk <= d) {
#pragma unroll
            for (int t = 0; t < kFewLoads; ++t) v[t] = *reinterpret_cast<const f32x4u *>(row + k0 + 16 * t);
        } else {
#pragma unroll
            for (int t = 0; t < kFewLoads; ++t) {
                const int k = k0 + 16 * t;
                if (k + 4 <= d) {
                    v[t] = *reinterpret_cast<const f32x4u *>(row + k);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[t][e] = k + e < d ? row[k + e] : 0.f;
                }
            }
        }
    };
    auto row_of = [&](int64_t tile) -> const float * {
        const int64_t j = tile * 16 + l16;
        return C + (j < n ? j : n - 1) * d;
    };
    f32x4 acc[MT];
    float nrm = 0.f, mx = 0.f;
    auto use = [&](const f32x4 (&v)[kFewLoads], int kc) {
#pragma unroll
        for (int t = 0; t < kFewLoads; ++t) {
            if (kc * kFewChunk + 16 * t >= d) break;  // (the same for all lanes)
            f32x4 a[MT];
#pragma unroll
            for (int i = 0; i < MT; ++i)
                a[i] = *reinterpret_cast<const f32x4 *>(qa + i * 16 * ld + kc * kFewChunk + 16 * t);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                nrm = fmaf(v[t][e], v[t][e], nrm);
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], v[t][e], acc[i], 0, 0, 0);
            }
        }
    };

    int64_t tile = (int64_t)blockIdx.x * waves + wave;
    const float *row = row_of(tile < tiles ? tile : tiles - 1);
    f32x4 cur[kFewLoads], nxt[kFewLoads];
    load(cur, row, 0);
    for (; tile < tiles; tile += step) {
        const float *const next = row_of(tile + step < tiles ? tile + step : tile);
#pragma unroll
        for (int i = 0; i < MT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        nrm = 0.f;
        for (int kc = 0; kc < nk; ++kc) {
            if (kc + 1 < nk) load(nxt, row, kc + 1);
            else load(nxt, next, 0);
            use(cur, kc);
#pragma unroll
            for (int t = 0; t < kFewLoads; ++t) cur[t] = nxt[t];
        }
        row = next;
        nrm += shfl_xor_any(nrm, 16);
        nrm += shfl_xor_any(nrm, 32);
        mx = fmaxf(mx, nrm);
        const int64_t j = tile * 16 + l16;
        if (j < n) {
            float *o = out + j;
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int q = i * 16 + 4 * (int)g + r;
                    if (q < m) o[(int64_t)q * n] = fmaf(-2.0f, acc[i][r], nrm);
                }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, shfl_xor_any(mx, off));
    if (lane == 0) wmax[wave] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (uint32_t w = 1; w < waves; ++w) mx = fmaxf(mx, wmax[w]);
        atomicMax(max_bits, __float_as_uint(mx));
    }
}

// ---- host side --------------------------------------------------------------
template <int MT>
static hipError_t launch_few_t(const float *Q, int64_t m, const float *C, int64_t n, int d, float *out, float *qnorm2,
                               unsigned int *max_bits, int num_cu, hipStream_t stream) {
    const size_t lds = few_lds_bytes(MT, d);
    const int64_t tiles = (n + 15) / 16;
    // all waves per CU where the corpus gives every CU that many; fewer, so that
    // more CUs work, where it does not
    int waves = few_waves(MT);
    while (waves > 4 && tiles < (int64_t)waves * num_cu) waves /= 2;
    int64_t grid = (tiles + waves - 1) / waves;
    if (grid > num_cu) grid = num_cu;
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(dist_few_kernel<MT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((dist_few_kernel<MT>), dim3((unsigned)grid), dim3((unsigned)(waves * kWave)), lds, stream, Q,
                       (int)m, C, n, d, out, qnorm2, max_bits);
    return hipGetLastError();
}

hipError_t launch_dist_few(const float *Q, int64_t m, const float *C, int64_t n, int d, float *out, float *qnorm2,
                           unsigned int *max_bits, int num_cu, hipStream_t stream) {
    if (m == 0 || n == 0) return hipSuccess;
    if (few_passes(m, d) == 0) return hipErrorInvalidValue;
    const int tiles = few_tiles(m, d);
    hipError_t e = hipSuccess;
    for (int64_t i0 = 0; i0 < m && e == hipSuccess; i0 += 16 * tiles) {
        const int64_t mb = m - i0 < 16 * tiles ? m - i0 : 16 * tiles;
        const float *q = Q + i0 * d;
        float *o = out + i0 * n, *qn = qnorm2 + i0;
        if (tiles == 1) e = launch_few_t<1>(q, mb, C, n, d, o, qn, max_bits, num_cu, stream);
        else if (tiles == 2) e = launch_few_t<2>(q, mb, C, n, d, o, qn, max_bits, num_cu, stream);
        else if (tiles == 4) e = launch_few_t<4>(q, mb, C, n, d, o, qn, max_bits, num_cu, stream);
        else e = launch_few_t<8>(q, mb, C, n, d, o, qn, max_bits, num_cu, stream);
    }
    return e;
}

}  // namespace knn
