// Device helpers shared by the HIP kernels of libknn: ordered keys, wavefront
// vote helpers, in-register and LDS bitonic sorts.  gfx950, wave64.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace knn {

constexpr int kWave = 64;

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr uint64_t kKeyMax = ~0ull;       // above every real key (indices are < 2^31)
constexpr uint32_t kOrdNaN = 0xFFFFFFFFu;  // every NaN maps here
constexpr uint32_t kOrdZero = 0x80000000u; // -0 and +0 map here

// Order-preserving map of an FP32 value to uint32 under the total order used by
// selection: -0 == +0, NaN == NaN above +inf, otherwise IEEE order.
__device__ __forceinline__ uint32_t ord32(float v) {
    uint32_t u = __float_as_uint(v);
    u = (v == 0.0f) ? 0u : u;
    uint32_t o = u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
    return (v != v) ? kOrdNaN : o;
}

// ord32 of a value known not to be NaN.
__device__ __forceinline__ uint32_t ord32_not_nan(float v) {
    uint32_t u = __float_as_uint(v);
    u = (v == 0.0f) ? 0u : u;
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

// Inverse of ord32 for every class that has one representative (not for the
// zero class, which returns +0, nor the NaN class).
__device__ __forceinline__ float ord_to_float(uint32_t o) {
    uint32_t u = (o & 0x80000000u) ? (o ^ 0x80000000u) : ~o;
    return __uint_as_float(u);
}

// A selection key: value class in the high word, column index in the low word,
// so keys are distinct and ties resolve to the lower index.
__device__ __forceinline__ uint64_t make_key(float v, uint32_t idx) {
    return ((uint64_t)ord32(v) << 32) | idx;
}
// The same from an ordered value class, as a register pair (no 64-bit shift or add).
__device__ __forceinline__ uint64_t key_of(uint32_t ord, uint32_t idx) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 w = {idx, ord};
    return __builtin_bit_cast(uint64_t, w);
}
__device__ __forceinline__ uint32_t key_idx(uint64_t k) { return (uint32_t)k; }
__device__ __forceinline__ uint32_t key_ord(uint64_t k) { return (uint32_t)(k >> 32); }

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & (kWave - 1); }

// Number of set bits of `m` in lanes below this lane.
__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ uint32_t wave_bcast0(uint32_t v) {
    return __builtin_amdgcn_readfirstlane(v);
}

// A pivot key prepared for fast comparison against (value, index) pairs.
struct Pivot {
    float pv;       // representative value of the pivot's class (+0 for zeros)
    uint32_t pidx;  // pivot index
    uint32_t nan;   // pivot is in the NaN class
    uint32_t inf;   // pivot is the +infinity sentinel (every key is below)
};

__device__ __forceinline__ Pivot make_pivot(uint64_t key) {
    Pivot p;
    uint32_t o = key_ord(key);
    p.inf = (key == kKeyMax) ? 1u : 0u;
    p.nan = (o == kOrdNaN) ? 1u : 0u;
    p.pv = (o == kOrdZero) ? 0.0f : ord_to_float(o);
    p.pidx = key_idx(key);
    return p;
}

// (v, j) < pivot in the key order.
__device__ __forceinline__ bool key_below(float v, uint32_t j, const Pivot &p) {
    if (p.inf) return true;
    bool lt = p.nan ? (v == v) : (v < p.pv);
    bool eq = p.nan ? (v != v) : (v == p.pv);
    return lt || (eq && j < p.pidx);
}

// Lanes whose bit b (1, 2, .. 32) is clear.
constexpr uint64_t lanes_clear(uint32_t b) {
    return b == 1 ? 0x5555555555555555ull : b == 2 ? 0x3333333333333333ull : b == 4 ? 0x0F0F0F0F0F0F0F0Full
         : b == 8 ? 0x00FF00FF00FF00FFull : b == 16 ? 0x0000FFFF0000FFFFull : 0x00000000FFFFFFFFull;
}
// This lane's bit of a mask that is the same in every lane.
__device__ __forceinline__ bool mine(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

// The value of lane (lane ^ mask), every lane of the wave active.  Masks 1, 2
// and 8 are single DPP moves (quad permutations, a rotation by 8 within rows
// of 16), mask 4 two DPP moves (half-row mirror, quad reversal), masks 16 and 32
// a swap of odd with even rows of 16 or of halves of 32 between two copies (each
// lane's partner is then in one copy or the other); others go through the LDS
// crossbar.
__device__ __forceinline__ uint32_t xor_lanes32(uint32_t v, int mask) {
    const int x = (int)v;
    switch (mask) {
        case 1: return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, false);  // quad_perm 1,0,3,2
        case 2: return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, false);  // quad_perm 2,3,0,1
        case 4: {
            // lane ^ 7 within groups of 8 (row_half_mirror), then lane ^ 3
            // within quads: (i ^ 7) ^ 3 = i ^ 4
            const int m = __builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, false);  // row_half_mirror
            return (uint32_t)__builtin_amdgcn_mov_dpp(m, 0x1B, 0xF, 0xF, false);  // quad_perm 3,2,1,0
        }
        case 8: return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x128, 0xF, 0xF, false);  // row_ror:8
        case 16: {
            const auto w = __builtin_amdgcn_permlane16_swap(v, v, false, false);
            return mine(lanes_clear(16)) ? w[1] : w[0];
        }
        case 32: {
            const auto w = __builtin_amdgcn_permlane32_swap(v, v, false, false);
            return mine(lanes_clear(32)) ? w[1] : w[0];
        }
        default: return (uint32_t)__shfl_xor(x, mask);
    }
}

// For masks known at compile time (unrolled loops): the DPP forms above.
__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int mask) {
    const uint32_t lo = xor_lanes32((uint32_t)v, mask);
    const uint32_t hi = xor_lanes32((uint32_t)(v >> 32), mask);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t shfl_xor_any(uint64_t v, int mask) { return shfl_xor_u64(v, mask); }
__device__ __forceinline__ uint32_t shfl_xor_any(uint32_t v, int mask) { return xor_lanes32(v, mask); }
__device__ __forceinline__ float shfl_xor_any(float v, int mask) {
    return __uint_as_float(xor_lanes32(__float_as_uint(v), mask));
}

// A structure at an address that is the same in every lane, held in scalar
// registers (vector loads of the same words, then the first lane's copy).
template <class T>
__device__ __forceinline__ T uniform_load(const T *p) {
    static_assert(sizeof(T) % 4 == 0, "whole dwords");
    T v;
    const uint32_t *src = reinterpret_cast<const uint32_t *>(p);
    uint32_t *dst = reinterpret_cast<uint32_t *>(&v);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) dst[i] = __builtin_amdgcn_readfirstlane(src[i]);
    return v;
}

// A lane mask (the same in every lane) with the constant C's bits flipped, by
// literal operands of scalar instructions: the constants of a network's steps
// are then part of its code, where the compiler would keep them in scalar
// registers across a loop over rows (some two hundred, spilled).
template <uint64_t C>
__device__ __forceinline__ uint64_t flip(uint64_t m) {
    uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
    if constexpr ((uint32_t)C != 0) asm("s_xor_b32 %0, %1, %2" : "=s"(lo) : "s"(lo), "i"((uint32_t)C) : "scc");
    if constexpr ((uint32_t)(C >> 32) != 0)
        asm("s_xor_b32 %0, %1, %2" : "=s"(hi) : "s"(hi), "i"((uint32_t)(C >> 32)) : "scc");
    return ((uint64_t)hi << 32) | lo;
}

// f(integral_constant 0), f(integral_constant 1), ..
template <class F, int... I>
__device__ __forceinline__ void static_for(std::integer_sequence<int, I...>, F f) {
    (f(std::integral_constant<int, I>{}), ...);
}
// Steps of a bitonic sort of n keys, and the (size, stride) of step i.
constexpr int bitonic_steps(uint32_t n) {
    int c = 0;
    for (uint32_t size = 2; size <= n; size <<= 1)
        for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) ++c;
    return c;
}
constexpr uint32_t bitonic_at(int i, bool want_size) {
    for (uint32_t size = 2;; size <<= 1)
        for (uint32_t stride = size >> 1; stride > 0; stride >>= 1)
            if (i-- == 0) return want_size ? size : stride;
}

// One step of a bitonic network between lanes: every lane keeps its key or takes
// its partner's, the smaller where A ^ B ^ dyn has a clear bit.  The
// comparison's mask is combined with the direction in scalar registers.
template <uint64_t C, class K>
__device__ __forceinline__ K lane_step(K key, K other, uint64_t dyn = 0) {
    return mine(flip<C>(__ballot(key < other)) ^ dyn) ? key : other;
}

// Ascending bitonic sort of 64 J keys across a wave (key l J + j in lane l).
template <int J, class K>
__device__ __forceinline__ void wave_sort_regs(K (&k)[J]) {
    constexpr uint32_t N = (uint32_t)kWave * J, UJ = J;
    static_for(std::make_integer_sequence<int, bitonic_steps(N)>{}, [&](auto i) {
        constexpr uint32_t size = bitonic_at(decltype(i)::value, true), stride = bitonic_at(decltype(i)::value, false);
        // kept where (key < other) == take_min, take_min = (bit stride clear) == (bit size clear)
        constexpr uint64_t D = size == N ? ~0ull : (size >= UJ ? lanes_clear(size / UJ > 0 ? size / UJ : 1) : 0ull);
        if constexpr (stride < UJ) {
#pragma unroll
            for (int j = 0; j < J; ++j)
                if ((j & stride) == 0) {
                    const K a = k[j], b = k[j + stride];
                    bool swap;
                    if constexpr (size < UJ) swap = (a > b) == ((j & size) == 0);
                    else swap = mine(flip<~D>(__ballot(a > b)));
                    k[j] = swap ? b : a;
                    k[j + stride] = swap ? a : b;
                }
        } else {
#pragma unroll
            for (int j = 0; j < J; ++j)
                k[j] = lane_step<lanes_clear(stride / UJ) ^ D>(k[j], shfl_xor_any(k[j], (int)(stride / UJ)));
        }
    });
}
__device__ __forceinline__ uint64_t wave_sort64(uint64_t key) {
    uint64_t k[1] = {key};
    wave_sort_regs<1>(k);
    return k[0];
}

__device__ __forceinline__ uint64_t wave_readlane_u64(uint64_t v, int lane) {
    uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, lane);
    uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint32_t wave_readlane_any(uint32_t v, int lane) {
    return __builtin_amdgcn_readlane(v, lane);
}
__device__ __forceinline__ uint64_t wave_readlane_any(uint64_t v, int lane) { return wave_readlane_u64(v, lane); }
// Key p (the same in every lane) of a sorted run of 64 J keys across a wave.
template <int J, class K>
__device__ __forceinline__ K wave_key(const K (&k)[J], uint32_t p) {
    K v = wave_readlane_any(k[0], (int)(p / J));
#pragma unroll
    for (int j = 1; j < J; ++j) {
        const K o = wave_readlane_any(k[j], (int)(p / J));
        v = p % J == (uint32_t)j ? o : v;
    }
    return v;
}

// Ascending bitonic sort of NT * J keys of buf (J = 1, 2, 4 or 8), with the keys
// in registers: thread t holds keys t*J .. t*J + J - 1, so compare-exchange
// partners less than J apart are in the same thread, partners less than 64*J
// apart are in the same wave (one shuffle), and only the strides of J*64 and
// above go through LDS, with a barrier each.
//
// The keys come from load(i) for i in [0, NT * J); buf is the exchange area and
// receives the sorted keys.  With SYNC the threads wait for each other after
// loading (needed when load reads LDS that other threads overwrite).
//
// The direction of a step depends on bits of t: below 64 lanes it is a constant
// lane mask, above it is the same for a whole wave.
template <int NT, int J, bool SYNC, class Load>
__device__ __forceinline__ void block_sort_regs_from(uint64_t *buf, Load load) {
    constexpr uint32_t N = (uint32_t)NT * J, UJ = J, W = kWave;
    uint32_t t = threadIdx.x;
    asm volatile("" : "+v"(t));  // (opaque: nothing below is formed ahead of a caller's loop and kept)
    const uint32_t wave = __builtin_amdgcn_readfirstlane(t / kWave);
    uint64_t k[J];
#pragma unroll
    for (int j = 0; j < J; ++j) k[j] = load(t * J + j);
    if (SYNC) __syncthreads();
    static_for(std::make_integer_sequence<int, bitonic_steps(N)>{}, [&](auto i) {
        constexpr uint32_t size = bitonic_at(decltype(i)::value, true), stride = bitonic_at(decltype(i)::value, false);
        // ascending lanes of this size: all (the last), by a lane's bit (D), or
        // by the wave's (dyn)
        constexpr uint32_t sb = size / UJ;
        constexpr uint64_t D = size == N ? ~0ull : (size >= UJ && sb < W ? lanes_clear(sb > 0 ? sb : 1) : 0ull);
        uint64_t dyn = 0;
        if constexpr (size < N && sb >= W) dyn = (wave & (sb / W)) ? 0ull : ~0ull;
        if constexpr (stride < UJ) {
#pragma unroll
            for (int j = 0; j < J; ++j)
                if ((j & stride) == 0) {
                    const uint64_t a = k[j], b = k[j + stride];
                    bool swap;
                    if constexpr (size < UJ) swap = (a > b) == ((j & size) == 0);
                    else swap = mine(flip<~D>(__ballot(a > b)) ^ dyn);
                    k[j] = swap ? b : a;
                    k[j + stride] = swap ? a : b;
                }
        } else {
            // partners in other threads: the direction is the same for all J keys
            // of a thread (stride and size are multiples of J)
            constexpr uint32_t ls = stride / UJ;
            uint64_t o[J];
            if constexpr (ls < W) {
#pragma unroll
                for (int j = 0; j < J; ++j) o[j] = shfl_xor_any(k[j], (int)ls);
#pragma unroll
                for (int j = 0; j < J; ++j) k[j] = lane_step<lanes_clear(ls) ^ D>(k[j], o[j], dyn);
            } else {
                const uint32_t i0 = t * J;
#pragma unroll
                for (int j = 0; j < J; ++j) buf[i0 + j] = k[j];
                __syncthreads();
#pragma unroll
                for (int j = 0; j < J; ++j) o[j] = buf[(i0 + j) ^ stride];
                __syncthreads();
                dyn ^= (wave & (ls / W)) ? 0ull : ~0ull;
#pragma unroll
                for (int j = 0; j < J; ++j) k[j] = lane_step<D>(k[j], o[j], dyn);
            }
        }
    });
#pragma unroll
    for (int j = 0; j < J; ++j) buf[t * J + j] = k[j];
    __syncthreads();
}

// In place: every thread loads exactly the positions it later writes.
template <int NT, int J>
__device__ __forceinline__ void block_sort_regs(uint64_t *buf) {
    block_sort_regs_from<NT, J, false>(buf, [buf](uint32_t i) { return buf[i]; });
}

// Ascending sort of the first n keys of buf (n <= MAXJ * NT, MAXJ = 4 or 8):
// pads to the next of NT, 2 NT, 4 NT (, 8 NT) keys with the largest key, then
// sorts in registers (the buffer must hold the padded length).  Callers have
// made the n keys visible (barrier).
template <int NT, int MAXJ = 4>
__device__ __forceinline__ void block_sort(uint64_t *buf, uint32_t n) {
    static_assert(MAXJ == 4 || MAXJ == 8, "4 or 8 keys per thread at most");
    const uint32_t m = n <= (uint32_t)NT ? NT : (n <= 2u * NT ? 2 * NT : (n <= 4u * NT ? 4 * NT : 8 * NT));
    for (uint32_t t = n + threadIdx.x; t < m; t += NT) buf[t] = kKeyMax;
    __syncthreads();
    if (m == (uint32_t)NT)
        block_sort_regs<NT, 1>(buf);
    else if (m == 2u * NT)
        block_sort_regs<NT, 2>(buf);
    else if (MAXJ == 4 || m == 4u * NT)
        block_sort_regs<NT, 4>(buf);
    else
        block_sort_regs<NT, MAXJ>(buf);
}

}  // namespace knn
