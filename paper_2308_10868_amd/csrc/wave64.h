// Reductions over a 64-lane wavefront by cross-lane register moves (DPP and
// lane swaps), a few cycles a step where a shuffle goes through LDS and waits
// ~100, and small helpers of the search kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>
#include <utility>

namespace nrr {

// f(0) .. f(N - 1) with the index as a compile-time constant.
template <typename F, int... I>
__device__ __attribute__((always_inline)) inline void static_for_seq(
    F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>()), ...);
}
template <int N, typename F>
__device__ __attribute__((always_inline)) inline void static_for(F &&f) {
    static_for_seq(f, std::make_integer_sequence<int, N>());
}

// a / b for 0 <= a < 2^20, 0 < b: (a + 1/2) / b is at least 1 / (2 b) away from
// the next integer, beyond the rounding of the reciprocal and the product.
__device__ inline int quotient(int a, int b) {
    return (int)(((float)a + 0.5f) * __builtin_amdgcn_rcpf((float)b));
}

// A value that every lane of the wavefront holds, in scalar registers.
__device__ inline float uniform(float v) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(v)));
}
__device__ inline double uniform(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u),
                   hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return __builtin_bit_cast(double, hi << 32 | lo);
}

// A struct in memory that the wavefront shares, in scalar registers.
template <typename T>
__device__ inline T uniform_copy(const T &v) {
    static_assert(sizeof(T) % 4 == 0, "whole words");
    struct Words {
        uint32_t w[sizeof(T) / 4];
    } s = __builtin_bit_cast(Words, v);
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 4; ++i)
        s.w[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)s.w[i]);
    return __builtin_bit_cast(T, s);
}

template <int CTRL>
__device__ inline uint32_t dpp_move(uint32_t old, uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, 0xf, 0xf, false);
}

// Word of lane i ^ OFF.  OFF 8 and below by moves within the 16-lane row; for
// OFF 4 a rotation by 4, which equals the exchange where the values are already
// the same 8 lanes apart (after the step of OFF 8).
template <int OFF>
__device__ inline uint32_t xor_word(uint32_t v) {
    if constexpr (OFF == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return (threadIdx.x & 32) ? r[0] : r[1];
    } else if constexpr (OFF == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (threadIdx.x & 16) ? r[0] : r[1];
    } else {
        constexpr int CTRL = OFF == 8 ? 0x128 : OFF == 4 ? 0x124 : OFF == 2 ? 0x4e : 0xb1;
        return dpp_move<CTRL>(v, v);
    }
}

template <int OFF, typename T>
__device__ inline T xor_lane(T v) {
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "one or two words");
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, xor_word<OFF>(__builtin_bit_cast(uint32_t, v)));
    } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const uint64_t lo = xor_word<OFF>((uint32_t)u), hi = xor_word<OFF>((uint32_t)(u >> 32));
        return __builtin_bit_cast(T, hi << 32 | lo);
    }
}

// Sum over the wavefront in the order of the xor butterfly 32, 16, 8, 4, 2, 1
// (every lane gets the same bits as from shuffles in that order).
template <typename T>
__device__ inline T wave_xor_sum(T v) {
    v += xor_lane<32>(v);
    v += xor_lane<16>(v);
    v += xor_lane<8>(v);
    v += xor_lane<4>(v);
    v += xor_lane<2>(v);
    v += xor_lane<1>(v);
    return v;
}

// Applies f(move) for the six row shifts and broadcasts after which lane 63
// has met every lane; move(old, v) gives the lane's partner's word, or old.
template <typename F>
__device__ inline void dpp_steps(F &&f) {
    f([](uint32_t o, uint32_t v) { return dpp_move<0x111>(o, v); });  // row_shr 1, 2, 4, 8
    f([](uint32_t o, uint32_t v) { return dpp_move<0x112>(o, v); });
    f([](uint32_t o, uint32_t v) { return dpp_move<0x114>(o, v); });
    f([](uint32_t o, uint32_t v) { return dpp_move<0x118>(o, v); });
    f([](uint32_t o, uint32_t v) { return dpp_move<0x142>(o, v); });  // row_bcast 15, 31
    f([](uint32_t o, uint32_t v) { return dpp_move<0x143>(o, v); });
}

// Largest word of the wavefront (valid in lane 63).
__device__ inline uint32_t wave_max(uint32_t v) {
    dpp_steps([&](auto move) {
        const uint32_t o = move(0u, v);
        v = v > o ? v : o;
    });
    return v;
}

// Largest key, smallest index among equal ones (valid in lane 63).
template <typename Key>
__device__ inline void wave_best(Key &bk, int &bi) {
    dpp_steps([&](auto move) {
        Key ok;
        if constexpr (sizeof(Key) == 4) {
            const uint32_t u = __builtin_bit_cast(uint32_t, bk);
            ok = __builtin_bit_cast(Key, move(u, u));
        } else {
            const uint64_t u = __builtin_bit_cast(uint64_t, bk);
            const uint32_t l = (uint32_t)u, h = (uint32_t)(u >> 32);
            ok = __builtin_bit_cast(Key, (uint64_t)move(h, h) << 32 | move(l, l));
        }
        const int oi = (int)move((uint32_t)bi, (uint32_t)bi);
        const bool take = (ok > bk) | ((ok == bk) & (oi < bi));
        bk = take ? ok : bk;
        bi = take ? oi : bi;
    });
}

}  // namespace nrr
