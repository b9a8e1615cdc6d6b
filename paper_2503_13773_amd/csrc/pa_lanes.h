// Exchanges between the lanes of a wavefront inside the vector ALU (gfx950).  A shuffle through the LDS pipe takes 100 cycles
// and more, and a reduction over 64 lanes is a chain of six: most of the time between the arrival of the context lengths and
// the first request for a tile, in calls that are a few microseconds long.  Decode, 32 / 8 heads of 128, us, by shuffles / so:
// one sequence of 1000 tokens 8.8 / 8.0, of 3217 11.45 / 10.67, of 20000 21.2 / 20.2, 64 lognormal 37.9 / 37.5; heads of 64, 12
// of up to 4000 10.8 / 9.9.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kvc {
namespace lanes {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <class T>
__device__ inline uint32_t bits(T x) { return __builtin_bit_cast(uint32_t, x); }

// DPP controls: permutations of a quad, mirrors of 8 and 16 lanes, rotations of a row of 16, shifts along it, its last lane to the next rows.
constexpr int kXor1 = 0xb1, kXor2 = 0x4e, kMirror8 = 0x141, kMirror16 = 0x140, kRor4 = 0x124, kRor8 = 0x128, kShr = 0x110, kBcast15 = 0x142,
              kBcast31 = 0x143;
template <int CTRL, int ROWS = 0xf, class T>
__device__ inline T permuted(T x) {  // 0 in lanes that nothing is moved to
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, ROWS, 0xf, ROWS == 0xf));
}

// What lanes l and l ^ OFF hold, OFF = 16 or 32: first[] in the lane whose bit OFF is clear, second[] in the other; the same two
// in both lanes.
template <class T>
struct Pair { T first, second; };
template <int OFF, class T>
__device__ inline Pair<T> pair_of(T x) {
    static_assert(OFF == 16 || OFF == 32, "halves, or neighbouring rows of 16 lanes");
    const u32x2 b = OFF == 32 ? __builtin_amdgcn_permlane32_swap(bits(x), bits(x), false, false)
                              : __builtin_amdgcn_permlane16_swap(bits(x), bits(x), false, false);
    const uint32_t first = b[0], second = b[1];
    return {__builtin_bit_cast(T, first), __builtin_bit_cast(T, second)};
}

// op over lanes l and l ^ 32.
__device__ inline float max_over_halves(float x) {
    const Pair<float> b = pair_of<32>(x);
    return fmaxf(b.first, b.second);
}
__device__ inline float sum_over_halves(float x) {
    const Pair<float> b = pair_of<32>(x);
    return b.first + b.second;
}

// op over lanes l, l ^ 16, l ^ 32 and l ^ 48.
template <class T, class Op>
__device__ inline T over_rows(T x, Op op) {
    const Pair<T> a = pair_of<16>(x);
    x = op(a.first, a.second);
    const Pair<T> b = pair_of<32>(x);
    return op(b.first, b.second);
}
__device__ inline float max_over_rows(float x) { return over_rows(x, [](float a, float b) { return fmaxf(a, b); }); }
__device__ inline float sum_over_rows(float x) { return over_rows(x, [](float a, float b) { return a + b; }); }

// op over all 64 lanes, in the order of a butterfly with distances 32, 16, 8, 4, 2, 1 (the rotations are such steps on
// values that already agree at twice the distance).
template <class T, class Op>
__device__ inline T over_wave(T x, Op op) {
    const Pair<T> a = pair_of<32>(x);
    x = op(a.first, a.second);
    const Pair<T> b = pair_of<16>(x);
    x = op(b.first, b.second);
    x = op(x, permuted<kRor8>(x));
    x = op(x, permuted<kRor4>(x));
    x = op(x, permuted<kXor2>(x));
    return op(x, permuted<kXor1>(x));
}
__device__ inline int wave_sum(int x) {
    return __builtin_amdgcn_readfirstlane(over_wave(x, [](int a, int b) { return a + b; }));
}
__device__ inline int wave_max(int x) {
    return __builtin_amdgcn_readfirstlane(over_wave(x, [](int a, int b) { return a > b ? a : b; }));
}
__device__ inline float wave_sum(float x) { return over_wave(x, [](float a, float b) { return a + b; }); }
__device__ inline float wave_max(float x) { return over_wave(x, [](float a, float b) { return fmaxf(a, b); }); }

// Sum over lanes 0 .. l: along the rows of 16 lanes, then from row to row.
__device__ inline int prefix_sum(int x) {
    x += permuted<kShr + 1>(x);
    x += permuted<kShr + 2>(x);
    x += permuted<kShr + 4>(x);
    x += permuted<kShr + 8>(x);
    x += permuted<kBcast15, 0xa>(x);
    return x + permuted<kBcast31, 0xc>(x);
}

}  // namespace lanes
}  // namespace kvc
