// What the two causal kernels on 32x32x16 matrix-core tiles share (gfx950, bf16, head_dim 128): the LDS image of a step of
// 32 tokens, its operands, and the loads and waits that fill it.  Which rows a wavefront loads stands in each kernel: as one
// struct for both it changed the registers of the 64-column kernel, 4096 tokens on blocks of 4, 32 / 8 heads, 127.8 -> 131.2 us.
#pragma once

#include <type_traits>

#include "kvc_internal.h"
#include "pa_mfma_tile.h"

namespace kvc {
namespace prefill32 {

using namespace mfma;

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int kStepTokens = 32;
constexpr int kStageBytes = kStepTokens * D * 2;  // K (or V) rows of a step: 32 rows x 256 bytes
constexpr int kRing = 4;       // stages of K and of V
constexpr float kBias = 7.0f;  // powers of two that the reference point is set above the largest score

template <int I, int N, class F>
__device__ inline void static_for(const F &f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// The value lane l ^ 32 holds, next to this lane's: one swap of the two 32-lane halves.
using lanes::max_over_halves;
using lanes::sum_over_halves;

// A operands of O^T += V^T . P^T straight from LDS.  The transposing read hands lane i of a
// 16-lane block the i-th 16-bit element of each of the four 16-element groups that lanes
// 4k .. 4k+3 of the block point at (8 bytes each).  Block (half, w) of this wavefront covers
// dims 32b + 16w .. +15; its lanes 4k .. 4k+3 point at dims +0, 4, 8, 12 of token
// 16n + 8g + 4*half + k, so the lane of dim 32b + c receives that dim of the four tokens
// 16n + 8g + 4*half .. +3: depth slots 8*half + 4g .. +3 of slice n, the order the score layout
// fixed.  Row R of a V stage keeps its 64-byte granule b at granule position (b + R) % 4, and
// R % 4 = k for the row a lane points at, so the byte offset of the lane inside a stage for
// dim block b is v_lane_offset(b) + (16n + 8g) rows.
__device__ inline int v_lane_offset(int b, int half, int c) {
    const int i16 = c & 15, k = i16 >> 2;
    return (4 * half + k) * 256 + ((b + k) & 3) * 64 + 32 * (c >> 4) + 8 * (i16 & 3);
}
// Half H of the operand of slice N.
template <int N, int H>
__device__ inline uint2 read_v_half(const unsigned char *vlane) {
    typedef short v4i16 __attribute__((ext_vector_type(4)));
    typedef v4i16 __attribute__((address_space(3))) * lds_v4i16_ptr;
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_ptr)(vlane + (16 * N + 8 * H) * 256)));
}

// V rows at or past `vlim` (tokens of the step visible to any column of this wavefront) are
// zeroed in the operand of slice N: their weights are zero for every column and the rows may
// hold NaN.
template <int N>
__device__ inline void mask_v_operand(uint2 (&va)[2], int vlim, int half) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const int tok = 16 * N + 8 * g + 4 * half;
        va[g].x &= (tok < vlim ? 0xffffu : 0u) | (tok + 1 < vlim ? 0xffff0000u : 0u);
        va[g].y &= (tok + 2 < vlim ? 0xffffu : 0u) | (tok + 3 < vlim ? 0xffff0000u : 0u);
    }
}

__device__ inline bf16x8 v_operand(const uint2 (&va)[2]) {
    const uint4 aw = {va[0].x, va[0].y, va[1].x, va[1].y};
    return __builtin_bit_cast(bf16x8, aw);
}

__device__ inline bf16x8 four_words(const uint32_t (&w)[8], int n) {
    const uint4 v = {w[4 * n], w[4 * n + 1], w[4 * n + 2], w[4 * n + 3]};
    return __builtin_bit_cast(bf16x8, v);
}

// K operand j of a step from LDS (a stage is 32 rows of 256 bytes, 16-byte chunks XOR-permuted
// by row % 16); lane (half, c) reads row c, dims 16j + 8*half .. +7.
template <int J>
__device__ inline bf16x8 read_k_operand(const unsigned char *krow, int half, int c) {
    return *reinterpret_cast<const bf16x8 *>(krow + (((2 * J + half) ^ (c & 15)) << 4));
}

// 16 bytes per lane from global memory straight into LDS, to lds_addr + 16 * lane (lds_addr uniform), and a second 1 KiB
// from and to 1 KiB further on.  The compiler does not see these accesses: barriers order them against LDS reads,
// wait_for() counts them.
__device__ inline void load_rows(const void *base, uint32_t off0, uint32_t off1_minus_1k, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %3\n\tglobal_load_lds_dwordx4 %2, %3 offset:1024"
                 :: "s"(lds_addr), "v"(off0), "v"(off1_minus_1k), "s"(base) : "memory");
}
__device__ inline void load_lane_to_lds(const void *addr, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds_addr), "v"(addr) : "memory");
}
// Waits until at most LOADS of the wavefront's loads (and stores) and LDS of its LDS reads are under way.
template <int LOADS, int LDS>
__device__ inline void wait_for() {
    static_assert(LOADS < 64 && LDS < 16, "fields of the wait instruction");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((LOADS & 15) | (LOADS >> 4) << 14 | 7 << 4 | LDS << 8);
    asm volatile("" ::: "memory");
}
__device__ inline void barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Nothing moves across this point when the compiler orders the instructions of a turn.
#define KVC_PIN() __builtin_amdgcn_sched_barrier(0)

}  // namespace prefill32
}  // namespace kvc
