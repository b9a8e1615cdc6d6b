// What the one-launch decode kernels share: the shape of a tile for a head dimension, how partials of a
// context that several wavefronts or workgroups hold travel between them, and the launch modes.
#pragma once

#include "pa_mfma_tile.h"

namespace kvc {
namespace mfma {

__device__ inline int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Partials cross from one wavefront to another inside a launch, between XCDs whose L2 caches
// are not coherent with each other.  They are therefore written and read with device-scope
// accesses (the sc1 cache policy: each access goes to the point of coherence of the whole
// device by itself), 16 bytes per lane, through raw buffer instructions, instead of ordinary
// stores followed by a write-back of the whole L2: that write-back, issued by 1024 wavefronts,
// doubled the kernel time when it was measured.
constexpr int kDeviceScope = 16;  // cache-policy operand of the buffer builtins: sc1
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ inline __amdgpu_buffer_rsrc_t raw_buffer(const void *base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00020000);
}
__device__ inline void store4_device_scope(__amdgpu_buffer_rsrc_t b, uint32_t byte_off, float x, float y, float z, float w) {
    const u32x4 v = {__float_as_uint(x), __float_as_uint(y), __float_as_uint(z), __float_as_uint(w)};
    __builtin_amdgcn_raw_buffer_store_b128(v, b, byte_off, 0, kDeviceScope);
}
__device__ inline float4 load4_device_scope(__amdgpu_buffer_rsrc_t b, uint32_t byte_off) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(b, byte_off, 0, kDeviceScope);
    return float4{__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w)};
}
__device__ inline void store2_device_scope(__amdgpu_buffer_rsrc_t b, uint32_t byte_off, float x, float y) {
    const u32x2 v = {__float_as_uint(x), __float_as_uint(y)};
    __builtin_amdgcn_raw_buffer_store_b64(v, b, byte_off, 0, kDeviceScope);
}
__device__ inline float2 load2_device_scope(__amdgpu_buffer_rsrc_t b, uint32_t byte_off) {
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(b, byte_off, 0, kDeviceScope);
    return float2{__uint_as_float(v.x), __uint_as_float(v.y)};
}

// What depends on the head dimension: tokens of a tile (8 KiB of K and V either way), the registers a
// tile is loaded into, Q operands, softmax state, dims a lane holds of its head.
template <int HD>
struct Shape;
template <>
struct Shape<128> {
    static constexpr int kTokens = kTileTokens, kTokensLog2 = 4, kQ = 4, kVecs = 8;
    using State = HeadStateN<8>;
    struct Tile { uint4 k[4], v[4]; };
};
template <>
struct Shape<64> {
    static constexpr int kTokens = kTileTokens64, kTokensLog2 = 5, kQ = 2, kVecs = 4;
    using State = HeadStateN<4>;
    struct Tile { uint4 k[4]; uint2 v[8]; };
};

// Partial slot layout (fp32): [HD / 16 vectors][quad][head][4]; vector v of (quad, head) = dims
// HD/4 * quad + 4v .. +3 of the head's accumulator; (max, sum) per head in a second array.  One
// store or load instruction of a wavefront then covers whole 128-byte lines.  Offsets in bytes.
template <int HD>
__device__ inline uint32_t slot_vec(int slot, int G, int v, int quad, int head) {
    return (uint32_t(slot) * uint32_t(G * HD) + uint32_t(((v * 4 + quad) * G + head) * 4)) * 4u;
}
__device__ inline uint32_t slot_ml(int slot, int G, int head) { return uint32_t(slot * G + head) * 8u; }
// vector v of a lane's accumulator registers: dims 4v .. 4v+3 of its slice of HD / 4 dims
__device__ inline float4 acc_vec(const HeadStateN<8> &x, int v) {
    const int e = 4 * (v & 1), i = v >> 1;
    return float4{x.acc[e][i], x.acc[e + 1][i], x.acc[e + 2][i], x.acc[e + 3][i]};
}
__device__ inline float4 acc_vec(const HeadStateN<4> &x, int v) {
    return float4{x.acc[0][v], x.acc[1][v], x.acc[2][v], x.acc[3][v]};
}

// What a launch does with the placement of the workers (the start-up work that depends only on
// block_tables and context_lens, which all layers of one decode step share):
//   kDirect     computes it and streams (the stateless call);
//   kBuild      computes it and writes it to a schedule buffer, nothing else;
//   kScheduled  reads it from a schedule buffer and streams: the prefix table, the worker's plan
//               and its first tile addresses arrive in one memory round trip instead of the
//               three dependent ones (context lengths, block table, first tile) of kDirect.
enum : int { kDirect = 0, kBuild = 1, kScheduled = 2 };
constexpr int kPlanInts = 16;  // a worker's plan in the schedule buffer

}  // namespace mfma
}  // namespace kvc
