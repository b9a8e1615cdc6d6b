// Second pass of split-K paged decode attention (gfx950): combine the per-partition
// (max, sum, un-normalised accumulator) triples of every (sequence, query head) whose
// context was split, normalise and cast.
//
// One wavefront per (sequence, head); the arithmetic is pa_merge_row.h.  (m, l) of the first 64 partials are loaded
// speculatively together with the context length, so the kernel is two memory round trips deep.
//
// The number of partials of a row is ceil(context_len / partition_tokens); rows finished by
// the partial kernel (one partial, or an empty context) are skipped.  The balanced kernel
// merges inside its own launch and does not use this one, nor does the vector-ALU kernel where it
// counts the partitions of a row.
#include <math.h>

#include "kvc_internal.h"
#include "pa_merge_row.h"

namespace kvc {

namespace {

__device__ inline uint16_t f32_to_bf16_rne(float x) {
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7fffffffu) > 0x7f800000u) return uint16_t((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return uint16_t(u >> 16);
}
__device__ inline void store_out(float *o, float x) { *o = x; }
__device__ inline void store_out(uint16_t *o, float x) { *o = f32_to_bf16_rne(x); }

template <typename T, int D, bool BASE2>
__global__ __launch_bounds__(kThreads) void pa_merge_kernel(const int32_t *__restrict__ context_lens,
                                                            T *__restrict__ out, Workspace ws,
                                                            AttnParams p) {
    constexpr int DPL = D / 64;  // dims per lane
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int row = blockIdx.x * kWaves + wave;  // seq * num_q_heads + head
    if (row >= p.num_seqs * p.num_q_heads) return;
    const int seq = row / p.num_q_heads;
    const int head = row - seq * p.num_q_heads;
    const float *ml = ws.ml + size_t(row) * p.max_partitions * 2;
    const float *acc = ws.acc + size_t(row) * p.max_partitions * D + lane * DPL;

    // Two independent loads go out together: the context length and (speculatively, whatever
    // the slots hold) the (max, sum) pairs of the first 64 slots.
    const int ctx = min(context_lens[seq], p.max_context_len);
    float2 ml0 = float2{-INFINITY, 0.f};
    if (lane < p.max_partitions) ml0 = *reinterpret_cast<const float2 *>(ml + 2 * lane);
    int nparts = (ctx + p.partition_tokens - 1) / p.partition_tokens;  // <= 1: finished already, or empty
    if (nparts <= 1) return;
    nparts = __builtin_amdgcn_readfirstlane(min(nparts, p.max_partitions));

    float a[DPL], L;
    auto ml_of = [&](int i) { return *reinterpret_cast<const float2 *>(ml + 2 * i); };
    auto acc_of = [&](int i, float (&x)[DPL]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < DPL; ++j) x[j] = acc[size_t(i) * D + j];
    };
    if (nparts <= 64) L = merge_row<DPL, BASE2, 16, true>(ml0, nparts, lane, ml_of, acc_of, a);
    else L = merge_row<DPL, BASE2, 8, false>(ml0, nparts, lane, ml_of, acc_of, a);
#pragma unroll
    for (int j = 0; j < DPL; ++j) store_out(out + size_t(row) * D + lane * DPL + j, a[j] / L);
}

template <typename T, int D>
void launch(bool base2, const int32_t *cl, void *out, Workspace ws, const AttnParams &p, int grid,
            hipStream_t stream) {
    T *o = static_cast<T *>(out);
    const dim3 g(grid), b(kThreads);
    if (base2)
        pa_merge_kernel<T, D, true><<<g, b, 0, stream>>>(cl, o, ws, p);
    else
        pa_merge_kernel<T, D, false><<<g, b, 0, stream>>>(cl, o, ws, p);
}

__global__ void workspace_init_kernel(int32_t *header) {
    header[blockIdx.x * blockDim.x + threadIdx.x] = 0;
}

}  // namespace

hipError_t launch_merge(const int32_t *context_lens, void *out, Workspace ws, const AttnParams &p,
                        int dtype, int head_dim, bool base2, int grid, hipStream_t stream) {
    if (dtype == KVC_F32) {
        if (head_dim == 64) launch<float, 64>(base2, context_lens, out, ws, p, grid, stream);
        else launch<float, 128>(base2, context_lens, out, ws, p, grid, stream);
    } else {
        if (head_dim == 64) launch<uint16_t, 64>(base2, context_lens, out, ws, p, grid, stream);
        else launch<uint16_t, 128>(base2, context_lens, out, ws, p, grid, stream);
    }
    return hipGetLastError();
}

hipError_t launch_workspace_init(void *workspace, hipStream_t stream) {
    constexpr int kWords = int(kWorkspaceHeaderBytes / sizeof(int32_t));
    workspace_init_kernel<<<dim3(kWords / kThreads), dim3(kThreads), 0, stream>>>(static_cast<int32_t *>(workspace));
    return hipGetLastError();
}

}  // namespace kvc
