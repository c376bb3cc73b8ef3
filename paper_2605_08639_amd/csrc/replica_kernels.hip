// Layer-shared replica buffer (Section 5.1): the parameter arrays carry EP*r replica slots behind
// the E home experts, refilled for every micro-batch and layer.  The forward push copies each
// live replica's home parameters into its slot, the gradient pull adds each live slot's gradient
// into its home block.  Both are meant to run beside compute on a second stream, so the launch takes
// a small, caller-chosen number of workgroups (the counterpart of the paper's few-SM persistent
// copy kernel).
//
// What bounds them is how many bytes one compute unit keeps in flight: the caller gives 16 units by
// default, and a unit's rate is its outstanding loads over the memory latency.  A workgroup is
// therefore as large as a compute unit takes (1024 threads) and every thread issues all its loads of
// a chunk before it stores.  The table of slots is compacted into LDS in parallel first: read entry by
// entry it costs a memory round trip per slot and position.  Measured with 16 workgroups, 8 live slots
// of 3 x 2048 x 768 parameters: push (151 MB moved) 125 us, 153 us with 256 threads and four loads each;
// pull (453 MB) 425 us, 1384 us with 256 threads and one position at a time.  Both then move about 70 GB/s
// per compute unit; half the loads per thread cost 12 and 1 %, half the threads 12 and 5 %.
#include "common.h"

namespace relibra {

constexpr int kReplicaThreads = 1024;
constexpr int kPushLoads = 16, kPullLoads = 8;             // 16-byte pieces per thread and chunk (pull: of both operands)
constexpr int kTableChunk = kReplicaThreads;               // slots listed at a time
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// The live ones of table entries base .. base + kTableChunk - 1, in ascending slot order.
struct LiveSlots {
    int n;
    int expert[kTableChunk], slot[kTableChunk];
    int next[kTableChunk];                                 // pull: next entry with the same expert, -1: none
    int head[kTableChunk];                                 // pull: 1 if no earlier entry has the same expert
    int wave_n[kReplicaThreads / 64];
};

__device__ __forceinline__ void list_live(const int32_t *__restrict__ replica_expert, int base, int n_slots, int E, LiveSlots &l,
                                          bool &bad)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int e = base + tid < n_slots ? replica_expert[base + tid] : -1;
    if (e >= E) { bad = true; e = -1; }
    const uint64_t live = __ballot(e >= 0);
    __syncthreads();                                       // the previous list is no longer read
    if (lane == 0) l.wave_n[wave] = __popcll(live);
    __syncthreads();
    int at = 0, n = 0;
    for (int w = 0; w < kReplicaThreads / 64; ++w) {
        if (w < wave) at += l.wave_n[w];
        n += l.wave_n[w];
    }
    if (e >= 0) {
        at += __popcll(live & (((uint64_t)1 << lane) - 1));
        l.expert[at] = e;
        l.slot[at] = base + tid;
    }
    if (tid == 0) l.n = n;
    __syncthreads();
}

// For every live slot s (replica_expert[s] = e >= 0): the three parameter blocks of expert e
// (per_expert_vec 16-byte vectors each) are copied to slot E + s.  The (slot, tensor, chunk) units
// are dealt to the workgroups round robin.
__global__ void __launch_bounds__(kReplicaThreads)
replica_push_kernel(u32x4_t *__restrict__ Wg, u32x4_t *__restrict__ Wu, u32x4_t *__restrict__ Wd,
                    const int32_t *__restrict__ replica_expert, int n_slots, int E, size_t per_expert_vec,
                    int32_t *__restrict__ err_flag)
{
    __shared__ LiveSlots l;
    constexpr size_t CHUNK = (size_t)kReplicaThreads * kPushLoads;
    const size_t chunks = (per_expert_vec + CHUNK - 1) / CHUNK, units = 3 * chunks;      // per slot
    bool bad = false;
    for (int base = 0; base < n_slots; base += kTableChunk) {
        list_live(replica_expert, base, n_slots, E, l, bad);
        for (size_t u = blockIdx.x; u < (size_t)l.n * units; u += gridDim.x) {
            const int i = (int)(u / units);
            const size_t c = u - (size_t)i * units, which = c / chunks;
            u32x4_t *__restrict__ W = which == 0 ? Wg : which == 1 ? Wu : Wd;
            const size_t at = (c - which * chunks) * CHUNK;
            const int n = (int)min(CHUNK, per_expert_vec - at);
            const u32x4_t *__restrict__ src = W + (size_t)l.expert[i] * per_expert_vec + at;
            u32x4_t *__restrict__ dst = W + (size_t)(E + l.slot[i]) * per_expert_vec + at;
            if (n < (int)CHUNK) {                          // the block's last chunk
                for (int j = threadIdx.x; j < n; j += kReplicaThreads) dst[j] = src[j];
                continue;
            }
            u32x4_t v[kPushLoads];
#pragma unroll
            for (int j = 0; j < kPushLoads; ++j) v[j] = src[threadIdx.x + j * kReplicaThreads];
#pragma unroll
            for (int j = 0; j < kPushLoads; ++j) dst[threadIdx.x + j * kReplicaThreads] = v[j];
        }
    }
    if (bad && blockIdx.x == 0) atomicOr(err_flag, RELIBRA_ERR_ID_RANGE);
}

// Gradient return: for every live slot s (replica_expert[s] = e >= 0), in ascending slot order,
// dW[e] += dW[E + s], for the three gradient tensors (per_expert_vec f32x4_t vectors each).  An
// expert's slots are added up in registers, its home block is read and written once.  The workgroup
// that owns a chunk of an expert's block depends on the expert and the chunk only, not on the place in
// the list, and a thread owns its elements inside the chunk: every element's sum has the same fixed
// order as the in-line sum of the backward call, also across lists; results are identical bit for bit.
__global__ void __launch_bounds__(kReplicaThreads)
replica_pull_kernel(f32x4_t *__restrict__ dWg, f32x4_t *__restrict__ dWu, f32x4_t *__restrict__ dWd,
                    const int32_t *__restrict__ replica_expert, int n_slots, int E, size_t per_expert_vec,
                    int32_t *__restrict__ err_flag)
{
    __shared__ LiveSlots l;
    constexpr size_t CHUNK = (size_t)kReplicaThreads * kPullLoads;
    const size_t chunks = (per_expert_vec + CHUNK - 1) / CHUNK, units = 3 * chunks;      // per expert
    bool bad = false;
    for (int base = 0; base < n_slots; base += kTableChunk) {
        list_live(replica_expert, base, n_slots, E, l, bad);
        if ((int)threadIdx.x < l.n) {
            const int mine = l.expert[threadIdx.x];
            int head = 1, next = -1;
            for (int j = 0; j < l.n; ++j)
                if (l.expert[j] == mine) {
                    if (j < (int)threadIdx.x) head = 0;
                    else if (j > (int)threadIdx.x && next < 0) next = j;
                }
            l.head[threadIdx.x] = head;
            l.next[threadIdx.x] = next;
        }
        __syncthreads();
        for (int i = 0; i < l.n; ++i) {
            if (!l.head[i]) continue;
            const int e = l.expert[i];
            const size_t turn = (size_t)e * units % gridDim.x;       // unit c of expert e belongs to workgroup (turn + c) % grid
            for (size_t c = (blockIdx.x + gridDim.x - turn) % gridDim.x; c < units; c += gridDim.x) {
                const size_t which = c / chunks;
                f32x4_t *__restrict__ dW = which == 0 ? dWg : which == 1 ? dWu : dWd;
                const size_t at = (c - which * chunks) * CHUNK;
                const int n = (int)min(CHUNK, per_expert_vec - at);
                f32x4_t *__restrict__ home = dW + (size_t)e * per_expert_vec + at;
                int idx[kPullLoads];
                f32x4_t d[kPullLoads];
#pragma unroll
                for (int j = 0; j < kPullLoads; ++j) {     // past the end: the last vector again, not stored
                    idx[j] = min((int)threadIdx.x + j * kReplicaThreads, n - 1);
                    d[j] = home[idx[j]];
                }
                for (int k = i; k >= 0; k = l.next[k]) {
                    const f32x4_t *__restrict__ src = dW + (size_t)(E + l.slot[k]) * per_expert_vec + at;
                    f32x4_t v[kPullLoads];
#pragma unroll
                    for (int j = 0; j < kPullLoads; ++j) v[j] = src[idx[j]];
#pragma unroll
                    for (int j = 0; j < kPullLoads; ++j) d[j] += v[j];
                }
#pragma unroll
                for (int j = 0; j < kPullLoads; ++j)
                    if ((int)threadIdx.x + j * kReplicaThreads < n) home[idx[j]] = d[j];
            }
        }
    }
    if (bad && blockIdx.x == 0) atomicOr(err_flag, RELIBRA_ERR_ID_RANGE);
}

}  // namespace relibra

using namespace relibra;

extern "C" int relibra_replica_push(void *Wg_dev, void *Wu_dev, void *Wd_dev,
                                    const int32_t *replica_expert_dev, int E, int EP, int r, int h, int hff,
                                    int n_workgroups, int32_t *err_flag_dev, relibra_stream stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (E < 1 || EP < 1 || r < 0 || h < 8 || hff < 8 || n_workgroups < 1) return RELIBRA_EINVAL;
    if (((size_t)h * hff) % 8) return RELIBRA_EUNSUPPORTED;
    if (r == 0) return RELIBRA_OK;
    if (!Wg_dev || !Wu_dev || !Wd_dev || !replica_expert_dev || !err_flag_dev) return RELIBRA_EINVAL;
    if (!aligned16(Wg_dev) || !aligned16(Wu_dev) || !aligned16(Wd_dev)) return RELIBRA_EINVAL;
    const size_t per_expert_vec = (size_t)h * hff / 8;
    const int grid = n_workgroups > 4096 ? 4096 : n_workgroups;
    RELIBRA_LAUNCH(RELIBRA_K_REPLICA_PUSH, stream, replica_push_kernel<<<grid, kReplicaThreads, 0, stream>>>(
        (u32x4_t *)Wg_dev, (u32x4_t *)Wu_dev, (u32x4_t *)Wd_dev, replica_expert_dev, EP * r, E, per_expert_vec, err_flag_dev));
    RELIBRA_HIP_TRY(launch_check());
    return RELIBRA_OK;
}

extern "C" int relibra_replica_pull(float *dWg_dev, float *dWu_dev, float *dWd_dev,
                                    const int32_t *replica_expert_dev, int E, int EP, int r, int h, int hff,
                                    int n_workgroups, int32_t *err_flag_dev, relibra_stream stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (E < 1 || EP < 1 || r < 0 || h < 4 || hff < 4 || n_workgroups < 1) return RELIBRA_EINVAL;
    if (((size_t)h * hff) % 4) return RELIBRA_EUNSUPPORTED;
    if (r == 0) return RELIBRA_OK;
    if (!dWg_dev || !dWu_dev || !dWd_dev || !replica_expert_dev || !err_flag_dev) return RELIBRA_EINVAL;
    if (!aligned16(dWg_dev) || !aligned16(dWu_dev) || !aligned16(dWd_dev)) return RELIBRA_EINVAL;
    const size_t per_expert_vec = (size_t)h * hff / 4;
    const int grid = n_workgroups > 4096 ? 4096 : n_workgroups;
    RELIBRA_LAUNCH(RELIBRA_K_REPLICA_PULL, stream, replica_pull_kernel<<<grid, kReplicaThreads, 0, stream>>>(
        (f32x4_t *)dWg_dev, (f32x4_t *)dWu_dev, (f32x4_t *)dWd_dev, replica_expert_dev, EP * r, E, per_expert_vec, err_flag_dev));
    RELIBRA_HIP_TRY(launch_check());
    return RELIBRA_OK;
}
