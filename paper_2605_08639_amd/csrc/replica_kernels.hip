// Layer-shared replica buffer (Section 5.1): the parameter arrays carry EP*r replica slots behind
// the E home experts, refilled for every micro-batch and layer.  The forward push copies each
// live replica's home parameters into its slot, the gradient pull adds each live slot's gradient
// into its home block.  Both are meant to run beside compute on a second stream, so the launch takes
// a small, caller-chosen number of workgroups (the counterpart of the paper's few-SM persistent
// copy kernel).
//
// What bounds them is how many bytes one compute unit keeps in flight (the caller gives 16 units by default, and a
// unit's rate is its outstanding loads over the memory latency) and, beside compute, when a workgroup gets to start.
// Every thread issues all its loads of a chunk before it stores.  A workgroup is 512 threads of at most 128
// registers: it fits on a unit next to one workgroup of the narrow row tiles (two to a unit, 232 registers,
// 72 KiB of LDS), so it starts when one of the two ends.  1024 threads, which a unit takes only when it is
// empty, waited for that as long as tiles were queued.  The table of slots is compacted into LDS in parallel first:
// read entry by entry it costs a memory round trip per slot and position.
// Measured with 8 live slots of 3 x 2048 x 768 parameters, 16 and 64 workgroups, us; in turn 256 threads with four
// loads each (pull: one position at a time), 1024 threads (16 and 8 loads), this:
//                                       push 16        push 64        pull 16           pull 64
//   alone                               98  86  88     32  31  28     1085  334  332    293  114  114
//   beside narrow tiles, 64 experts
//     of 3136 x 1408, 400 rows each    525 770 289    209 637 157     2898 1114  698    794  751  277
//   beside wide tiles, 2048 x 1536     437 241 242    158 105 106     2685  633  637    754  217  212
//   beside short groups' weight
//     gradients, 2048 x 1408           686 271 272    251 107 104     4525  904  925   1213  292  280
// Alone on larger blocks 1024 threads are 5 % faster (8 slots of 3 x 4096 x 1536, push 16: 485 against 510).
#include "common.h"
#include <type_traits>

namespace relibra {

constexpr int kReplicaThreads = 512;
constexpr int kPushLoads = 24, kPullLoads = 12;            // 16-byte pieces per thread and chunk (pull: of both operands)
constexpr int kPushTail = 8;                               // the same in a block's last, partial chunk (of a small block: its only one)
constexpr int kTableChunk = kReplicaThreads;               // slots listed at a time
constexpr int kReplicaWaves = 4;                           // waves per SIMD that the registers leave room for: at most 128 each
// Sizes inside a block are 32-bit: 64 GiB, and three tensors of at least two blocks do not fit the card.  (Besides, a
// 64-bit chunk length used both as a branch condition and as a value has come out of the compiler as a select on
// a condition code that something else had set.)
constexpr size_t kMaxVec = 0xffff0000u;
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
// A wave-uniform pointer as a scalar base of its own: a lane's address is that base and one 32-bit offset, the same for
// all its loads.  (Otherwise the compiler forms a 64-bit address per load, two more registers each.)
#define RELIBRA_GLOBAL __attribute__((address_space(1)))
template <class T> __device__ __forceinline__ RELIBRA_GLOBAL T *scalar_base(T *p)
{
    RELIBRA_GLOBAL T *g = (RELIBRA_GLOBAL T *)p;
#ifdef __HIP_DEVICE_COMPILE__
    asm("" : "+s"(g));
#endif
    return g;
}

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
// (vec 16-byte vectors each) are copied to slot E + s.  The (slot, tensor, chunk) units
// are dealt to the workgroups round robin.
__global__ void __launch_bounds__(kReplicaThreads, kReplicaWaves)
replica_push_kernel(u32x4_t *__restrict__ Wg, u32x4_t *__restrict__ Wu, u32x4_t *__restrict__ Wd,
                    const int32_t *__restrict__ replica_expert, int n_slots, int E, uint32_t vec,
                    int32_t *__restrict__ err_flag)
{
    __shared__ LiveSlots l;
    constexpr uint32_t CHUNK = kReplicaThreads * kPushLoads;
    const uint32_t chunks = (vec + CHUNK - 1) / CHUNK, units = 3 * chunks;      // per slot
    bool bad = false;
    for (int base = 0; base < n_slots; base += kTableChunk) {
        list_live(replica_expert, base, n_slots, E, l, bad);
        const int live = uniform(l.n);
        for (uint32_t u = blockIdx.x; u < (uint32_t)live * units; u += gridDim.x) {
            const uint32_t i = u / units, c = u - i * units, which = c / chunks;
            u32x4_t *__restrict__ W = which == 0 ? Wg : which == 1 ? Wu : Wd;
            const uint32_t at = (c - which * chunks) * CHUNK, n = vec - at;      // vectors from here to the block's end
            const u32x4_t *src = W + (size_t)uniform(l.expert[i]) * vec + at;
            u32x4_t *dst = W + (size_t)(E + uniform(l.slot[i])) * vec + at;
            if (n >= CHUNK) {
                u32x4_t v[kPushLoads];
#pragma unroll
                for (int j = 0; j < kPushLoads; ++j) v[j] = scalar_base(src + j * kReplicaThreads)[threadIdx.x];
#pragma unroll
                for (int j = 0; j < kPushLoads; ++j) scalar_base(dst + j * kReplicaThreads)[threadIdx.x] = v[j];
                continue;
            }
            for (uint32_t from = 0; from < n; from += kPushTail * kReplicaThreads) {       // past the block's end: its last vector again, not stored
                u32x4_t v[kPushTail];
#pragma unroll
                for (int j = 0; j < kPushTail; ++j) v[j] = scalar_base(src)[min(from + j * kReplicaThreads + threadIdx.x, n - 1)];
#pragma unroll
                for (int j = 0; j < kPushTail; ++j)
                    if (from + j * kReplicaThreads + threadIdx.x < n) scalar_base(dst)[from + j * kReplicaThreads + threadIdx.x] = v[j];
            }
        }
    }
    if (bad && blockIdx.x == 0) atomicOr(err_flag, RELIBRA_ERR_ID_RANGE);
}

// Gradient return: for every live slot s (replica_expert[s] = e >= 0), in ascending slot order,
// dW[e] += dW[E + s], for the three gradient tensors (vec f32x4_t vectors each).  An
// expert's slots are added up in registers, its home block is read and written once.  The workgroup
// that owns a chunk of an expert's block depends on the expert and the chunk only, not on the place in
// the list, and a thread owns its elements inside the chunk: every element's sum has the same fixed
// order as the in-line sum of the backward call, also across lists; results are identical bit for bit.
__global__ void __launch_bounds__(kReplicaThreads, kReplicaWaves)
replica_pull_kernel(f32x4_t *__restrict__ dWg, f32x4_t *__restrict__ dWu, f32x4_t *__restrict__ dWd,
                    const int32_t *__restrict__ replica_expert, int n_slots, int E, uint32_t vec,
                    int32_t *__restrict__ err_flag)
{
    __shared__ LiveSlots l;
    constexpr uint32_t CHUNK = kReplicaThreads * kPullLoads;
    const uint32_t chunks = (vec + CHUNK - 1) / CHUNK, units = 3 * chunks;      // per expert
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
        const int live = uniform(l.n);
        for (int i = 0; i < live; ++i) {
            if (!uniform(l.head[i])) continue;
            const int e = uniform(l.expert[i]);
            const uint32_t turn = (uint32_t)e % gridDim.x * (units % gridDim.x) % gridDim.x;       // unit c of expert e belongs to workgroup (turn + c) % grid
            for (uint32_t c = (blockIdx.x + gridDim.x - turn) % gridDim.x; c < units; c += gridDim.x) {
                const uint32_t which = c / chunks;
                f32x4_t *__restrict__ dW = which == 0 ? dWg : which == 1 ? dWu : dWd;
                const uint32_t at = (c - which * chunks) * CHUNK, n = vec - at;      // vectors from here to the block's end
                f32x4_t *home = dW + (size_t)e * vec + at;
                auto pull = [&](auto whole) __attribute__((always_inline)) {
                    // past the block's end: its last vector again, not stored
                    auto lane_at = [&](auto *p, int j) __attribute__((always_inline)) {
                        return scalar_base(decltype(whole)::value ? p + j * kReplicaThreads : p) + (decltype(whole)::value ? threadIdx.x : min(j * kReplicaThreads + threadIdx.x, n - 1));
                    };
                    f32x4_t d[kPullLoads];
#pragma unroll
                    for (int j = 0; j < kPullLoads; ++j) d[j] = *lane_at(home, j);
                    for (int k = i; k >= 0; k = uniform(l.next[k])) {
                        const f32x4_t *src = dW + (size_t)(E + uniform(l.slot[k])) * vec + at;
                        f32x4_t v[kPullLoads];
#pragma unroll
                        for (int j = 0; j < kPullLoads; ++j) v[j] = *lane_at(src, j);
#pragma unroll
                        for (int j = 0; j < kPullLoads; ++j) d[j] += v[j];
                    }
#pragma unroll
                    for (int j = 0; j < kPullLoads; ++j)
                        if (decltype(whole)::value || j * kReplicaThreads + threadIdx.x < n) *lane_at(home, j) = d[j];
                };
                if (n >= CHUNK) pull(std::true_type{});
                else pull(std::false_type{});
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
    const size_t per_expert = (size_t)h * hff / 8;
    if (per_expert > kMaxVec) return RELIBRA_EUNSUPPORTED;
    const uint32_t vec = (uint32_t)per_expert;
    const int grid = n_workgroups > 4096 ? 4096 : n_workgroups;
    RELIBRA_LAUNCH(RELIBRA_K_REPLICA_PUSH, stream, replica_push_kernel<<<grid, kReplicaThreads, 0, stream>>>(
        (u32x4_t *)Wg_dev, (u32x4_t *)Wu_dev, (u32x4_t *)Wd_dev, replica_expert_dev, EP * r, E, vec, err_flag_dev));
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
    const size_t per_expert = (size_t)h * hff / 4;
    if (per_expert > kMaxVec) return RELIBRA_EUNSUPPORTED;
    const uint32_t vec = (uint32_t)per_expert;
    const int grid = n_workgroups > 4096 ? 4096 : n_workgroups;
    RELIBRA_LAUNCH(RELIBRA_K_REPLICA_PULL, stream, replica_pull_kernel<<<grid, kReplicaThreads, 0, stream>>>(
        (f32x4_t *)dWg_dev, (f32x4_t *)dWu_dev, (f32x4_t *)dWd_dev, replica_expert_dev, EP * r, E, vec, err_flag_dev));
    RELIBRA_HIP_TRY(launch_check());
    return RELIBRA_OK;
}
