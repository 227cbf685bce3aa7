// Greedy disjoint layer-pair selection (Alg. 1, second loop; Sec. 4.2): one workgroup per
// conversation; the method itself is select_adjacent() in krul_select_core.h.
#include "krul_common.h"
#include "krul_select_core.h"

namespace krul {
namespace {

constexpr int kSelThreads = 256;

__global__ __launch_bounds__(kSelThreads) void select_pairs_kernel(
    const float *__restrict__ pair_score, const uint8_t *__restrict__ eligible, int n_layers,
    int n_select, int32_t *__restrict__ out_pairs, int32_t *__restrict__ out_count)
{
    extern __shared__ unsigned char sel_smem[];
    const int NP = n_layers - 1;
    float *score = reinterpret_cast<float *>(sel_smem);          // [NP]
    const int b = blockIdx.x;
    for (int l = threadIdx.x; l < NP; l += kSelThreads) score[l] = pair_score[(size_t)b * NP + l];
    select_adjacent(score, eligible ? eligible + (size_t)b * n_layers : nullptr, n_layers, n_select,
                    out_pairs + (size_t)b * n_select, out_count + b, score + NP);
}

// Averages over the heads and the greedy choice of one conversation per workgroup: two steps whose launches cost more
// than the work in them.  Bound by latency: a half-wave per pair reads its head values and adds them by DPP and
// permlane swaps (the same bits as finalize_pairs_kernel), so that one load and five such adds stand between the launch and the
// scores.  (Staged in LDS and added by a thread per pair, head after head: 9.4 us for 31 pairs of 32 heads, 4.8 us now.)
constexpr int kPsThreads = 1024;

__global__ __launch_bounds__(kPsThreads) void pairs_select_kernel(PairsSelectArgs a)
{
    extern __shared__ unsigned char sel_smem[];
    const int NP = a.L - 1, b = blockIdx.x, lane = threadIdx.x & 31;
    float *pc = reinterpret_cast<float *>(sel_smem);   // [NP] pair scores
    for (int i = threadIdx.x >> 5; i < NP; i += kPsThreads / 32) {
        const size_t at = (size_t)b * NP + i;
        const float cs = pair_average(a.head_cos + at * a.Hq, a.Hq, 1.0f, lane);
        const float ds = a.head_dist ? pair_average(a.head_dist + at * a.Hq, a.Hq, 1.0f, lane) : 0.f;
        if (lane == 0) {
            a.pair_cos[at] = pc[i] = cs;
            if (a.head_dist) a.pair_dist[at] = ds;
        }
    }
    // (select_adjacent starts with a barrier)
    select_adjacent(pc, a.eligible ? a.eligible + (size_t)b * a.L : nullptr, a.L, a.n_select,
                    a.out_pairs + (size_t)b * a.n_select, a.out_count + b, pc + NP);
}

}  // namespace

bool pairs_select_fits(int L, int Hq)   // (one workgroup reads a conversation's head values)
{
    return (long long)(L - 1) * Hq <= kPairsSelectMaxHeads;
}

hipError_t launch_pairs_select(const PairsSelectArgs &a, hipStream_t st)
{
    const size_t smem = (size_t)(a.L - 1) * sizeof(float) + select_scratch_bytes(a.L);
    hipLaunchKernelGGL(pairs_select_kernel, dim3(a.B), dim3(kPsThreads), smem, st, a);
    return hipGetLastError();
}

hipError_t launch_select(const float *pair_score, const uint8_t *eligible, int batch, int n_layers,
                         int n_select, int32_t *out_pairs, int32_t *out_count, hipStream_t st)
{
    const int NP = n_layers - 1;
    const size_t smem = (size_t)NP * sizeof(float) + select_scratch_bytes(n_layers);
    hipLaunchKernelGGL(select_pairs_kernel, dim3(batch), dim3(kSelThreads), smem, st, pair_score,
                       eligible, n_layers, n_select, out_pairs, out_count);
    return hipGetLastError();
}

}  // namespace krul
