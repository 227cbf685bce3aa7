// Row similarity and token-wise aggregation (Sec. 5 / Sec. 7: per-token similarities
// are added up; Sec. 4.2: the average over heads).
//
// finalize_heads: one workgroup per (conversation, pair, query head).  A few lanes
// share each query row: they merge the row's partial records of the two layers
// onto a common reference exponent (fixed butterfly order), form the cosine and
// (from the a^2 + b^2 - 2ab expansion of Sec. 7) the Euclidean distance of the two
// attention rows, and the workgroup sums over rows in a fixed tree order.
// finalize_pairs: 32 lanes per (conversation, pair) average the heads (pair_average).
//
// These kernels are bound by the latency of their few loads, unless there are thousands of rows: record addresses are
// one multiplication apart, and a lane asks for the records of four partials at once.  (One merge after the other,
// each load waited for: 7.9 us for 64 rows of 992 heads with 16 partials, 6.9 us now; 36 -> 29 us for 2048 rows.)
#include "krul_common.h"
#include "krul_select_core.h"

namespace krul {
namespace {

constexpr int kThreads = 256;

__device__ inline float block_sum(float v, float *red)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    float s = 0.f;
    for (int i = 0; i < kThreads / 64; ++i) s += red[i];
    return s;
}

// Running merge of partial records of one row for a layer pair (a = layer l, b = l+1):
// exponents Ma, Mb; Z and N2 of both layers and the cross term C, all relative to them.  (exp2f, not the bare instruction: a
// sum all of whose terms lie 2^126 to 2^149 below the row's largest exponential is subnormal, not zero.)
struct RowAcc {
    float Ma, Za, Na, Mb, Zb, Nb, C;
};

__device__ inline void merge_into(RowAcc &r, float ma, float za, float na, float mb, float zb, float nb, float c)
{
    const float Ma = fmaxf(r.Ma, ma), Mb = fmaxf(r.Mb, mb);
    const float fa0 = exp2f(r.Ma - Ma), fa1 = exp2f(ma - Ma);
    const float fb0 = exp2f(r.Mb - Mb), fb1 = exp2f(mb - Mb);
    r.Za = r.Za * fa0 + za * fa1;
    r.Na = r.Na * (fa0 * fa0) + na * (fa1 * fa1);
    r.Zb = r.Zb * fb0 + zb * fb1;
    r.Nb = r.Nb * (fb0 * fb0) + nb * (fb1 * fb1);
    r.C = r.C * (fa0 * fb0) + c * (fa1 * fb1);
    r.Ma = Ma;
    r.Mb = Mb;
}

// Where a row's records of layer l are: partial p at at + p * step (see state_index).
struct RowRecords {
    size_t at, step;
    int next_layer;   // from a layer's record to the next layer's
};
__device__ inline RowRecords row_records(const StateLayout &y, int u, int r, int l)
{
    RowRecords q;
    if (y.variant == kGeneric) {
        q.step = (size_t)y.n_layers;
        q.next_layer = 1;
    } else {
        const int r_wg = y.wr * y.rb * 32;
        q.step = (size_t)y.n_row_tiles * y.n_layers * r_wg;
        q.next_layer = r_wg;
    }
    q.at = state_index(y, u, r, 0, l);
    return q;
}

constexpr int kBatch = 4;   // partials whose records a lane asks for at once

struct HeadsArgs {
    StateLayout lay;
    const float4 *state;
    const float *state_ir;
    int L, Hq, Hkv, Tq, G;
    int want_dist, accumulate;
    int n_items;   // (conversation, pair, head) triples; the (conversation, layer, head) triples of the layer test follow
    int n_all;
    int first;     // of this launch
    float *head_cos, *head_dist, *head_ir;
};

// G lanes of a wave (G a power of two, lanes g*(64/G) + r for g < G) share one query row:
// each merges the partials p = g, g+G, ... and a butterfly over g joins them.  Lanes with
// the same g read consecutive rows, i.e. consecutive records.
//
// PER_WAVE (few rows: all of a head's rows fit the lanes of one wave, G * Tq <= 64): every wave takes a
// (conversation, pair, query head) of its own and sums the rows by shuffles -- a decode step has one row
// per head, and a workgroup per head would be 252 idle threads and four times the workgroups.
//
// Calls f(t, row, g, RW) for the lanes' rows; RW rows share a wave's 64 lanes.
template <bool PER_WAVE, class F>
__device__ inline void for_rows(const HeadsArgs &p, int h, F f)
{
    const int lane = threadIdx.x & 63, wave = PER_WAVE ? 0 : threadIdx.x >> 6;
    const int RW = 64 / p.G;   // rows per wave
    for (int t0 = 0; t0 < p.Tq; t0 += (PER_WAVE ? 1 : kThreads / 64) * RW) {
        const int t = t0 + wave * RW + lane % RW;
        f(t, (h % (p.Hq / p.Hkv)) * p.Tq + t, lane / RW, RW);
    }
}
template <bool PER_WAVE>
__device__ inline float sum_rows(float v, float *red)
{
    if constexpr (!PER_WAVE) return block_sum(v, red);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// IR: also the Initial-Recent layer test (Sec. 4.2; Alg. 1 first loop): per (conversation, layer, head) the
// mean over query rows of Zir / Z -- the attention mass on T_initial and T_recent -- from the
// partial records of each row, merged onto a common exponent like the similarity sums.
template <bool PER_WAVE, bool IR>
__global__ __launch_bounds__(kThreads) void finalize_heads_kernel(HeadsArgs p)
{
    __shared__ float red[kThreads / 64];
    int item = p.first + (PER_WAVE ? blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6) : blockIdx.x);
    if (PER_WAVE && item >= p.n_all) return;   // (a whole wave: no barrier follows in this form)
    const bool first = (PER_WAVE ? threadIdx.x & 63 : threadIdx.x) == 0;
    const int P = p.lay.partials;

    if (IR && item >= p.n_items) {
        item -= p.n_items;
        const int h = item % p.Hq, l = item / p.Hq % p.L, u = item / (p.Hq * p.L) * p.Hkv + h / (p.Hq / p.Hkv);
        float mass = 0.f;
        for_rows<PER_WAVE>(p, h, [&](int t, int r, int g, int RW) {
            float M = kMInit, Z = 0.f, I = 0.f;
            if (t < p.Tq) {
                const RowRecords q = row_records(p.lay, u, r, l);
                for (int p0 = g; p0 < P; p0 += kBatch * p.G) {
                    float am[kBatch], az[kBatch], ai[kBatch];
#pragma unroll
                    for (int i = 0; i < kBatch; ++i) {
                        const size_t idx = q.at + (size_t)min(p0 + i * p.G, P - 1) * q.step;
                        am[i] = p.state[idx].x;
                        az[i] = p.state[idx].y;
                        ai[i] = p.state_ir[idx];
                    }
#pragma unroll
                    for (int i = 0; i < kBatch; ++i) {
                        if (p0 + i * p.G >= P) continue;
                        const float Mn = fmaxf(M, am[i]);
                        const float f0 = exp2f(M - Mn), f1 = exp2f(am[i] - Mn);
                        Z = Z * f0 + az[i] * f1;
                        I = I * f0 + ai[i] * f1;
                        M = Mn;
                    }
                }
            }
            for (int off = 32; off >= RW; off >>= 1) {
                const float m2 = __shfl_xor(M, off, 64), z2 = __shfl_xor(Z, off, 64), i2 = __shfl_xor(I, off, 64);
                const float Mn = fmaxf(M, m2);
                const float f0 = exp2f(M - Mn), f1 = exp2f(m2 - Mn);
                Z = Z * f0 + z2 * f1;
                I = I * f0 + i2 * f1;
                M = Mn;
            }
            if (t < p.Tq && g == 0) mass += I / Z;
        });
        mass = sum_rows<PER_WAVE>(mass, red);
        if (first) p.head_ir[item] = mass / (float)p.Tq;
        return;
    }

    const int NP = p.L - 1, h = item % p.Hq, l = item / p.Hq % NP, u = item / (p.Hq * NP) * p.Hkv + h / (p.Hq / p.Hkv);
    float cs = 0.f, ds = 0.f;
    for_rows<PER_WAVE>(p, h, [&](int t, int r, int g, int RW) {
        RowAcc acc = {kMInit, 0.f, 0.f, kMInit, 0.f, 0.f, 0.f};
        if (t < p.Tq) {
            const RowRecords q = row_records(p.lay, u, r, l);
            for (int p0 = g; p0 < P; p0 += kBatch * p.G) {
                float4 a[kBatch], c[kBatch];
#pragma unroll
                for (int i = 0; i < kBatch; ++i) {
                    const float4 *rec = p.state + q.at + (size_t)min(p0 + i * p.G, P - 1) * q.step;
                    a[i] = rec[0];
                    c[i] = rec[q.next_layer];
                }
#pragma unroll
                for (int i = 0; i < kBatch; ++i)
                    if (p0 + i * p.G < P) merge_into(acc, a[i].x, a[i].y, a[i].z, c[i].x, c[i].y, c[i].z, c[i].w);
            }
        }
        for (int off = 32; off >= RW; off >>= 1) {
            const float ma = __shfl_xor(acc.Ma, off, 64), za = __shfl_xor(acc.Za, off, 64);
            const float na = __shfl_xor(acc.Na, off, 64), mb = __shfl_xor(acc.Mb, off, 64);
            const float zb = __shfl_xor(acc.Zb, off, 64), nb = __shfl_xor(acc.Nb, off, 64);
            const float c = __shfl_xor(acc.C, off, 64);
            merge_into(acc, ma, za, na, mb, zb, nb, c);
        }
        if (t < p.Tq && g == 0) {
            cs += acc.C * rsqrtf(acc.Na * acc.Nb);
            if (p.want_dist) {   // (Z is only accumulated when the distance is asked for)
                const float ia = 1.f / acc.Za, ib = 1.f / acc.Zb;
                const float d2 = acc.Na * ia * ia + acc.Nb * ib * ib - 2.f * acc.C * ia * ib;
                ds += sqrtf(fmaxf(d2, 0.f));
            }
        }
    });
    cs = sum_rows<PER_WAVE>(cs, red);
    ds = sum_rows<PER_WAVE>(ds, red);
    if (first) {
        if (p.accumulate) {   // token-wise running sums over several calls (Sec. 5, Sec. 7 "adds up")
            p.head_cos[item] += cs;
            if (p.want_dist) p.head_dist[item] += ds;
        } else {
            p.head_cos[item] = cs / (float)p.Tq;
            p.head_dist[item] = ds / (float)p.Tq;
        }
    }
}

struct PairsArgs {
    unsigned n_pairs, n_layers;   // of all conversations; n_layers 0 without the layer test
    unsigned first;               // of this launch
    int Hq;
    float scale;             // of the head values: 1 for means, 1/tokens for running sums
    const float *head_cos, *head_dist, *head_ir;
    float *head_out;         // head_cos * scale, or null; may be head_cos
    float *pair_cos, *pair_dist;
    float gamma;
    float *ir_mass;
    uint8_t *eligible;
};

// averages over the heads by 32 lanes per (conversation, pair), and per (conversation, layer) of the Initial-Recent
// test, with the test against gamma
__global__ __launch_bounds__(kThreads) void finalize_pairs_kernel(PairsArgs a)
{
    unsigned i = a.first + blockIdx.x * (kThreads / 32) + (threadIdx.x >> 5);
    const int lane = threadIdx.x & 31;
    if (i >= a.n_pairs + a.n_layers) return;   // (a whole half-wave)
    if (i >= a.n_pairs) {
        i -= a.n_pairs;
        const float m = pair_average(a.head_ir + (size_t)i * a.Hq, a.Hq, 1.0f, lane);
        if (lane != 0) return;
        if (a.ir_mass) a.ir_mass[i] = m;
        if (a.eligible) a.eligible[i] = m >= a.gamma ? 1 : 0;   // below gamma: not an Initial-Recent layer, set aside
        return;
    }
    const float cs = pair_average(a.head_cos + (size_t)i * a.Hq, a.Hq, a.scale, lane,
                                  a.head_out ? a.head_out + (size_t)i * a.Hq : nullptr);
    if (lane == 0) a.pair_cos[i] = cs;
    if (a.pair_dist) {
        const float ds = pair_average(a.head_dist + (size_t)i * a.Hq, a.Hq, a.scale, lane);
        if (lane == 0) a.pair_dist[i] = ds;
    }
}

constexpr int kMostBlocks = 1 << 22;   // of a launch: HIP numbers at most 2^32 threads

hipError_t launch_pairs(PairsArgs a, hipStream_t st)
{
    constexpr unsigned per_block = kThreads / 32, step = (unsigned)kMostBlocks * per_block;
    const unsigned n = a.n_pairs + a.n_layers;
    for (a.first = 0; a.first < n; a.first += step) {
        const unsigned here = n - a.first < step ? n - a.first : step;
        hipLaunchKernelGGL(finalize_pairs_kernel, dim3((here + per_block - 1) / per_block), dim3(kThreads), 0, st, a);
    }
    return hipGetLastError();
}

template <bool PER_WAVE>
void launch_heads(HeadsArgs p, bool ir, hipStream_t st)
{
    constexpr int per_block = PER_WAVE ? kThreads / 64 : 1, step = kMostBlocks * per_block;
    for (long long first = 0; first < p.n_all; first += step) {
        p.first = (int)first;
        const long long here = p.n_all - first < step ? p.n_all - first : step;
        const dim3 grid((unsigned)((here + per_block - 1) / per_block));
        if (ir) hipLaunchKernelGGL((finalize_heads_kernel<PER_WAVE, true>), grid, dim3(kThreads), 0, st, p);
        else hipLaunchKernelGGL((finalize_heads_kernel<PER_WAVE, false>), grid, dim3(kThreads), 0, st, p);
    }
}

}  // namespace

hipError_t launch_finalize(const StateLayout &lay, const float4 *state, int B, int L, int Hq, int Hkv,
                           int Tq, float *head_cos, float *head_dist, float *pair_cos,
                           float *pair_dist, bool accumulate, const IrArgs *ir, hipStream_t st)
{
    HeadsArgs p = {};
    p.lay = lay;
    p.state = state;
    p.L = L;
    p.Hq = Hq;
    p.Hkv = Hkv;
    p.Tq = Tq;
    p.want_dist = pair_dist != nullptr;
    p.accumulate = accumulate ? 1 : 0;
    p.n_items = B * (L - 1) * Hq;
    p.n_all = p.n_items + (ir ? B * L * Hq : 0);
    p.head_cos = head_cos;
    p.head_dist = head_dist;
    if (ir) {
        p.state_ir = ir->state_ir;
        p.head_ir = ir->head_ir;
    }
    p.G = 1;
    if (Tq <= 8) {   // few rows: a wave per head, G lanes per row with G * Tq <= 64
        while (p.G * 2 * Tq <= 64 && p.G < lay.partials) p.G <<= 1;
        launch_heads<true>(p, ir != nullptr, st);
    } else {
        // lanes per row: enough to keep a workgroup's 256 threads busy, at most one per partial
        while (p.G < 64 && p.G * Tq < kThreads && p.G < lay.partials) p.G <<= 1;
        launch_heads<false>(p, ir != nullptr, st);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || accumulate || !pair_cos) return e;   // (no pair scores asked for: the caller forms them)
    PairsArgs a = {};
    a.n_pairs = B * (L - 1);
    a.Hq = Hq;
    a.scale = 1.0f;
    a.head_cos = head_cos;
    a.head_dist = head_dist;
    a.pair_cos = pair_cos;
    a.pair_dist = pair_dist;
    if (ir) {
        a.n_layers = B * L;
        a.head_ir = ir->head_ir;
        a.gamma = ir->gamma;
        a.ir_mass = ir->ir_mass;
        a.eligible = ir->eligible;
    }
    return launch_pairs(a, st);
}

hipError_t launch_scores_from_sums(const float *head_sum, const float *head_dist_sum, int n_pairs_total,
                                   int Hq, float inv_tokens, float *pair_cos, float *head_score,
                                   float *pair_dist, hipStream_t st)
{
    PairsArgs a = {};
    a.n_pairs = n_pairs_total;
    a.Hq = Hq;
    a.scale = inv_tokens;
    a.head_cos = head_sum;
    a.head_dist = head_dist_sum;
    a.head_out = head_score;
    a.pair_cos = pair_cos;
    a.pair_dist = pair_dist;
    return launch_pairs(a, st);
}

}  // namespace krul
