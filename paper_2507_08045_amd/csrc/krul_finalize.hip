// Row similarity and token-wise aggregation (Sec. 5 / Sec. 7: per-token similarities
// are added up; Sec. 4.2: the average over heads).
//
// finalize_heads: a workgroup per (conversation, pair, query head), or a wave per few heads of a kv head.  A few
// lanes share each query row: they merge the row's partial records of the two layers
// onto a common reference exponent (fixed butterfly order), form the cosine and
// (from the a^2 + b^2 - 2ab expansion of Sec. 7) the Euclidean distance of the two
// attention rows, and the sum over rows is taken in a fixed tree order.
// finalize_pairs: 32 lanes per (conversation, pair) average the heads (pair_average).
// heads_select: both, and the greedy choice, for models whose heads one workgroup takes at once.
//
// These kernels are bound by the latency of one chain of steps, unless there are thousands of rows: which rows, their
// records, the merges, the sums.  So the rows are found without a division, a lane asks for the records of four partials at once (one
// merge after the other, each load waited for: 7.9 us for 64 rows of 992 heads with 16 partials, 6.9 so) and
// everything between lanes goes by vector instructions (with
// divisions and shuffles: 4.0 us for 6 heads of 16 rows, 3.7 so; an empty kernel takes 2.5).
#include "krul_common.h"
#include "krul_select_core.h"

namespace krul {
namespace {

constexpr int kThreads = 256;

// Running merge of partial records of one row for a layer pair (a = layer l, b = l+1):
// exponents Ma, Mb; Z and N2 of both layers and the cross term C, all relative to them; with the layer test (IR) also the sums
// Ia, Ib over the initial and recent keys.  (exp2f, not the bare instruction: a
// sum all of whose terms lie 2^126 to 2^149 below the row's largest exponential is subnormal, not zero.)
struct RowAcc {
    float Ma, Za, Na, Mb, Zb, Nb, C, Ia, Ib;
};

template <bool IR>
__device__ inline void merge_into(RowAcc &r, const RowAcc &o)
{
    const float Ma = fmaxf(r.Ma, o.Ma), Mb = fmaxf(r.Mb, o.Mb);
    const float fa0 = exp2f(r.Ma - Ma), fa1 = exp2f(o.Ma - Ma);
    const float fb0 = exp2f(r.Mb - Mb), fb1 = exp2f(o.Mb - Mb);
    r.Za = r.Za * fa0 + o.Za * fa1;
    r.Na = r.Na * (fa0 * fa0) + o.Na * (fa1 * fa1);
    r.Zb = r.Zb * fb0 + o.Zb * fb1;
    r.Nb = r.Nb * (fb0 * fb0) + o.Nb * (fb1 * fb1);
    r.C = r.C * (fa0 * fb0) + o.C * (fa1 * fb1);
    if (IR) {
        r.Ia = r.Ia * fa0 + o.Ia * fa1;
        r.Ib = r.Ib * fb0 + o.Ib * fb1;
    }
    r.Ma = Ma;
    r.Mb = Mb;
}

template <int OFF, bool IR>
__device__ inline void join(RowAcc &r)
{
    const RowAcc o = {across<OFF>(r.Ma), across<OFF>(r.Za), across<OFF>(r.Na), across<OFF>(r.Mb), across<OFF>(r.Zb), across<OFF>(r.Nb),
                      across<OFF>(r.C), IR ? across<OFF>(r.Ia) : 0.f, IR ? across<OFF>(r.Ib) : 0.f};
    merge_into<IR>(r, o);
}

// n / d for n < 2^31 by a multiplication: m = floor(2^32 (2^s - d) / d) + 1 with s = ceil(log2 d) (Granlund and Montgomery, "Division by
// invariant integers using multiplication").
struct Div {
    unsigned d, m, s;
    static Div by(unsigned d)
    {
        const unsigned s = d > 1 ? 32 - (unsigned)__builtin_clz(d - 1) : 0;
        return {d, d == 1u << s ? 1u : (unsigned)((((1ull << s) - d) << 32) / d) + 1u, s};
    }
    __device__ unsigned operator()(unsigned n) const { return (__umulhi(n, m) + n) >> s; }
};

// Where a row's records of layer l are: partial p at at + p * step (see state_index).
struct RowRecords {
    size_t at, step;
    int next_layer;   // from a layer's record to the next layer's
};
__device__ inline RowRecords row_records(const StateLayout &y, const Div &by_tile, int u, int r, int l)
{
    RowRecords q;
    if (y.variant == kGeneric) {
        q.step = (size_t)y.n_layers;
        q.next_layer = 1;
        q.at = ((size_t)u * y.rows_per_unit + r) * y.n_split * y.n_layers + l;
    } else {
        const unsigned r_wg = by_tile.d, rt = by_tile((unsigned)r);
        q.step = (size_t)y.n_row_tiles * y.n_layers * r_wg;
        q.next_layer = (int)r_wg;
        q.at = (((size_t)u * y.n_split * y.n_row_tiles + rt) * y.n_layers + l) * r_wg + ((unsigned)r - rt * r_wg);
    }
    return q;
}

constexpr int kBatch = 4;   // partials whose records a lane asks for at once

struct HeadsArgs {
    StateLayout lay;
    const float4 *state;
    const float *state_ir;
    int L, Hq, Hkv, Tq;
    int G;               // lanes that share a row; a wave takes 64 / G rows
    int TP, H;           // PER_WAVE: rows of a head (Tq, to a power of two), heads of a wave
    int groups;          // ceil(heads per kv head / H)
    Div by_groups, by_hkv, by_pairs, by_tile;   // divisions by groups, Hkv, L - 1, the rows of a row tile
    int want_dist, accumulate;
    int n_items;   // (conversation, pair, kv head, group of heads)
    int first;     // of this launch
    float *head_cos, *head_dist, *head_ir;
};

// G lanes of a wave (G a power of two, lanes g*(64/G) + r for g < G) share one query row:
// each merges the partials p = g, g+G, ... and a butterfly over g joins them.  Lanes with
// the same g read consecutive rows, i.e. consecutive records.
//
// PER_WAVE (few rows): a wave takes H heads of a kv head by itself -- their rows lie one after the other --, lanes
// g*(64/G) + h*TP + t.  A decode step has one row per head: a wave per head would read 64 bytes for 16 and leave three lanes in
// four idle (8 x 992 heads of 8 partials: 10.0 us, 5.2 so).

// Sum over n lanes (a power of two), the same in each of them.
__device__ inline float sum_over(float v, int n)
{
    if (n > 32) v += across<32>(v);
    if (n > 16) v += across<16>(v);
    if (n > 8) v += across<8>(v);
    if (n > 4) v += across<4>(v);
    if (n > 2) v += across<2>(v);
    if (n > 1) v += across<1>(v);
    return v;
}

// A row's records of layers l and l + 1, merged by the lanes that share it (row: there is one), the same in each of them.
template <bool IR>
__device__ inline RowAcc merged_row(const HeadsArgs &p, bool row, int u, int r, int l, int g, int RW, bool last)
{
    const int P = p.lay.partials;
    RowAcc acc = {kMInit, 0.f, 0.f, kMInit, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (row) {
        const RowRecords q = row_records(p.lay, p.by_tile, u, r, l);
        for (int p0 = g; p0 < P; p0 += kBatch * p.G) {
            float4 a[kBatch], c[kBatch];
            float ia[kBatch], ib[kBatch];
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                const size_t at = q.at + (size_t)min(p0 + i * p.G, P - 1) * q.step;
                a[i] = p.state[at];
                c[i] = p.state[at + q.next_layer];
                ia[i] = IR ? p.state_ir[at] : 0.f;
                ib[i] = last ? p.state_ir[at + q.next_layer] : 0.f;
            }
#pragma unroll
            for (int i = 0; i < kBatch; ++i)
                if (p0 + i * p.G < P)
                    merge_into<IR>(acc, RowAcc{a[i].x, a[i].y, a[i].z, c[i].x, c[i].y, c[i].z, c[i].w, ia[i], ib[i]});
        }
    }
    if (RW <= 32) join<32, IR>(acc);
    if (RW <= 16) join<16, IR>(acc);
    if (RW <= 8) join<8, IR>(acc);
    if (RW <= 4) join<4, IR>(acc);
    if (RW <= 2) join<2, IR>(acc);
    if (RW <= 1) join<1, IR>(acc);
    return acc;
}

// ... and what the row adds to its head's sums.
__device__ inline void add_row(const RowAcc &acc, int want_dist, float &cs, float &ds)
{
    cs += acc.C * rsqrtf(acc.Na * acc.Nb);
    if (want_dist) {   // (Z is only accumulated when the distance is asked for)
        const float ia = 1.f / acc.Za, ib = 1.f / acc.Zb;
        const float d2 = acc.Na * ia * ia + acc.Nb * ib * ib - 2.f * acc.C * ia * ib;
        ds += sqrtf(fmaxf(d2, 0.f));
    }
}

// IR: also the Initial-Recent layer test (Sec. 4.2; Alg. 1 first loop): per (conversation, layer, head) the
// mean over query rows of Zir / Z -- the attention mass on T_initial and T_recent -- from the same records: a pair's first
// layer's, the last pair's second layer's too.  (As items of their own, which read every record once more: 17.9 us for 2 x
// 32 layers of 32 heads of 77 rows with the pairs' scores, 15.4 so.)
template <bool PER_WAVE, bool IR>
__global__ __launch_bounds__(kThreads) void finalize_heads_kernel(HeadsArgs p)
{
    __shared__ float4 red[PER_WAVE ? 1 : kThreads / 64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int item = p.first + (PER_WAVE ? blockIdx.x * (kThreads / 64) + wave : blockIdx.x);
    if (PER_WAVE && item >= p.n_items) return;   // (a whole wave: no barrier follows in this form)

    // (conversation b, pair l, kv head, group of heads): each is the remainder of a division
    const int t1 = p.groups > 1 ? (int)p.by_groups(item) : item, group = item - t1 * p.groups;
    const int bl = (int)p.by_hkv(t1), kvh = t1 - bl * p.Hkv;
    const int b = (int)p.by_pairs(bl), l = bl - b * (p.L - 1), u = b * p.Hkv + kvh;
    const int RW = 64 / p.G, g = lane / RW, in_wave = lane % RW;   // (powers of two)
    const int heads = p.lay.rows_per_unit / p.Tq;   // of the kv head
    const int head = group * p.H + (PER_WAVE ? in_wave / p.TP : 0), t_first = PER_WAVE ? in_wave % p.TP : wave * RW + in_wave;
    const int out = bl * p.Hq + kvh * heads + head;
    const bool writes = head < heads && (PER_WAVE ? g == 0 && t_first == 0 : threadIdx.x == 0);
    float old_cos = 0.f, old_dist = 0.f;   // token-wise running sums over several calls (Sec. 5, Sec. 7 "adds up")
    if (p.accumulate && writes) {
        old_cos = p.head_cos[out];
        if (p.want_dist) old_dist = p.head_dist[out];
    }
    const bool last = IR && l == p.L - 2;
    float cs = 0.f, ds = 0.f, mass_a = 0.f, mass_b = 0.f;
    for (int t = t_first; t - t_first < p.Tq; t += PER_WAVE ? 64 : kThreads / 64 * RW) {   // (PER_WAVE: once)
        const bool row = t < p.Tq && head < heads;
        const RowAcc acc = merged_row<IR>(p, row, u, head * p.Tq + t, l, g, RW, last);
        if (row && g == 0) {
            add_row(acc, p.want_dist, cs, ds);
            if (IR) mass_a += acc.Ia / acc.Za;
            if (last) mass_b += acc.Ib / acc.Zb;
        }
    }
    cs = sum_over(cs, PER_WAVE ? p.TP : RW);
    ds = sum_over(ds, PER_WAVE ? p.TP : RW);
    if (IR) {
        mass_a = sum_over(mass_a, PER_WAVE ? p.TP : RW);
        mass_b = sum_over(mass_b, PER_WAVE ? p.TP : RW);
    }
    if constexpr (!PER_WAVE) {
        if (lane == 0) red[wave] = make_float4(cs, ds, mass_a, mass_b);
        __syncthreads();
        cs = ds = mass_a = mass_b = 0.f;
        for (int i = 0; i < kThreads / 64; ++i) {
            const float4 v = red[i];
            cs += v.x;
            ds += v.y;
            if (IR) mass_a += v.z;
            if (IR) mass_b += v.w;
        }
    }
    if (writes) {
        if (p.accumulate) {
            p.head_cos[out] = old_cos + cs;
            if (p.want_dist) p.head_dist[out] = old_dist + ds;
        } else {
            p.head_cos[out] = cs / (float)p.Tq;
            p.head_dist[out] = ds / (float)p.Tq;
        }
        if (IR) {   // [B][L][Hq]: pair (b, l) is layer (b, l) after b layers more
            float *mass = p.head_ir + out + (size_t)b * p.Hq;
            mass[0] = mass_a / (float)p.Tq;
            if (last) mass[p.Hq] = mass_b / (float)p.Tq;
        }
    }
}

// A small model's heads, averages and greedy choice in one launch, a workgroup per conversation (krul_pair_similarity_select): a wave
// per group of heads, all of them at once (the same bits as finalize_heads_kernel and pairs_select_kernel).  The chain of steps is theirs,
// without the launch between them: 16 float32 tokens over 256 keys of 4 layers, 2 heads, 3.6 and 2.6 us -> 4.2, the call, which the host
// bounds, 20.8 -> 18.6.
constexpr int kTailWaves = 16;

__global__ __launch_bounds__(kTailWaves * 64) void heads_select_kernel(HeadsArgs p, PairsSelectArgs a)
{
    extern __shared__ float tail_smem[];
    const int NP = p.L - 1, b = blockIdx.x, lane = threadIdx.x & 63, item = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float *const hc = tail_smem, *const hd = hc + NP * p.Hq, *const pc = hd + NP * p.Hq;   // head values, [NP] pair scores
    {
        const int t1 = p.groups > 1 ? (int)p.by_groups(item) : item, group = item - t1 * p.groups;
        const int l = (int)p.by_hkv(t1), kvh = t1 - l * p.Hkv;
        const int RW = 64 / p.G, g = lane / RW, in_wave = lane % RW;   // (powers of two)
        const int heads = p.lay.rows_per_unit / p.Tq, head = group * p.H + in_wave / p.TP, t = in_wave % p.TP;
        const bool row = t < p.Tq && head < heads;
        const RowAcc acc = merged_row<false>(p, row, b * p.Hkv + kvh, head * p.Tq + t, l, g, RW, false);
        float cs = 0.f, ds = 0.f;
        if (row && g == 0) add_row(acc, p.want_dist, cs, ds);
        cs = sum_over(cs, p.TP);
        ds = sum_over(ds, p.TP);
        if (head < heads && g == 0 && t == 0) {
            const int out = l * p.Hq + kvh * heads + head;
            hc[out] = cs / (float)p.Tq;
            hd[out] = ds / (float)p.Tq;
            if (p.head_cos) p.head_cos[(size_t)b * NP * p.Hq + out] = hc[out];
        }
    }
    __syncthreads();
    for (int i = threadIdx.x >> 5; i < NP; i += blockDim.x >> 5) {
        const float cs = pair_average(hc + i * p.Hq, p.Hq, 1.0f, lane & 31);
        const float ds = p.want_dist ? pair_average(hd + i * p.Hq, p.Hq, 1.0f, lane & 31) : 0.f;
        if ((lane & 31) == 0) {
            a.pair_cos[(size_t)b * NP + i] = pc[i] = cs;
            if (p.want_dist) a.pair_dist[(size_t)b * NP + i] = ds;
        }
    }
    // (select_adjacent starts with a barrier)
    select_adjacent(pc, a.eligible ? a.eligible + (size_t)b * a.L : nullptr, a.L, a.n_select,
                    a.out_pairs + (size_t)b * a.n_select, a.out_count + b, pc + NP);
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
    for (long long first = 0; first < p.n_items; first += step) {
        p.first = (int)first;
        const long long here = p.n_items - first < step ? p.n_items - first : step;
        const dim3 grid((unsigned)((here + per_block - 1) / per_block));
        if (ir) hipLaunchKernelGGL((finalize_heads_kernel<PER_WAVE, true>), grid, dim3(kThreads), 0, st, p);
        else hipLaunchKernelGGL((finalize_heads_kernel<PER_WAVE, false>), grid, dim3(kThreads), 0, st, p);
    }
}

}  // namespace

namespace {
// Rows to lanes; per_wave: which of the two forms of finalize_heads_kernel.
HeadsArgs heads_args(const StateLayout &lay, const float4 *state, int B, int L, int Hq, int Hkv, int Tq, bool want_dist, bool *per_wave_form)
{
    HeadsArgs p = {};
    p.lay = lay;
    p.state = state;
    p.L = L;
    p.Hq = Hq;
    p.Hkv = Hkv;
    p.Tq = Tq;
    p.want_dist = want_dist ? 1 : 0;
    const int heads = Hq / Hkv;
    p.G = p.TP = p.H = 1;
    const bool per_wave = *per_wave_form = Tq <= 8;
    if (per_wave) {   // few rows: heads of a kv head as long as a lane has one batch of partials, lanes left over share rows
        while (p.TP < Tq) p.TP <<= 1;
        while (p.H < heads && 2 * p.H * p.TP <= 64 && 64 / (2 * p.H * p.TP) * kBatch >= lay.partials) p.H <<= 1;
        while (p.G * 2 * p.H * p.TP <= 64 && p.G < lay.partials) p.G <<= 1;
    } else {
        // lanes per row: runs of rows, each of batches of loads (three times a join's time) and of joins.  (As many lanes as fill the
        // workgroup once: 77 rows, the layers above, 15.4 us in two runs of four lanes a row, 10.3 in one of two; 100 rows over 4000 keys
        // of 24 layers 92.7 and 90.3 us a call.)
        int best = 0;
        for (int lg = 0; 1 << lg <= 64 && (lg == 0 || 1 << (lg - 1) < lay.partials); ++lg) {
            const int runs = ((Tq << lg) + kThreads - 1) / kThreads, batches = (lay.partials + (kBatch << lg) - 1) >> lg >> 2;
            const int cost = runs * (3 * batches + lg);
            if (best == 0 || cost < best) {
                best = cost;
                p.G = 1 << lg;
            }
        }
    }
    p.groups = (heads + p.H - 1) / p.H;
    p.by_groups = Div::by((unsigned)p.groups);
    p.by_hkv = Div::by((unsigned)Hkv);
    p.by_pairs = Div::by((unsigned)L - 1);
    p.by_tile = Div::by(lay.variant == kGeneric ? 1u : (unsigned)(lay.wr * lay.rb * 32));
    p.n_items = B * (L - 1) * Hkv * p.groups;
    return p;
}
}  // namespace

hipError_t launch_finalize(const StateLayout &lay, const float4 *state, int B, int L, int Hq, int Hkv,
                           int Tq, float *head_cos, float *head_dist, float *pair_cos,
                           float *pair_dist, bool accumulate, const IrArgs *ir, hipStream_t st)
{
    bool per_wave;
    HeadsArgs p = heads_args(lay, state, B, L, Hq, Hkv, Tq, pair_dist != nullptr, &per_wave);
    p.accumulate = accumulate ? 1 : 0;
    p.head_cos = head_cos;
    p.head_dist = head_dist;
    if (ir) {
        p.state_ir = ir->state_ir;
        p.head_ir = ir->head_ir;
    }
    if (per_wave) launch_heads<true>(p, ir != nullptr, st);
    else launch_heads<false>(p, ir != nullptr, st);
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

namespace {
// Rows to the lanes of heads_select_kernel; false where it does not take the call.
// One launch where all of a conversation's heads are at work at once.  (In two rounds the chain of steps, 3 us, outlasts what a
// launch costs, 1 to 1.5 on the GPU and 3 on the host: 12.7 -> 16.6 us of GPU time.)
bool heads_select_args(const StateLayout &lay, const float4 *state, int B, int L, int Hq, int Hkv, int Tq, bool want_dist, HeadsArgs *out, int *waves)
{
    bool per_wave;
    HeadsArgs p = heads_args(lay, state, B, L, Hq, Hkv, Tq, want_dist, &per_wave);
    const int RW = 64 / p.G, heads = Hq / Hkv;
    if (!per_wave && Tq <= RW) {   // heads of a wave here too
        while (p.TP < Tq) p.TP <<= 1;
        while (p.H < heads && 2 * p.H * p.TP <= RW) p.H <<= 1;
        p.groups = (heads + p.H - 1) / p.H;
        p.by_groups = Div::by((unsigned)p.groups);
    }
    const long long items = (long long)(L - 1) * Hkv * p.groups;
    *out = p;
    *waves = (int)items;
    return items <= kTailWaves && p.TP >= Tq;
}
}  // namespace

bool select_in_one_launch(const StateLayout &lay, int B, int L, int Hq, int Hkv, int Tq)
{
    HeadsArgs p;
    int waves;
    return heads_select_args(lay, nullptr, B, L, Hq, Hkv, Tq, true, &p, &waves);
}

hipError_t launch_finalize_select(const StateLayout &lay, const float4 *state, int Hkv, int Tq, float *head_out,
                                  float *head_cos, float *head_dist, const PairsSelectArgs &a, hipStream_t st)
{
    HeadsArgs p;
    int waves;
    if (heads_select_args(lay, state, a.B, a.L, a.Hq, Hkv, Tq, a.pair_dist != nullptr, &p, &waves)) {
        p.head_cos = head_out;
        const size_t smem = (size_t)(a.L - 1) * (2 * a.Hq + 1) * sizeof(float) + select_scratch_bytes(a.L);
        hipLaunchKernelGGL(heads_select_kernel, dim3(a.B), dim3((unsigned)waves * 64), smem, st, p, a);
        return hipGetLastError();
    }
    const hipError_t e = launch_finalize(lay, state, a.B, a.L, a.Hq, Hkv, Tq, head_cos, head_dist, nullptr, a.pair_dist, false, nullptr, st);
    return e == hipSuccess ? launch_pairs_select(a, st) : e;
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
