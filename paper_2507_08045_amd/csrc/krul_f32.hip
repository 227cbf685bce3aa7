// Similarity kernel for float32 inputs, and for 16-bit inputs whose heads are larger than the 16-bit kernels' 128, for
// gfx950.
//
// Float32 logits on the bfloat16 matrix cores.  v_mfma_f32_32x32x2_f32 runs at 1/16 of the 16-bit rate and, measured,
// shares its unit with the vector instructions (two of them per MFMA: 155 -> 135 TFLOP/s, nothing overlaps).  Instead
// each operand is split into three bfloat16 of 8 bits each -- x = h + m + l, exactly: 24 bits -- and a product is
// hh + (hm + mh + mm + hl + lh), six bfloat16 MFMAs with float32 sums.  What is left out is ml + lm + ll.  h is x cut off
// after 8 bits (nothing overflows), m the rest rounded to 8 bits, so l has either sign: |m| <= 2^-7 and |l| <= 2^-16 for x in
// [1, 2), and the products of 1 <= x, y < 2 miss at most 2^-22, as often too much as too little.  (With m cut off as well
// |l| reaches 2^-15, always with x's sign: every product came out too small, by up to 2^-21.)  The sum over 128 elements in float32
// arithmetic rounds by several times that.  (One row block to a wave: the large terms and the small ones have an accumulator each.)
//
// What bounds it.  32 keys x 32 rows at head_dim 128 are 48 MFMAs of 32 cycles; splitting the keys takes 352 vector
// instructions per 32 keys of a wave, the exponentials, the share in the query rows' split and the sums some 250 per
// row block, in part beside the MFMAs.  So with more than 32 rows a wave takes two row blocks on one split of the keys, with more than 64 three
// in workgroups of eight waves, one to a CU (24 query tokens over 1021 keys, 96 rows in place of 128 padded ones: this kernel 75 -> 56 us; 1.2 of
// that factor are the rows, less the layers that more pieces of the chain read twice).  No one part bounds the kernel of three row blocks: of a call of 58.5 us without selection a
// build without its MFMAs takes 49.9, without exponentials and sums 52.5, without loads of keys 54.1, without merges 56.4, without the query rows'
// loads 57.1 or their split 57.1, without the keys' split, which hides beside the MFMAs, 59.0.
//
// A workgroup of four (eight) waves owns 32 * RB query rows of a unit (conversation, kv head), a key split and a chunk of
// layers.  It walks the split in tiles of 128 (256) keys (32 per wave) and, inside a tile, the layers of the chunk in order,
// so that the previous layer's exponentials are in registers when the cross term is taken (as in sim_mfma_kernel).
// Keys go from memory to the registers of the one wave that uses them, a layer ahead, with three row blocks half a layer; query rows
// are split once per workgroup and handed round in LDS.  In the MFMA result a lane owns one query row and 16 keys; the row's eight (sixteen)
// partials (two half-waves of each wave) and its running record over the tiles before (its row record, stored after
// every tile) are merged one step late, every wave taking a share of a block's rows.
//
// Measured (one conversation, 32 layers, 32 query / 8 kv heads of 128, the whole call): 24 query tokens over 1021 keys 3080 -> 67 us
// (this kernel 56), 64 over 4096 31400 -> 499 us, against one wave per query row on the vector units, every row fetching the keys
// anew (float32 MFMAs in this kernel's place: 115 and 740 us).  Errors against a float64 evaluation, geometric means over 12 calls drawn
// over the float32 sizes: cosines 4.1e-8, distances 4.7e-8 of themselves (the vector units' float32 products: 5.6e-8 and 6.3e-8); over 700 calls
// in 96-row tiles 4.95e-8 and 4.85e-8, the same calls in 64-row tiles 4.97e-8 and 4.82e-8.
#include "krul_common.h"

namespace krul {
namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;

// Eight consecutive elements as they lie in memory, and as MFMA operands: three bfloat16 planes, or the 16-bit
// elements themselves.
template <typename T> struct Elem8;
template <> struct Elem8<float> {
    static constexpr int kPlanes = 3;
    f32x4 a, b;
    __device__ void split_pair(int i, u32x4 (&o)[3]) const   // elements 2i and 2i + 1
    {
        float x = i < 2 ? a[2 * i] : b[2 * i - 4], y = i < 2 ? a[2 * i + 1] : b[2 * i - 3];
        const auto upper_halves = [](float u, float v) { return __builtin_amdgcn_perm(__float_as_uint(v), __float_as_uint(u), 0x07060302); };
        o[0][i] = upper_halves(x, y);
        x -= __uint_as_float(__float_as_uint(x) & 0xFFFF0000u);   // (exact)
        y -= __uint_as_float(__float_as_uint(y) & 0xFFFF0000u);
        o[1][i] = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{x, y}), bf16x2));   // (to nearest)
        x -= __uint_as_float(o[1][i] << 16);                      // (exact, and of 8 bits)
        y -= __uint_as_float(o[1][i] & 0xFFFF0000u);
        o[2][i] = upper_halves(x, y);
    }
};
template <> struct Elem8<uint16_t> {
    static constexpr int kPlanes = 1;
    u32x4 a;
    __device__ void split_pair(int i, u32x4 (&o)[1]) const { o[0][i] = a[i]; }
};
template <> struct Elem8<_Float16> {
    static constexpr int kPlanes = 1;
    u32x4 a;
    __device__ void split_pair(int i, u32x4 (&o)[1]) const { o[0][i] = a[i]; }
};
// (loads through pointers to global memory: a generic one would wait for LDS as well)
__device__ inline void load8(Elem8<float> &e, uintptr_t p)
{
    typedef const __attribute__((address_space(1))) f32x4 *gp;
    e.a = ((gp)p)[0];
    e.b = ((gp)p)[1];
}
template <typename T>
__device__ inline void load8(Elem8<T> &e, uintptr_t p)
{
    typedef const __attribute__((address_space(1))) u32x4 *gp;
    e.a = *(gp)p;
}

template <typename T>
__device__ inline f32x16 mfma8(u32x4 a, u32x4 b, f32x16 c)
{
    if constexpr (__is_same(T, _Float16))
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// A barrier for data in LDS: it waits for the wave's LDS operations and leaves its loads from memory in flight
// (__syncthreads would wait for those too).
__device__ inline void lds_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Over the P = 8 or 16 lanes that share lane % (64 / P), by vector instructions (shuffles go through LDS and take ten times as long):
// op applied as a butterfly over (4,) 8, 16 and 32, the same in each of them.
template <int P, class Op>
__device__ inline float over_partials(float v, Op op)
{
    static_assert(P == 8 || P == 16, "partials of a row");
    v = op(v, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x128, 0xF, 0xF, true)));   // row_ror 8
    if constexpr (P == 16) v = op(v, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x124, 0xF, 0xF, true)));   // row_ror 4
    const unsigned u = __float_as_uint(v);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    v = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const unsigned w = __float_as_uint(v);
    const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    return op(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
template <int P> __device__ inline float partials_max(float v) { return over_partials<P>(v, [](float a, float b) { return fmaxf(a, b); }); }
template <int P> __device__ inline float partials_sum(float v) { return over_partials<P>(v, [](float a, float b) { return a + b; }); }

constexpr int q_pitch(int ks) { return ks * 32 + 16; }   // bytes of a query row's plane in LDS: 16 rows' 16-byte reads fall into different banks

// KS: MFMA steps of 16 elements that cover the head (head_dim up to 16 * KS; what is past it counts as zero); RB: 32-row blocks per wave; IR: the
// Initial-Recent test too.  Three row blocks take eight waves.
template <typename T, int KS, int RB, bool IR>
__global__ __launch_bounds__(RB == 3 ? 512 : 256) __attribute__((amdgpu_waves_per_eu(KS == 16 && Elem8<T>::kPlanes == 3 ? 1 : 2, 2))) void sim_f32_kernel(SimParams p)
{
    constexpr int PL = Elem8<T>::kPlanes, R_WG = 32 * RB, PITCH = q_pitch(KS);
    constexpr int kWaves = RB == 3 ? 8 : 4, kThreads = kWaves * 64, kTileKeys = kWaves * 32;
    constexpr int TPR = kThreads / 32, QG = (2 * KS + TPR - 1) / TPR;   // threads that stage a query row, and groups of 8 elements for each
    constexpr int P = 2 * kWaves, RPM = 64 / P;                         // partials of a row; rows of a block that a wave merges
    // keys in registers, ahead: a layer's, or half (three row blocks leave no more)
    constexpr int KR = RB == 3 ? KS / 2 : KS;
    typedef __attribute__((address_space(1))) f32x4 *global_f32x4;
    typedef __attribute__((address_space(1))) float *global_f32;
    typedef __attribute__((address_space(3))) f32x4 *lds_f32x4;
    typedef __attribute__((address_space(3))) float *lds_f32;
    __shared__ __attribute__((aligned(16))) unsigned char qlds[RB * PL * 32 * PITCH];   // [row block][plane][row]
    __shared__ f32x4 part[RB][kWaves][64];      // every lane's record of the last step
    __shared__ f32x4 run0[R_WG];                // running records of a chunk's first layer, if they have no place in p.state
    __shared__ float part_ir[IR ? RB : 1][IR ? kWaves : 1][64];
    __shared__ float run0_ir[IR ? R_WG : 1];

    constexpr int DMIN = KS == 16 ? (PL == 1 ? 136 : 200) : KS == 12 ? 136 : KS == 8 ? 104 : KS == 6 ? 72 : 8;   // smallest head size that comes here
    const int d = p.d;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nrt = p.lay.n_row_tiles, nsplit = p.lay.n_split;
    // workgroups: layer chunk, unit, key split, row tile (fastest: they share the keys, and an XCD gets a contiguous run)
    int w;
    {
        const int n = gridDim.x, q = n >> 3, rem = n & 7, x = blockIdx.x & 7;
        w = x * q + min(x, rem) + ((int)blockIdx.x >> 3);
    }
    const int rt = w % nrt, sp = w / nrt % nsplit, uc = w / (nrt * nsplit), n_units = p.B * p.Hkv;
    const int u = uc % n_units, lc = uc / n_units;
    const int b = u / p.Hkv, kvh = u % p.Hkv;
    // the chunk's layers [l_first, l_first + L): the first of them is the last of the chunk before
    const int l_first = (p.L - 1) * lc / p.lay.n_layer_chunks;
    const int L = (p.L - 1) * (lc + 1) / p.lay.n_layer_chunks + 1 - l_first;
    const int S = p.S, Rk = p.lay.rows_per_unit;
    const size_t rec0 = (((size_t)((size_t)u * nsplit + sp) * nrt + rt) * p.L + l_first) * R_WG;   // (see state_index)

    const int key_begin = sp * p.keys_per_split;
    int key_end = min(S, key_begin + p.keys_per_split);
    int row_end[RB];   // causal reading: this lane's query rows see the keys j < row_end
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) row_end[rb] = S;
    if (p.causal) {
        const int r_lo = rt * R_WG, r_hi = min(r_lo + R_WG, Rk) - 1;
        const int t_max = r_lo / p.Tq != r_hi / p.Tq ? p.Tq - 1 : r_hi % p.Tq;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) row_end[rb] = S - p.Tq + min(rt * R_WG + rb * 32 + l32, Rk - 1) % p.Tq + 1;
        key_end = min(key_end, S - p.Tq + t_max + 1);
        if (key_end <= key_begin) {   // no row sees a key of this split
            for (int i = tid + (l_first > 0 ? R_WG : 0); i < L * R_WG; i += kThreads) {
                p.state[rec0 + i] = make_float4(kMInit, 0.f, 0.f, 0.f);
                if (IR) p.state_ir[rec0 + i] = 0.f;
            }
            return;
        }
    }
    const int ntiles = (key_end - key_begin + kTileKeys - 1) / kTileKeys, nsteps = ntiles * L;

    // All loads below are unconditional -- a place that has nothing of its own reads another's, and what must not count
    // is zeroed or masked where it is used -- so that the compiler can count them: a wait for the keys of this step
    // then leaves the loads behind them in flight.

    // ---- query rows of a layer: thread (row tid / TPR, groups tid % TPR, + TPR, ...) -> registers -> split -> LDS.  (Rows
    // past the last are copies of it; their results are never read.  Elements past the head size are zeros, written
    // once below, so that whatever the keys have there does not count.)
    const int qrow = tid / TPR, qc = tid % TPR;
    const T *Q[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
        Q[rb] = static_cast<const T *>(p.q) + (((size_t)b * p.L + l_first) * p.Hq * p.Tq + (size_t)kvh * Rk +
                                               min(rt * R_WG + rb * 32 + qrow, Rk - 1)) * d;
    const size_t q_layer = (size_t)p.Hq * p.Tq * d;
    Elem8<T> qs[RB][QG];
    auto load_q = [&](int l) __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int i = 0; i < QG; ++i) load8(qs[rb][i], (uintptr_t)(Q[rb] + (size_t)l * q_layer + ((i + 1) * TPR * 8 <= DMIN ? (qc + TPR * i) * 8 : min((qc + TPR * i) * 8, d - 8))));
    };
    auto store_q = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int i = 0; i < QG; ++i) {
                if ((i + 1) * TPR * 8 > DMIN && (qc + TPR * i) * 8 >= d) continue;
                u32x4 o[PL];
#pragma unroll
                for (int e = 0; e < 4; ++e) qs[rb][i].split_pair(e, o);
#pragma unroll
                for (int pl = 0; pl < PL; ++pl)
                    *reinterpret_cast<u32x4 *>(qlds + ((rb * PL + pl) * 32 + qrow) * PITCH + (qc + TPR * i) * 16) = o[pl];
            }
    };

    // ---- keys: lane l32 of both half-waves reads key l32 of the wave's 32, half h the elements 16 ks + 8 h .. + 7
    size_t koff = 0;   // of this lane's key in its layer
    auto find_key = [&](int tile) __attribute__((always_inline)) {
        const int key = min(key_begin + tile * kTileKeys + wave * 32 + l32, S - 1);   // (keys past the last are masked)
        koff = (size_t)kvh * p.k_stride_h + half * 8;
        if (p.block_table)
            koff += (size_t)p.block_table[(size_t)b * p.max_blocks + (key >> p.page_shift)] * p.k_stride_page +
                    (size_t)(key & ((1 << p.page_shift) - 1)) * p.k_stride_s;
        else
            koff += (size_t)b * p.k_stride_b + (size_t)key * p.k_stride_s;
    };
    auto key_ptr = [&](int l) __attribute__((always_inline)) -> uintptr_t {
        typedef const __attribute__((address_space(4))) unsigned long long *const_u64_ptr;   // constant memory: scalar loads
        const uintptr_t layer = p.k_tab ? (uintptr_t)((const_u64_ptr)(uintptr_t)p.k_tab)[l_first + l]
                                        : (uintptr_t)(static_cast<const T *>(p.k) + (size_t)(l_first + l) * p.k_stride_l);
        return layer + koff * sizeof(T);
    };
    Elem8<T> kr[KR];
    auto load_k = [&](uintptr_t key, int ks) __attribute__((always_inline)) {
        // (key: the lane's half is in it already where no clamp to the head size is needed)
        if (ks * 16 + 16 <= DMIN) load8(kr[ks % KR], key + ks * 16 * sizeof(T));
        else load8(kr[ks % KR], key + (size_t)(min(ks * 16 + half * 8, d - 8) - half * 8) * sizeof(T));
    };

    float ep[RB][16];   // the previous layer's exponentials of this lane's keys
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int v = 0; v < 16; ++v) ep[rb][v] = 0.f;

    // ---- merge of the rows' partials, one step late: wave w takes RPM rows of a block from RPM * w on, lane (i, r) partial i
    // of row RPM * w + r; the P partials are joined by a butterfly.  f_prev took this lane's partial onto the merged
    // exponent of the previous layer, f_run the row's running record over the tiles before.
    float f_prev[RB], f_run[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) f_prev[rb] = f_run[rb] = 1.f;
    auto merge = [&](int l, int tile) __attribute__((always_inline)) {
        const bool foreign = l == 0 && l_first > 0;   // the layer's records belong to the chunk before
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int mrow = wave * RPM + lane % RPM, pw = lane / RPM >> 1, pl = (lane / RPM & 1) * 32 + mrow;
            const f32x4 v = part[rb][pw][pl];
            float M = partials_max<P>(v.x);
            const int rrow = rb * 32 + mrow;
            const size_t rec = rec0 + (size_t)l * R_WG + rrow;
            // (pointers that say which memory they lead to: chosen between at run time they would be generic, and a
            // generic access waits for everything in flight)
            f32x4 rr = {kMInit, 0.f, 0.f, 0.f};
            float ri = 0.f;
            if (tile > 0) {
                if (foreign) {
                    rr = *(lds_f32x4)(run0 + rrow);
                    if (IR) ri = *(lds_f32)(run0_ir + rrow);
                } else {
                    rr = *(global_f32x4)(uintptr_t)(p.state + rec);
                    if (IR) ri = *(global_f32)(uintptr_t)(p.state_ir + rec);
                }
                M = fmaxf(M, rr.x);
            }
            const float f = __builtin_amdgcn_exp2f(v.x - M), fr = __builtin_amdgcn_exp2f(rr.x - M);
            const float zs = partials_sum<P>(v.y * f), ns = partials_sum<P>(v.z * (f * f)), cc = partials_sum<P>(v.w * (f * f_prev[rb]));
            float zi = IR ? partials_sum<P>(part_ir[rb][pw][pl] * f) : 0.f;
            const f32x4 out = {M, fmaf(rr.y, fr, zs), fmaf(rr.z, fr * fr, ns), fmaf(rr.w, fr * f_run[rb], cc)};
            if (IR) zi = fmaf(ri, fr, zi);
            f_prev[rb] = f;
            f_run[rb] = fr;
            if (lane < RPM) {
                if (foreign) {
                    *(lds_f32x4)(run0 + rrow) = out;
                    if (IR) *(lds_f32)(run0_ir + rrow) = zi;
                } else {
                    *(global_f32x4)(uintptr_t)(p.state + rec) = out;
                    if (IR) *(global_f32)(uintptr_t)(p.state_ir + rec) = zi;
                }
            }
        }
    };

    if (d < KS * 16) {
        for (int i = tid; i < RB * PL * 32 * PITCH / 16; i += kThreads) reinterpret_cast<u32x4 *>(qlds)[i] = u32x4{0u, 0u, 0u, 0u};
        lds_barrier();
    }
    load_q(0);
    find_key(0);
    uintptr_t key = key_ptr(0);   // of the layer at hand, and of the next
#pragma unroll
    for (int ks = 0; ks < KR; ++ks) load_k(key, ks);
    store_q();

    const float c = p.c;
    int l = 0, tile = 0, l_before = 0, tile_before = 0;
    for (int step = 0; step < nsteps; ++step) {
        // the next step's layer and tile (the last step fetches its own once more)
        const bool has_next = step + 1 < nsteps;
        const int ln = !has_next ? l : (l + 1 == L ? 0 : l + 1), tn = has_next && l + 1 == L ? tile + 1 : tile;
        lds_barrier();   // query rows of this step are in LDS, and the records of the step before
        load_q(ln);
        if (step > 0) merge(l_before, tile_before);
        const int key0 = key_begin + tile * kTileKeys + wave * 32;
        if (tn != tile) find_key(tn);
        const uintptr_t key_now = key;
        key = key_ptr(ln);
        // the keys KR steps after step ks, this layer's or the next one's, take the registers' place
        auto load_after = [&](int ks) __attribute__((always_inline)) { load_k(ks + KR < KS ? key_now : key, (ks + KR) % KS); };

        // ---- logits
        f32x16 acc[RB], low;   // (with two row blocks their chains run side by side, and there are no registers for a second pair)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            low[v] = 0.f;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) acc[rb][v] = 0.f;
        }
        const unsigned char *const qr = qlds + l32 * PITCH + half * 16;
        u32x4 ko[2][PL];   // the keys' operands of MFMA step ks, and of ks + 1
#pragma unroll
        for (int e = 0; e < 4; ++e) kr[0].split_pair(e, ko[0]);
        load_after(0);
        asm volatile("" ::: "memory");   // (now: the compiler would put these loads, of no use before the next step, last)
        // Three row blocks: the query rows' operands of a step are read a plane at a time, for the next step, as soon as the plane's last product is on
        // its way, so that no product waits for LDS and no further registers are taken.  (One block or two, with a second workgroup on
        // the CU: all planes before the step; a plane at a time 63 tokens over 1150 keys took 188 us, 181 so.)
        constexpr bool AHEAD = RB == 3;
        u32x4 qo[RB][PL];
        auto read_plane = [&](int pl, int ks) __attribute__((always_inline)) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) qo[rb][pl] = *reinterpret_cast<const u32x4 *>(qr + (rb * PL + pl) * 32 * PITCH + ks * 32);
        };
        if constexpr (AHEAD) read_plane(1, 0), read_plane(2, 0), read_plane(0, 0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if constexpr (!AHEAD) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int pl = 0; pl < PL; ++pl)
                        qo[rb][pl] = *reinterpret_cast<const u32x4 *>(qr + (rb * PL + pl) * 32 * PITCH + ks * 32);
            }
            const auto &kc = ko[ks & 1];
            auto &kn = ko[(ks + 1) & 1];
            // The six products in turn -- the chains of two row blocks, or of the large and the small terms, side by
            // side -- and between them, pinned by the empty statements, the split of the next step's keys two elements
            // at a time: matrix and vector units then work at once.
            constexpr int kTerms[2][6][2] = {{{1, 1}, {0, 2}, {0, 0}, {2, 0}, {0, 1}, {1, 0}}, {{1, 1}, {0, 1}, {0, 2}, {2, 0}, {1, 0}, {0, 0}}};   // (planes of the keys, of the query rows)
#pragma unroll
            for (int t = 0; t < (PL == 3 ? 6 : 1); ++t) {
                if (ks + 1 < KS && t < 4) {
#pragma unroll
                    for (int e = (PL == 3 ? t : 0); e < (PL == 3 ? t + 1 : 4); ++e) {
                        kr[(ks + 1) % KR].split_pair(e, kn);
                        if constexpr (PL == 3) asm volatile("" : "+v"(kn[0][e]), "+v"(kn[1][e]), "+v"(kn[2][e]));
                    }
                    if (t == 3 || PL == 1) load_after(ks + 1);
                }
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const int ka = PL == 3 ? kTerms[AHEAD][t][0] : 0, qa = PL == 3 ? kTerms[AHEAD][t][1] : 0;
                    f32x16 &to = PL == 3 && RB == 1 && t != 2 ? low : acc[rb];
                    to = mfma8<T>(kc[ka], qo[rb][qa], to);
                    asm volatile("" : "+v"(to));
                }
                if (AHEAD && ks + 1 < KS) {
                    asm volatile("" ::: "memory");
                    if (t == 1) read_plane(1, ks + 1);
                    if (t == 2) read_plane(2, ks + 1);
                    if (t == 5) read_plane(0, ks + 1);
                }
            }
            asm volatile("" ::: "memory");
        }
        lds_barrier();   // every wave has read the query rows
        store_q();
        // ---- exponentials and sums of this lane's 16 keys: element v is key key0 + 8*(v/4) + 4*half + v%4
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            float x[16], m = kMInit;
            const int lim = min(key_end, row_end[rb]) - key0 - half * 4;
#pragma unroll
            for (int v = 0; v < 16; ++v) x[v] = PL == 3 && RB == 1 ? (acc[rb][v] + low[v]) * c : acc[rb][v] * c;
            if (__any(lim < 32)) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (8 * (v >> 2) + (v & 3) >= lim) x[v] = -INFINITY;
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) m = fmaxf(m, x[v]);
            f32x4 o = {m, 0.f, 0.f, 0.f};
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                x[v] = __builtin_amdgcn_exp2f(x[v] - m);
                o.y += x[v];
                o.z = fmaf(x[v], x[v], o.z);
                o.w = fmaf(x[v], ep[rb][v], o.w);
                ep[rb][v] = x[v];
            }
            part[rb][wave][lane] = o;
            if (IR) {
                float zi = 0.f;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int k0 = key0 + 8 * (v >> 2) + 4 * half + (v & 3);
                    if (k0 < p.ir_init_end || k0 >= p.ir_recent_begin) zi += x[v];
                }
                part_ir[rb][wave][lane] = zi;
            }
        }
        l_before = l;
        tile_before = tile;
        l = ln;
        tile = tn;
    }
    lds_barrier();
    merge(l_before, tile_before);
}

template <typename T, int KS, int RB>
hipError_t launch(const SimParams &p, int n_workgroups, hipStream_t st)
{
    if (p.want_ir)
        hipLaunchKernelGGL((sim_f32_kernel<T, KS, RB, true>), dim3(n_workgroups), dim3(RB == 3 ? 512 : 256), 0, st, p);
    else
        hipLaunchKernelGGL((sim_f32_kernel<T, KS, RB, false>), dim3(n_workgroups), dim3(RB == 3 ? 512 : 256), 0, st, p);
    return hipGetLastError();
}

template <int RB>
hipError_t launch_rows(const SimParams &p, int n_workgroups, hipStream_t st)
{
    if (p.d > 96) return launch<float, 8, RB>(p, n_workgroups, st);
    if (p.d > 64) return launch<float, 6, RB>(p, n_workgroups, st);
    if constexpr (RB < 3) return launch<float, 4, RB>(p, n_workgroups, st);
    return hipErrorInvalidValue;   // (three row blocks: heads above 64)
}

}  // namespace

hipError_t launch_sim_f32(const SimParams &p, int dtype, int n_workgroups, hipStream_t st)
{
    if (dtype == KRUL_BF16) return launch<uint16_t, 16, 1>(p, n_workgroups, st);
    if (dtype == KRUL_F16) return launch<_Float16, 16, 1>(p, n_workgroups, st);
    if (p.d > 192) return launch<float, 16, 1>(p, n_workgroups, st);
    if (p.d > 128) return launch<float, 12, 1>(p, n_workgroups, st);
    return p.lay.rb == 3 ? launch_rows<3>(p, n_workgroups, st) : p.lay.rb == 2 ? launch_rows<2>(p, n_workgroups, st) : launch_rows<1>(p, n_workgroups, st);
}

}  // namespace krul
