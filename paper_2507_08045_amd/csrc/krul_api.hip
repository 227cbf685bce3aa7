// C ABI of libkrul: argument checks, kernel choice, launches.  See include/krul.h for
// the contract of each entry point.
#include <math.h>

#include <mutex>

#include "krul_common.h"

namespace krul {
namespace {

constexpr size_t kAlign = 256;

size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

}  // namespace

int check_shape(const krul_shape_t *s)
{
    if (!s) return KRUL_EINVAL;
    if (s->dtype != KRUL_F32 && s->dtype != KRUL_BF16 && s->dtype != KRUL_F16) return KRUL_EDTYPE;
    if (s->batch <= 0 || s->n_layers < 2 || s->n_q_heads <= 0 || s->n_kv_heads <= 0 ||
        s->head_dim <= 0 || s->n_hist <= 0 || s->n_query <= 0)
        return KRUL_EINVAL;
    if (s->n_q_heads % s->n_kv_heads != 0) return KRUL_EINVAL;
    if (!(s->scale >= 0.f) || !isfinite(s->scale)) return KRUL_EINVAL;
    if (s->flags & ~(KRUL_FLAG_CAUSAL | KRUL_FLAG_GENERIC_KERNEL | KRUL_FLAG_SINGLE_SPLIT)) return KRUL_EINVAL;
    if ((s->flags & KRUL_FLAG_CAUSAL) && s->n_hist < s->n_query) return KRUL_EINVAL;
    if (s->head_dim % 8 != 0 || s->head_dim > 256) return KRUL_EUNSUPPORTED;
    if (s->n_layers > 2048) return KRUL_EUNSUPPORTED;
    return KRUL_OK;
}


namespace {

long long ceil_div(long long a, long long b) { return (a + b - 1) / b; }

// The tile shapes of the 16-bit matrix-core kernels and what a layer step of a workgroup takes.
struct MfmaForm {
    int variant, wr, wk, rb;
    int kt;               // keys per tile
    int resident;         // workgroups that share a CU
    // for calls of more than kShortCall us, see choose_long
    float step[3];        // us per layer step (one key tile, one layer) with every place taken, heads up to 64, 96, 128
    float stream[3];      // TB/s it draws from memory when the whole chip streams keys
    float in_phase;       // steps of two workgroups on a CU that started together take longer: they want the same units at once
    float start[3];       // us before a workgroup's first step and after its last
    // for shorter ones, see choose_short
    float short_step[2], short_stream[2];   // the same at head_dim 64, 128
    constexpr int rows() const { return wr * rb * 32; }
};
// Long calls: fitted (one MI355X) to 3870 times of 190 calls of one to 2048 tokens over 72 to 32254 keys, each under up to 40 plans, dense
// and with strides; the streams of the one-token shapes to calls over 4096 to 131072 keys, beyond the last-level cache.  Short calls: steps of
// few workgroups, keys in the last-level cache, and full rounds where they are slower; streams of one to eight query tokens over 4096 to
// 131072 keys, 16 tokens over 32768.
constexpr MfmaForm kWideForm = {kMfmaWide, 4, 2, 1, 256, 1, {2.55f, 2.75f, 3.2f}, {3.8f, 4.4f, 4.8f}, 1.f, {6.f, 4.f, 2.3f}, {3.1f, 3.4f}, {4.6f, 5.6f}};
constexpr MfmaForm kWideShortForm = {kMfmaWideShort, 4, 2, 1, 128, 1, {1.65f, 1.9f, 2.05f}, {3.5f, 3.8f, 4.4f}, 1.f, {2.3f, 2.3f, 2.3f}, {1.85f, 2.2f}, {4.6f, 5.6f}};
constexpr MfmaForm kWideDeepForm = {kMfmaWideDeep, 4, 2, 1, 512, 1, {}, {}, 1.f, {}, {}, {}};   // (taken by rule, see choose_mfma)
constexpr MfmaForm kMidForm = {kMfmaMid, 2, 4, 1, 512, 1, {2.55f, 3.f, 3.4f}, {5.4f, 5.5f, 5.8f}, 1.f, {6.f, 4.f, 2.3f}, {3.2f, 3.7f}, {4.6f, 5.6f}};
constexpr MfmaForm kMidShortForm = {kMfmaMidShort, 2, 2, 1, 128, 2, {1.22f, 1.5f, 1.93f}, {4.5f, 4.6f, 4.9f}, 1.15f, {2.3f, 2.3f, 2.3f}, {1.55f, 2.2f}, {4.1f, 4.9f}};
constexpr MfmaForm kSlimDeepForm = {kMfmaSlimDeep, 1, 4, 1, 512, 1, {2.f, 3.6f, 4.f}, {5.7f, 5.9f, 6.1f}, 1.f, {6.f, 6.f, 6.f}, {3.0f, 5.87f}, {5.6f, 5.75f}};
constexpr MfmaForm kSlimShortForm = {kMfmaSlimShort, 1, 4, 1, 256, 2, {1.4f, 1.8f, 1.8f}, {5.3f, 5.45f, 5.65f}, 1.1f, {2.3f, 2.3f, 2.3f}, {1.9f, 2.6f}, {5.05f, 5.25f}};
constexpr MfmaForm kBigForm = {kMfmaBig, 4, 2, 2, 256, 1, {6.f, 6.f, 6.f}, {4.3f, 4.3f, 4.3f}, 1.f, {2.3f, 2.3f, 2.3f}, {}, {}};
constexpr float kShortCall = 82.0f;       // us of the estimate of choose_long (some 8 less than the call takes)
constexpr float kWorkgroupStart = 5.0f;   // short calls: us before a workgroup's first step and after its last
constexpr int kCUs = 256;

// What a plan's records may take: 512 MB, or what one round of 128-row workgroups, or `rows` query rows with a single key
// split, leave if that is more.  (Without a limit a plan took gigabytes for a few per cent: 8 x 100 tokens over 16384
// keys of an 80-layer model 4.7 GB in 64 splits.)
long long record_limit(const krul_shape_t *s, long long rows)
{
    const long long most = rows > 128ll * kCUs ? rows : 128ll * kCUs, floor = 512ll << 20;
    return most * s->n_layers * 16 > floor ? most * s->n_layers * 16 : floor;
}
// us that records take to be written and read back (long calls have a fit of their own).  A few of them are still in the caches when they are read and cost
// next to nothing (117 tokens over 566 keys of 32 heads: 57 us with 10 MB, 66 with the plan that leaves 6), except beside a
// prefill chunk's uneven splits.
double record_time(long long bytes, bool chunk)
{
    const double free_bytes = chunk ? 0.0 : 32.0 * (1 << 20);
    return fmax(0.0, (double)bytes - free_bytes) / 5e6;
}

// What the scratch area of krul_pair_similarity_static leaves for records beside the head values (whole multiples of
// kAlign; not positive: nothing).
long long static_limit(const krul_shape_t *s)
{
    return (long long)KRUL_STATIC_SCRATCH_BYTES -
           2 * (long long)round_up((size_t)s->batch * (s->n_layers - 1) * s->n_q_heads * sizeof(float), kAlign);
}

struct MfmaChoice {
    const MfmaForm *form;
    long long n_split, tiles_per_split, n_chunks;
};

long long record_bytes(const krul_shape_t *s, const MfmaForm &f, long long n_split)
{
    const long long rows = (long long)s->n_q_heads / s->n_kv_heads * s->n_query;
    return (long long)s->batch * s->n_kv_heads * ceil_div(rows, f.rows()) * f.rows() * n_split * s->n_layers * 16;
}

// The calls that 256 x 256 tiles may take: the rows fill 256-row tiles well and there are two rounds of workgroups or more.  One factor
// of their cross terms is held in binary16 (cosines of 49 rows over 14839 keys off by 2e-6, 4e-8 in the other shapes), so
// that no others are given to them, also where they would be faster.
bool many_query(const krul_shape_t *s, bool want_ir, bool plain_keys)
{
    const long long Rk = (long long)s->n_q_heads / s->n_kv_heads * s->n_query, nrt = ceil_div(Rk, 256), tiles = ceil_div(s->n_hist, 256);
    return plain_keys && !want_ir && !(s->flags & KRUL_FLAG_CAUSAL) && s->head_dim == 128 && Rk > 64 && nrt * 256 * 7 <= Rk * 8 &&
           (long long)s->batch * s->n_kv_heads * nrt * tiles >= 512;
}

// Which tile shape, how many key splits and how many layer chunks.
//
// A workgroup walks (tiles of its key split) x (layers of its chunk) steps one after the other, and workgroups run in
// rounds of CUs * resident.  Candidates are compared by an estimate of their time: rounds of steps, or what the keys take from
// memory, whichever is more.
//   - key splits: for a number of rounds, or one tile each;
//   - layer chunks (only where every key split is one tile): the chain of layers is cut into pieces that run side
//     by side, each reading its first layer a second time.  What a problem too small to fill the chip needs (one
//     token over 4096 keys 104 -> 60 us, 20 over 300 80 -> 30 us), and what fills a last round that would be nearly
//     empty;
//   - tile shapes: for more than 64 rows the 64-row shapes where 128-row tiles would leave much of the last one empty, for
//     many query rows on dense keys 256 x 256 tiles (two 32-row blocks per wave, the previous layer's exponentials kept
//     as binary16 pairs: a third fewer bytes per logit and half the operands, but longer workgroups).
//
// There are two estimates.  choose_short's is simple -- rounds, always whole, of steps and a start -- and takes the number of splits for many
// query rows by rule; its plans of calls of up to 90 us are within 1 % (prefill chunks 12 %) of the best of up to 40.  Longer calls
// lose by it (10 % on average, up to 1.8 times the time: 1042 tokens over 19743 keys of 32/8 heads 14.9 ms in 272
// workgroups, one round and a sixteenth, 9.4 in 1768), and choose_long has the last word where its own choice is 7 % faster by
// its estimate.
//
// fallback: set to the plan for a workspace that does not hold the fastest one, see Plan.
MfmaChoice choose_short(const krul_shape_t *s, bool want_ir, bool plain_keys, bool in_static, MfmaChoice *fallback)
{
    const long long B = s->batch, L = s->n_layers, Hkv = s->n_kv_heads, S = s->n_hist, Tq = s->n_query;
    const long long Rk = s->n_q_heads / Hkv * Tq, d = s->head_dim;
    const long long limit = in_static ? static_limit(s) : record_limit(s, B * Hkv * ceil_div(Rk, 128) * 128);
    const bool single = (s->flags & KRUL_FLAG_SINGLE_SPLIT) != 0, causal = (s->flags & KRUL_FLAG_CAUSAL) != 0;
    const auto splits = [&](const MfmaForm &f, long long want, long long chunks) {
        const long long tiles = ceil_div(S, f.kt), n = want < 1 || single ? 1 : (want < tiles ? want : tiles);
        const long long tps = ceil_div(tiles, n);
        return MfmaChoice{&f, ceil_div(tiles, tps), tps, chunks};
    };

    if (Rk > 64) {
        // Many query rows on a large problem: 256 x 256 tiles (two 32-row blocks per wave, the previous layer's
        // exponentials kept as binary16 pairs) move a third fewer bytes per logit and read half the operands.
        const long long tiles = ceil_div(S, 256);
        const bool big = many_query(s, want_ir, plain_keys);
        // Here, and where the 128-row tile has as many row tiles, four key splits (or the round's worth, if that is
        // more) per row tile: the workgroups running side by side on an XCD then form patches of 8 row tiles x 4 key
        // splits (patch_rows()) and share both their query rows and their keys through the L2.
        const MfmaForm &f = big ? kBigForm : kWideForm;
        const long long nrt = ceil_div(Rk, f.rows()), want = ceil_div(kCUs, B * Hkv * nrt);
        // (Not a prefill chunk on keys in place whose records at one tile per split stay small: see below.)
        const bool chunk = causal && !plain_keys && Tq > f.rows() && B * Hkv * nrt * tiles * L * f.rows() * 16 <= limit;
        if (big || (nrt % 8 == 0 && tiles >= 16 && want <= 4 && !chunk))
            return *fallback = splits(f, want < 4 && tiles >= 16 && nrt % 8 == 0 ? 4 : want, 1);
    }

    struct Best {
        MfmaChoice c;
        double t;
        long long bytes;
    } best = {}, best_whole = {};
    const auto consider = [&](const MfmaForm &f, long long want, long long chunks) {
        const MfmaChoice c = splits(f, want, chunks);
        if (chunks > 1 && c.tiles_per_split > 1) return;
        const long long nrt = ceil_div(Rk, f.rows()), n_splits_all = B * Hkv * nrt * c.n_split;
        const double slots = (double)kCUs * f.resident, n_wg = (double)(n_splits_all * chunks);
        const double steps = (double)(c.tiles_per_split * (ceil_div(L - 1, chunks) + 1));
        const double layers_read = (double)(L - 1 + chunks);
        const long long record_bytes = n_splits_all * L * f.rows() * 16;
        double t_steps = ceil(n_wg / slots) * (steps * f.short_step[d > 64] + kWorkgroupStart);
        const bool chunk = causal && Tq > f.rows();
        if (chunk) {
            // The tiles right of a row tile's diagonal are not walked and splits without a tile left stop at once.  Row
            // tiles see S - Tq/2 + rows/2 keys on average.  Splits of one tile are alike and come in rounds; longer
            // ones differ, so the last of them run beside idle CUs for about half a split.  One tile per split
            // measured best or near it (32/8 heads of 128, against the plan without this: 651 tokens over 1623 keys 721
            // -> 564 us, 1888 over 2707 2450 -> 1890, 700 over 16000 5990 -> 4990; 512 over 3575, where two splits make
            // one even round, 777 against 799).
            const double tiles_seen = fmin((double)ceil_div(S, f.kt), ((double)S - 0.5 * (double)(Tq - f.rows())) / f.kt + 0.5);
            const double live = (double)(B * Hkv * nrt * chunks) * (c.n_split > 1 ? fmin((double)c.n_split, tiles_seen / (double)c.tiles_per_split + (c.tiles_per_split > 1 ? 0.5 : 0.0)) : 1.0);
            const double tile_steps = (double)(ceil_div(L - 1, chunks) + 1) * f.short_step[d > 64];
            if (live > slots && c.tiles_per_split > 1)
                t_steps = (double)(B * Hkv * nrt) * tiles_seen * tile_steps / slots + 0.5 * (double)c.tiles_per_split * tile_steps + kWorkgroupStart;
            else
                t_steps = ceil(live / slots) * ((double)c.tiles_per_split * tile_steps + kWorkgroupStart);
            // (the short forms over several tiles: 4 x 200 tokens over 300 keys of 32 heads 264 us, 229 in 256-key tiles)
            if (c.tiles_per_split > 1 && f.kt <= 128) t_steps *= 1.2;
            if (chunks > 1) t_steps *= 1.25;   // (600 tokens over 700 keys: 247 us in two chunks, 241 in one)
        }
        // (idle places draw no keys: the stream is up to 15 % slower.  For up to 32 rows, which do little else than wait for it, also
        // those of a last round -- one token over 6000 keys in three chunks of layers, 576 workgroups for 512 places, 104 us, in two
        // 85, 3 of 5535 keys and 80 layers 629 and 532; not for more, which hide it: 57 tokens over 276 keys 62 us, 70 so; nor for heads
        // up to 64 where it makes one chunk, whose workgroups do not fill the places once, look better than several: 13 tokens of
        // 1652 keys and 24 layers in one chunk 69.6 us, in two 61.3, 2 of 11145 keys 70.4 and 62.9.)
        const bool last_round = Rk <= 32 && !(d <= 64 && chunks > 1 && n_splits_all < (long long)slots);
        const double bytes = (double)(B * d * 2) * (double)(Hkv * S + s->n_q_heads * Tq) * layers_read;
        const auto take = [&](Best &b, double taken) {
            const double t_stream = bytes / (f.short_stream[d > 64] * 1e6 * (0.85 + 0.15 * taken)) + kWorkgroupStart;
            // (slim tiles have next to nothing to do but wait for keys; the others' steps hide most of the stream)
            const double t = fmax(t_steps, t_stream) + record_time(record_bytes, chunk) + (Rk > 32 ? 0.1 * fmin(t_steps, t_stream) : 0.0);
            // The fastest within the limit on records; where none is, the one with the fewest.
            if (!b.c.form || (record_bytes <= limit ? b.bytes > limit || t < b.t : b.bytes > limit && record_bytes < b.bytes)) b = {c, t, record_bytes};
        };
        take(best, last_round ? n_wg / slots / ceil(n_wg / slots) : fmin(1.0, n_wg / slots));
        if (Rk <= 32) take(best_whole, fmin(1.0, n_wg / slots));
    };
    const auto consider_form = [&](const MfmaForm &f) {
        const long long tiles = ceil_div(S, f.kt), nrt = ceil_div(Rk, f.rows()), units = B * Hkv * nrt;
        const long long slots = (long long)kCUs * f.resident;
        // Splits of several tiles for a round, or up to eight (seven rounds of 8 x 100 tokens over 16384 keys of an 80-layer model
        // come out even, one to three do not: 30.5 ms against 34.6; a prefill chunk's splits are uneven by themselves: up to
        // three) -- not where the stream of keys is the bound: a split of
        // several tiles parks its running records in memory between tiles, and that cost a quarter of the bandwidth
        // (a decode step over 131072 tokens: 57 % of 8 TB/s against 74 % with one tile per split) -- then one tile per
        // split and the layers in chunks.
        if (Rk > 64)
            for (int r = 1; r <= (causal && Tq > f.rows() ? 3 : 8) && slots * r / units < tiles; ++r) consider(f, slots * r / units, 1);
        const long long most = tiles < 1024 ? tiles : 1024;
        consider(f, most, 1);
        if (most < tiles || single || &f == &kSlimDeepForm) return;   // (the deep ring takes too long to fill for a piece of the chain)
        // (Few cuts, spread over their logarithm; those of 31 pairs that shorten the longest chunk.  A model's own -- ceil(pairs / k) for k = 1,
        // 2, ... -- were tried in their place: 0.91 to 1.17 times the speed over 30 calls of 24 to 80 layers, 0.99 on average.)
        static const int kChunks[] = {2, 3, 4, 5, 6, 8, 11, 16, 31};
        for (const int c : kChunks) {
            if (c > L - 1 || units * tiles * c > 8 * slots) break;
            consider(f, tiles, c);
        }
    };
    if (Rk <= 32) {
        consider_form(kSlimDeepForm);
        consider_form(kSlimShortForm);
    } else {
        if (Rk > 64) {
            consider_form(kWideForm);
            consider_form(kWideShortForm);
        }
        consider_form(kMidForm);
        consider_form(kMidShortForm);
    }
    *fallback = Rk <= 32 ? best_whole.c : best.c;
    return best.c;
}

// o: the plan of choose_short, which stays unless there is one that takes 7 % less.
MfmaChoice choose_long(const krul_shape_t *s, bool want_ir, bool plain_keys, const MfmaChoice &o)
{
    const long long B = s->batch, L = s->n_layers, Hkv = s->n_kv_heads, S = s->n_hist, Tq = s->n_query;
    const long long Rk = s->n_q_heads / Hkv * Tq, d = s->head_dim;
    const long long limit = record_limit(s, B * Hkv * ceil_div(Rk, 128) * 128);
    const bool single = (s->flags & KRUL_FLAG_SINGLE_SPLIT) != 0, causal = (s->flags & KRUL_FLAG_CAUSAL) != 0;
    const auto splits = [&](const MfmaForm &f, long long want, long long chunks) {
        const long long tiles = ceil_div(S, f.kt), n = want < 1 || single ? 1 : (want < tiles ? want : tiles);
        const long long tps = ceil_div(tiles, n);
        return MfmaChoice{&f, ceil_div(tiles, tps), tps, chunks};
    };

    MfmaChoice best = {nullptr, 0, 0, 0};
    double best_t = 0.0;
    long long best_bytes = 0;
    const int dc = d <= 64 ? 0 : d <= 96 ? 1 : 2;
    // us of a plan but for what they all have in common
    const auto time_of = [&](const MfmaForm &f, const MfmaChoice &c, long long records) {
        const long long nrt = ceil_div(Rk, f.rows());
        const double slots = (double)kCUs * f.resident, n = (double)(B * Hkv * nrt * c.n_split * c.n_chunks), rounds = ceil(n / slots);
        // (workgroups in patches share keys and query rows through the L2: four splits of eight row tiles 61.4 ms, one 68.4)
        const int patch = patch_rows((int)nrt, (int)c.n_split);
        const double shared = f.variant == kMfmaBig && patch == 8 ? 0.96 : f.variant == kMfmaWide && patch ? 0.98 : 1.0;
        const double walk = (double)(c.tiles_per_split * (ceil_div(L - 1, c.n_chunks) + 1)) * f.step[dc] * shared;   // one workgroup's
        const auto part = [](double taken) { return 0.8 + 0.2 * taken; };   // of a step's time with that share of the places taken
        double t;
        if (causal && Tq > f.rows()) {
            // A prefill chunk: the tiles right of a row tile's diagonal are not walked and splits without a tile left stop at
            // once.  Row tiles see S - Tq/2 + rows/2 keys on average.  Splits of one tile are alike; longer ones differ, and the last of
            // them run beside idle CUs for about half a split.  Workgroups that stop at once upset the hand-out of the
            // others: more than a round with them is hardly better than two rounds.
            const double seen = fmin((double)ceil_div(S, f.kt), ((double)S - 0.5 * (double)(Tq - f.rows())) / f.kt + 0.5);
            const double of_splits = fmin((double)c.n_split, seen / (double)c.tiles_per_split + (c.tiles_per_split > 1 ? 0.5 : 0.0));
            const double live = (double)(B * Hkv * nrt * c.n_chunks) * of_splits;
            const double full = c.tiles_per_split > 1 ? fmin(1.0, seen / ((double)c.tiles_per_split * of_splits)) : 1.0;   // of a live split's tiles
            if (live > slots) t = (1.05 * full * live / slots + 0.5) * walk;
            else if (n > slots && live > 0.5 * slots) t = 1.7 * walk;
            else t = walk * (live > kCUs ? f.in_phase : 1.0) * part(live / slots);
            t += f.start[dc];
        } else {
            const double full = floor(n / slots), last = n / slots - full;
            t = (full + (last > 0.0 ? part(last) : 0.0)) * walk * (n > kCUs ? 1.0 + (f.in_phase - 1.0) / rounds : 1.0) + rounds * f.start[dc];
        }
        // (keys that several row tiles read are not always found in the L2; idle places draw none)
        const double bytes = (double)(B * d * 2) * ((double)(Hkv * S) * (nrt > 1 ? 1.28 : 1.0) + (double)(s->n_q_heads * Tq)) * (double)(L - 1 + c.n_chunks);
        const double stream = bytes / (f.stream[dc] * 1e6 * (0.77 + 0.23 * n / slots / rounds)) + f.start[dc];
        return sqrt(sqrt(t * t * t * t + stream * stream * stream * stream)) + 0.34 * fmax(0.0, (double)records / 1e6 - 10.0);
    };
    const double to_beat = 0.93 * time_of(*o.form, o, record_bytes(s, *o.form, o.n_split));
    if (to_beat <= kShortCall) return o;   // (the candidates take the host 1 to 5 us)
    const auto consider = [&](const MfmaForm &f, long long want, long long chunks, bool over_limit = false) {
        const MfmaChoice c = splits(f, want, chunks);
        if (chunks > 1 && c.tiles_per_split > 1) return;
        const long long bytes = record_bytes(s, f, c.n_split);
        const double t = time_of(f, c, bytes);
        // The fastest within the limit on records; where none is, the one with the fewest.
        const long long over = over_limit ? 0 : bytes;
        if (!best.form || (over <= limit ? best_bytes > limit || t < best_t : best_bytes > limit && over < best_bytes)) {
            best = c;
            best_t = t;
            best_bytes = over;
        }
    };
    const auto consider_form = [&](const MfmaForm &f) {
        const long long tiles = ceil_div(S, f.kt), nrt = ceil_div(Rk, f.rows()), units = B * Hkv * nrt;
        const long long slots = (long long)kCUs * f.resident;
        // Splits of several tiles for one to eight rounds, or all of the keys -- not for up to 64 rows, where the stream of keys is
        // the bound: a split of several tiles parks its running records in memory between tiles, and that cost a quarter of
        // the bandwidth (a decode step over 131072 tokens: 57 % of 8 TB/s against 74 % with one tile per split) -- then one
        // tile per split and the layers in chunks.
        if (Rk > 64) {
            for (int r = 1; r <= 8 && slots * r / units < tiles; ++r) consider(f, slots * r / units, 1);
            // row tiles in patches of eight by four splits (their records are allowed beyond the limit, up to four times
            // the least)
            if (nrt % 8 == 0 && tiles >= 16) consider(f, 4, 1, &f == &kBigForm);
        }
        const long long most = tiles < 1024 ? tiles : 1024;
        consider(f, most, 1);
        // (the deep ring takes too long to fill for a piece of the chain; the many-query kernel takes the whole of it)
        if (most < tiles || single || &f == &kSlimDeepForm || &f == &kBigForm) return;
        // (Few cuts, spread over their logarithm; those of 31 pairs that shorten the longest chunk.  A model's own -- ceil(pairs / k) for k = 1,
        // 2, ... -- were tried in their place: 0.91 to 1.17 times the speed over 30 calls of 24 to 80 layers, 0.99 on average.)
        static const int kChunks[] = {2, 3, 4, 5, 6, 8, 11, 16, 31};
        for (const int c : kChunks) {
            if (c > L - 1 || units * tiles * c > 8 * slots) break;
            consider(f, tiles, c);
        }
    };
    if (Rk <= 32) {
        consider_form(kSlimDeepForm);
        consider_form(kSlimShortForm);
    } else {
        if (Rk > 64) {
            consider_form(kWideForm);
            consider_form(kWideShortForm);
            if (many_query(s, want_ir, plain_keys)) consider_form(kBigForm);
        }
        consider_form(kMidForm);
        consider_form(kMidShortForm);
    }
    return best_t > kShortCall && best_t < to_beat ? best : o;
}

// in_static: for krul_pair_similarity_static.  Its limit on records is the library's own area: the plan of the call with a
// workspace where that fits, and otherwise choose_short's within the limit.  (What that does not fit is refused: large calls
// with many query rows, which should bring a workspace.)
MfmaChoice choose_mfma(const krul_shape_t *s, bool want_ir, bool plain_keys, bool in_static, MfmaChoice *fallback)
{
    MfmaChoice c = choose_long(s, want_ir, plain_keys, choose_short(s, want_ir, plain_keys, false, fallback));
    // Heads up to 64, wide tiles, an even number of them in a split: half as many tiles of twice the keys.  What a layer step
    // costs beside its blocks -- merging, waiting -- is a third of it there (2 x 128 tokens over 16384 keys of 24 layers, 16/4
    // heads, 467 us in tiles of 256 keys, 426 so; 256 over 16384 with strides 470 and 448).  With two of 256 it depends: 64 over
    // 16384 124 and 115, but 166 over 4718 with the causal mask 134 and 141, 33 over 2382 of few layers 26 and 27.  The layer
    // test has no registers for it.
    if (c.form == &kWideForm && s->head_dim <= 64 && !want_ir && c.tiles_per_split % 2 == 0 && c.tiles_per_split >= 4)
        c = MfmaChoice{&kWideDeepForm, c.n_split, c.tiles_per_split / 2, 1};
    if (!in_static) return c;
    const auto fits = [&](const MfmaChoice &m) { return record_bytes(s, *m.form, m.n_split) <= static_limit(s); };
    const MfmaChoice o = choose_short(s, want_ir, plain_keys, true, fallback);
    return fits(o) && fits(c) ? c : o;
}

}  // namespace

int make_plan(const krul_shape_t *s, Plan *pl, bool want_ir, bool plain_keys, bool in_static, bool take_fallback)
{
    const int rc = check_shape(s);
    if (rc != KRUL_OK) return rc;
    const long long B = s->batch, L = s->n_layers, Hq = s->n_q_heads, Hkv = s->n_kv_heads;
    const long long S = s->n_hist, Tq = s->n_query, g = Hq / Hkv, Rk = g * Tq;
    if (Rk > INT32_MAX || B * Hq * Tq > INT32_MAX) return KRUL_EUNSUPPORTED;

    const float scale = s->scale > 0.f ? s->scale : 1.0f / sqrtf((float)s->head_dim);
    pl->c = scale * 1.4426950408889634f;
    StateLayout &y = pl->lay;
    y.n_layers = (int)L;
    y.rows_per_unit = (int)Rk;

    // 16-bit inputs with a head size up to 128 take the matrix cores (64 and 128 as they are, the sizes between
    // zero-padded to the next of the two inside LDS)
    const bool mfma = (s->dtype == KRUL_BF16 || s->dtype == KRUL_F16) && s->head_dim <= 128 &&
                      !(s->flags & KRUL_FLAG_GENERIC_KERNEL);
    bool generic = (s->flags & KRUL_FLAG_GENERIC_KERNEL) != 0;
    long long n_wg = 0, records = 0, fallback_records = 0;
    if (mfma) {
        MfmaChoice fallback;
        MfmaChoice ch = choose_mfma(s, want_ir, plain_keys, in_static, &fallback);
        if (take_fallback) ch = fallback;
        fallback_records = record_bytes(s, *fallback.form, fallback.n_split) / 16;
        const MfmaForm &f = *ch.form;
        y.variant = f.variant;
        y.wr = f.wr;
        y.wk = f.wk;
        y.rb = f.rb;
        y.n_row_tiles = (int)ceil_div(Rk, f.rows());
        y.n_split = y.partials = (int)ch.n_split;
        y.n_layer_chunks = (int)ch.n_chunks;
        pl->keys_per_split = (int)(ch.tiles_per_split * f.kt);
        const long long n_splits_all = B * Hkv * y.n_row_tiles * ch.n_split;
        n_wg = n_splits_all * ch.n_chunks;
        records = n_splits_all * L * f.rows();
    } else if (!generic) {
        // float32 inputs and larger heads: tiles of 32 or 64 rows x 128 keys, two workgroups a CU, or of 96 rows x 256 keys, one
        y.variant = kF32;
        y.wr = y.wk = y.rb = 1;
        const long long ks = ceil_div(s->head_dim, 16);
        const int rb_most = Rk > 32 && s->head_dim <= 128 ? 2 : 1;
        const long long limit = in_static ? static_limit(s) : record_limit(s, B * Hkv * ceil_div(Rk, 32 * rb_most) * 32 * rb_most);
        long long best_ns = 1, best_nl = 1, best_bytes = 0, others_bytes = 0;   // others_bytes: of the best plan without 96-row tiles
        double best_t = 0.0;
        // 96-row tiles, which split the keys once for 96 rows, stand in for 64-row ones only: a wave with one row block keeps the small terms of its products in a
        // sum of their own, one with two or three has no registers for it (modelled over 128 unit-normal elements: 6.8e-7, 1.5e-6 and 1.4e-6
        // root mean square of a logit).  For heads above 64 (below, within 5 % either way but for one call of 60), on memory that the others'
        // plan takes too.  Their step is entered longer than it was best fitted (7.0), so that a close call stays with the others: 24
        // tokens over 1021 keys 84 -> 68 us; 140 drawn calls that take them are 1.10 to 1.50 times as fast (65 to 96 rows most of them, 128 padded
        // ones in the others), 110 that do not would be 0.59 to 1.17 times as fast in them.  Short calls are not asked: the
        // candidates take the host 1 us, and such calls wait for it.
        for (int rb = 1; rb <= rb_most || (rb == 3 && y.rb == 2 && Rk > 64 && s->head_dim > 64 && best_t >= 40.0); ++rb) {
            const long long nrt = ceil_div(Rk, 32 * rb), units = B * Hkv * nrt, tiles = ceil_div(S, rb == 3 ? 256 : 128);
            const long long resident = rb == 3 ? 1 : 2;
            // us per step for one workgroup a CU and for two, measured at head_dim 128
            const double step1 = rb == 1 ? 2.2 : rb == 2 ? 3.2 : 7.8;
            const double step2 = rb == 3 ? 7.8 * (0.5 + 0.5 * (double)ks / 8.0) : (rb == 1 ? 2.9 : 4.4) * (0.3 + 0.7 * (double)ks / 8.0);
            const long long cap = rb == 3 ? others_bytes : INT64_MAX;
            const auto consider = [&](long long ns, long long nl) {
                const long long tps = ceil_div(tiles, ns);
                if ((s->flags & KRUL_FLAG_SINGLE_SPLIT) && ns > 1) return;
                const double n = (double)(units * ceil_div(tiles, tps) * nl), steps = (double)(tps * (ceil_div(L - 1, nl) + 1));
                const long long bytes = units * ceil_div(tiles, tps) * L * 32 * rb * 16;
                const double t = (n <= kCUs ? steps * fmin(step1, step2) + 4.0 : ceil(n / (double)(resident * kCUs)) * (steps * step2 + 4.0)) +
                                 record_time(bytes, false);
                if (bytes > cap) return;
                if (best_t == 0.0 || (bytes <= limit ? best_bytes > limit || t < best_t : best_bytes > limit && bytes < best_bytes)) {   // (as in choose_mfma)
                    y.rb = rb;
                    best_ns = ceil_div(tiles, tps);
                    best_nl = nl;
                    best_t = t;
                    best_bytes = bytes;
                }
            };
            for (long long nl = 1; nl <= L - 1 && nl <= 31; ++nl) {   // (more, with 80 layers: 5 tokens over 300 keys 48.0 -> 49.5 us, one over 1000 78.5 -> 79.4)
                for (int r = 1; r <= 3; ++r) {   // a round of workgroups, two or three; one tile per split
                    const long long ns = resident * kCUs * r / (units * nl);
                    if (ns >= 1 && ns < tiles) consider(ns, nl);
                }
                consider(1, nl);
                if (tiles <= 1024) consider(tiles, nl);
                if (units * nl >= 6 * kCUs) break;
            }
            if (rb < 3) others_bytes = best_bytes;
        }
        const long long units = B * Hkv * ceil_div(Rk, 32 * y.rb);
        y.n_row_tiles = (int)ceil_div(Rk, 32 * y.rb);
        y.n_split = y.partials = (int)best_ns;
        y.n_layer_chunks = (int)best_nl;
        fallback_records = others_bytes / 16;
        const long long kt = y.rb == 3 ? 256 : 128;
        pl->keys_per_split = (int)(ceil_div(ceil_div(S, kt), best_ns) * kt);
        n_wg = units * best_ns;
        records = n_wg * L * 32 * y.rb;
        n_wg *= best_nl;
        // The portable kernel keeps records of the rows there are, without the padding to 32: what fits the static area with
        // it alone (one token of many conversations with a kv head per query head) runs, slower.
        generic = in_static && best_bytes > limit;
    }
    if (generic) {
        fallback_records = 0;
        y.variant = kGeneric;
        y.wr = y.wk = y.rb = 1;
        y.n_row_tiles = 1;
        y.n_layer_chunks = 1;
        const long long rows = B * Hq * Tq;
        long long want = (2048 + rows - 1) / rows;
        const long long max_split = (S + 255) / 256;
        long long nsplit = want < max_split ? want : max_split;
        if (nsplit < 1 || (s->flags & KRUL_FLAG_SINGLE_SPLIT)) nsplit = 1;
        long long kps = ((S + nsplit - 1) / nsplit + 63) / 64 * 64;
        nsplit = (S + kps - 1) / kps;
        y.n_split = (int)nsplit;
        y.partials = (int)nsplit;
        pl->keys_per_split = (int)kps;
        n_wg = rows * nsplit;
        records = n_wg * L;
    }
    if (n_wg > INT32_MAX) return KRUL_EUNSUPPORTED;
    pl->n_workgroups = (int)n_wg;
    const size_t head_bytes = round_up((size_t)(B * (L - 1) * Hq) * sizeof(float), kAlign);
    const auto layout = [&](size_t n) {   // of n records
        pl->head_cos_off = pl->state_bytes = round_up(n * sizeof(float4), kAlign);
        pl->head_dist_off = pl->head_cos_off + head_bytes;
        pl->total_bytes = pl->head_dist_off + head_bytes;
        pl->state_ir_off = pl->head_ir_off = 0;
        if (want_ir) {
            pl->state_ir_off = pl->total_bytes;
            pl->head_ir_off = pl->state_ir_off + round_up(n * sizeof(float), kAlign);
            pl->total_bytes = pl->head_ir_off + round_up((size_t)(B * L * Hq) * sizeof(float), kAlign);
        }
        return pl->total_bytes;
    };
    pl->fallback_bytes = layout((size_t)(fallback_records ? fallback_records : records));
    layout((size_t)records);
    return KRUL_OK;
}

int resolve_keys(const krul_shape_t *s, bool mfma, bool dense_2gib, const void *k, const krul_k_layout_t *kl,
                 const krul_k_pages_t *kp, KeyAddr *out)
{
    if ((k != nullptr) + (kl != nullptr) + (kp != nullptr) != 1) return KRUL_EINVAL;
    const long long d = s->head_dim, S = s->n_hist;
    KeyAddr a = {};
    if (k) {
        if ((uintptr_t)k & 15) return KRUL_EINVAL;
        if (mfma && dense_2gib && S * d * 2 >= (1ll << 31)) return KRUL_EUNSUPPORTED;
        a.k = k;
        a.stride_l = (long long)s->n_kv_heads * S * d;
        a.stride_b = (long long)s->n_layers * s->n_kv_heads * S * d;
        a.stride_h = S * d;
        a.stride_s = d;
    } else if (kl) {
        if (!kl->k_layers || ((uintptr_t)kl->k_layers & 7)) return KRUL_EINVAL;
        const long long sb = s->batch > 1 ? kl->k_stride_b : 8;   // (not used for one conversation)
        if (sb <= 0 || kl->k_stride_h <= 0 || kl->k_stride_s < d || ((sb | kl->k_stride_h | kl->k_stride_s) & 7))
            return KRUL_EINVAL;
        // the matrix-core kernels' 32-bit offsets and ranges need a layer's keys of one head to span
        // less than 2 GiB
        if (mfma && (kl->k_stride_s >= (1ll << 23) ||
                     (dense_2gib && kl->k_stride_s * 2 * S >= (1ll << 31))))
            return KRUL_EUNSUPPORTED;
        a.k_tab = kl->k_layers;
        a.stride_b = s->batch > 1 ? kl->k_stride_b : 0;
        a.stride_h = kl->k_stride_h;
        a.stride_s = kl->k_stride_s;
    } else {
        if (!kp->k_layers || !kp->block_table || ((uintptr_t)kp->k_layers & 7) || ((uintptr_t)kp->block_table & 3))
            return KRUL_EINVAL;
        const int bs = kp->block_size;
        if (bs < 8 || (bs & (bs - 1)) || kp->max_blocks < (S + bs - 1) / bs || kp->k_stride_block <= 0 ||
            kp->k_stride_h <= 0 || kp->k_stride_s < d || ((kp->k_stride_block | kp->k_stride_h | kp->k_stride_s) & 7))
            return KRUL_EINVAL;
        // (32-bit byte offsets over the keys one copy instruction moves)
        if (mfma && kp->k_stride_s >= (1ll << 27)) return KRUL_EUNSUPPORTED;
        a.k_tab = kp->k_layers;
        a.block_table = kp->block_table;
        a.max_blocks = kp->max_blocks;
        for (a.page_shift = 3; (1 << a.page_shift) < bs; ++a.page_shift) {}
        a.stride_page = kp->k_stride_block;
        a.stride_h = kp->k_stride_h;
        a.stride_s = kp->k_stride_s;
    }
    *out = a;
    return KRUL_OK;
}

}  // namespace krul

using namespace krul;

namespace {
__global__ __launch_bounds__(256) void calibration_copy_kernel(const uint4 *__restrict__ src,
                                                               uint4 *__restrict__ dst, size_t n)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}
}  // namespace

namespace {
// Selection asked for in the same call (krul_pair_similarity_select).
struct SelectArgs {
    const uint8_t *eligible;
    int n_select;
    int32_t *out_pairs, *out_count;
};

// The one implementation behind the similarity entry points.  ir: also run the Initial-Recent layer
// test (gamma, ir_mass, eligible as for krul_pair_similarity_ir).
// accumulate: head_score / pair_dist are the caller's running sums [B][L-1][Hq] (see
// krul_pair_similarity_accumulate) and pair_score is unused.
int run_similarity(const krul_shape_t *shape, const void *q, const void *k, float *pair_score,
                   float *head_score, float *pair_dist, bool ir, float gamma, float *ir_mass,
                   uint8_t *eligible, void *workspace, size_t workspace_bytes, void *stream,
                   void *event_begin, void *event_end, bool accumulate = false,
                   const krul_k_layout_t *kl = nullptr, const krul_k_pages_t *kp = nullptr,
                   const SelectArgs *sel = nullptr, bool in_static = false)
{
    Plan pl;
    const int rc = make_plan(shape, &pl, ir, k != nullptr && !kl && !kp, in_static);
    if (rc != KRUL_OK) return rc;
    if (!q || (accumulate ? !head_score : !pair_score)) return KRUL_EINVAL;
    if (ir && (shape->flags & KRUL_FLAG_CAUSAL)) return KRUL_EUNSUPPORTED;
    if ((uintptr_t)q & 15) return KRUL_EINVAL;
    if (((uintptr_t)pair_score | (uintptr_t)head_score | (uintptr_t)pair_dist | (uintptr_t)ir_mass) & 3)
        return KRUL_EINVAL;
    if (ir && (!(gamma >= 0.f) || !isfinite(gamma) || (!ir_mass && !eligible))) return KRUL_EINVAL;
    if (!workspace || ((uintptr_t)workspace & (kAlign - 1))) return KRUL_EWORKSPACE;
    if (workspace_bytes < pl.total_bytes) {
        if (in_static || workspace_bytes < pl.fallback_bytes ||
            make_plan(shape, &pl, ir, k != nullptr && !kl && !kp, false, true) != KRUL_OK)
            return KRUL_EWORKSPACE;
    }

    hipStream_t st = static_cast<hipStream_t>(stream);
    unsigned char *ws = static_cast<unsigned char *>(workspace);
    SimParams p;
    p.q = q;
    p.state = reinterpret_cast<float4 *>(ws);
    p.B = shape->batch;
    p.L = shape->n_layers;
    p.Hq = shape->n_q_heads;
    p.Hkv = shape->n_kv_heads;
    p.g = p.Hq / p.Hkv;
    p.d = shape->head_dim;
    p.S = shape->n_hist;
    p.Tq = shape->n_query;
    p.keys_per_split = pl.keys_per_split;
    p.c = pl.c;
    p.want_dist = pair_dist != nullptr || ir;   // the test needs Z as well
    p.want_ir = ir;
    p.causal = (shape->flags & KRUL_FLAG_CAUSAL) != 0;
    p.f16 = shape->dtype == KRUL_F16;
    // T_initial = T[:10% s], T_recent = T[90% s:] (Sec. 4.2): keys [0, floor(0.1 S)) and [floor(0.9 S), S)
    p.ir_init_end = (int)floor(0.1 * (double)p.S);
    p.ir_recent_begin = (int)floor(0.9 * (double)p.S);
    p.state_ir = reinterpret_cast<float *>(ws + pl.state_ir_off);
    p.lay = pl.lay;
    {
        KeyAddr ka;
        const int krc = resolve_keys(shape, pl.lay.variant != kGeneric && pl.lay.variant != kF32, true, k, kl, kp, &ka);
        if (krc != KRUL_OK) return krc;
        p.k = ka.k;
        p.k_tab = ka.k_tab;
        p.k_stride_l = ka.stride_l;
        p.k_stride_b = ka.stride_b;
        p.k_stride_h = ka.stride_h;
        p.k_stride_s = ka.stride_s;
        p.block_table = ka.block_table;
        p.page_shift = ka.page_shift;
        p.max_blocks = ka.max_blocks;
        p.k_stride_page = ka.stride_page;
    }

    if (event_begin && hipEventRecord(static_cast<hipEvent_t>(event_begin), st) != hipSuccess)
        return KRUL_ELAUNCH;
    hipError_t e = pl.lay.variant == kGeneric ? launch_sim_generic(p, shape->dtype, pl.n_workgroups, st)
                   : pl.lay.variant == kF32   ? launch_sim_f32(p, shape->dtype, pl.n_workgroups, st)
                                              : launch_sim_mfma(p, pl.n_workgroups, st);
    if (e != hipSuccess) return KRUL_ELAUNCH;
    if (event_end && hipEventRecord(static_cast<hipEvent_t>(event_end), st) != hipSuccess)
        return KRUL_ELAUNCH;
    float *head_cos = head_score ? head_score : reinterpret_cast<float *>(ws + pl.head_cos_off);
    float *head_dist = accumulate ? pair_dist : reinterpret_cast<float *>(ws + pl.head_dist_off);
    if (sel && pairs_select_fits(p.L, p.Hq)) {   // head scores, pairs and selection in one small launch or two
        const PairsSelectArgs a = {head_cos, pair_dist ? head_dist : nullptr, pair_score, pair_dist, sel->eligible,
                                   p.B, p.L, p.Hq, sel->n_select, sel->out_pairs, sel->out_count};
        e = launch_finalize_select(pl.lay, p.state, p.Hkv, p.Tq, head_score, head_cos, head_dist, a, st);
        return e == hipSuccess ? KRUL_OK : KRUL_ELAUNCH;
    }
    const IrArgs ir_args = {p.state_ir, reinterpret_cast<float *>(ws + pl.head_ir_off), gamma, ir_mass, eligible};
    e = launch_finalize(pl.lay, p.state, p.B, p.L, p.Hq, p.Hkv, p.Tq, head_cos, head_dist,
                        pair_score, pair_dist, accumulate, ir ? &ir_args : nullptr, st);
    if (e != hipSuccess) return KRUL_ELAUNCH;
    if (sel) {
        e = launch_select(pair_score, sel->eligible, p.B, p.L, sel->n_select, sel->out_pairs, sel->out_count, st);
        if (e != hipSuccess) return KRUL_ELAUNCH;
    }
    return KRUL_OK;
}
}  // namespace

extern "C" {

int krul_calibration_copy(const void *src, void *dst, size_t bytes, void *stream)
{
    if (!src || !dst || bytes == 0 || (bytes & 15) || (((uintptr_t)src | (uintptr_t)dst) & 15))
        return KRUL_EINVAL;
    hipLaunchKernelGGL(calibration_copy_kernel, dim3(256 * 8), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<const uint4 *>(src), static_cast<uint4 *>(dst), bytes / 16);
    return hipGetLastError() == hipSuccess ? KRUL_OK : KRUL_ELAUNCH;
}

int krul_pair_similarity_plan_of(const krul_shape_t *shape, int32_t in_static, krul_plan_t *plan)
{
    if (!plan) return KRUL_EINVAL;
    Plan pl;
    const int rc = make_plan(shape, &pl, false, true, in_static != 0);
    if (rc != KRUL_OK) return rc;
    if (in_static && pl.total_bytes > (size_t)KRUL_STATIC_SCRATCH_BYTES) return KRUL_ESCRATCH;
    const StateLayout &y = pl.lay;
    *plan = krul_plan_t{y.variant == kF32 ? 0 : y.variant, y.variant == kGeneric ? 1 : y.wr * y.rb * 32, pl.keys_per_split, y.n_split, y.n_layer_chunks,
                        pl.n_workgroups, 3};
    if (pairs_select_fits(shape->n_layers, shape->n_q_heads))
        plan->select_kernels = select_in_one_launch(y, shape->batch, shape->n_layers, shape->n_q_heads, shape->n_kv_heads, shape->n_query) ? 1 : 2;
    return KRUL_OK;
}

int krul_pair_similarity_plan(const krul_shape_t *shape, int32_t *n_workgroups, int32_t *n_key_splits)
{
    krul_plan_t pl;
    const int rc = krul_pair_similarity_plan_of(shape, 0, &pl);
    if (rc != KRUL_OK) return rc;
    if (n_workgroups) *n_workgroups = pl.n_workgroups;
    if (n_key_splits) *n_key_splits = pl.n_key_splits;
    return pl.form;
}

size_t krul_pair_similarity_workspace(const krul_shape_t *shape)
{
    // enough for the call on dense keys and for the calls on keys read in place (their plans may differ for more than 64 rows),
    // each with its fallback
    Plan pl;
    if (make_plan(shape, &pl) != KRUL_OK) return 0;
    size_t need = pl.total_bytes > pl.fallback_bytes ? pl.total_bytes : pl.fallback_bytes;
    if (pl.lay.variant == kGeneric || pl.lay.variant == kF32 || pl.lay.rows_per_unit <= 64) return need;
    if (make_plan(shape, &pl, false, true) != KRUL_OK) return 0;
    if (need < pl.total_bytes) need = pl.total_bytes;
    return need > pl.fallback_bytes ? need : pl.fallback_bytes;
}

int krul_pair_similarity(const krul_shape_t *shape, const void *q, const void *k,
                         float *pair_score, float *head_score, float *pair_dist,
                         void *workspace, size_t workspace_bytes, void *stream)
{
    return krul_pair_similarity_timed(shape, q, k, pair_score, head_score, pair_dist, workspace,
                                      workspace_bytes, stream, nullptr, nullptr);
}

int krul_pair_similarity_timed(const krul_shape_t *shape, const void *q, const void *k,
                               float *pair_score, float *head_score, float *pair_dist,
                               void *workspace, size_t workspace_bytes, void *stream,
                               void *event_begin, void *event_end)
{
    return run_similarity(shape, q, k, pair_score, head_score, pair_dist, false, 0.f, nullptr, nullptr,
                          workspace, workspace_bytes, stream, event_begin, event_end);
}

}  // extern "C"

namespace {
// The scratch area of krul_pair_similarity_static: device memory the code object brings along, one copy
// per GPU.  In host code the array's name only stands for the symbol; its device address is asked for
// once per GPU (that GPU current) and kept.
static __device__ __align__(256) unsigned char scratch[KRUL_STATIC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
void *scratch_ptr[kMaxDevices];   // by device ordinal; null until the first call on that device

int static_scratch(void **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return KRUL_ELAUNCH;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return KRUL_ELAUNCH;
        scratch_ptr[dev] = ptr;
    }
    *out = scratch_ptr[dev];
    return KRUL_OK;
}
}  // namespace

extern "C" {

int krul_pair_similarity_static(const krul_shape_t *shape, const void *q, const void *k,
                                float *pair_score, float *head_score, float *pair_dist, void *stream)
{
    Plan pl;
    const int rc = make_plan(shape, &pl, false, true, true);
    if (rc != KRUL_OK) return rc;
    if (pl.total_bytes > (size_t)KRUL_STATIC_SCRATCH_BYTES) return KRUL_ESCRATCH;
    void *ptr = nullptr;
    const int src = static_scratch(&ptr);
    if (src != KRUL_OK) return src;
    // Nothing in the area has to start at zero: every record the finalize kernels read is written by the
    // similarity kernel of the same call first.
    return run_similarity(shape, q, k, pair_score, head_score, pair_dist, false, 0.f, nullptr, nullptr,
                          ptr, (size_t)KRUL_STATIC_SCRATCH_BYTES, stream, nullptr, nullptr, false, nullptr, nullptr, nullptr, true);
}

int krul_pair_similarity_strided(const krul_shape_t *shape, const void *q, const krul_k_layout_t *k_layout,
                                 float *pair_score, float *head_score, float *pair_dist,
                                 void *workspace, size_t workspace_bytes, void *stream)
{
    if (!k_layout) return KRUL_EINVAL;
    return run_similarity(shape, q, nullptr, pair_score, head_score, pair_dist, false, 0.f, nullptr, nullptr,
                          workspace, workspace_bytes, stream, nullptr, nullptr, false, k_layout);
}

namespace {
// exactly one source of keys
bool one_source(const krul_keys_t *keys)
{
    return keys && (keys->dense != nullptr) + (keys->strided != nullptr) + (keys->paged != nullptr) == 1;
}
}  // namespace

int krul_all_pairs_similarity_in_place(const krul_shape_t *shape, const void *q, const krul_keys_t *keys,
                                       float *pair_score_all, float *pair_dist_all, float *head_score_all,
                                       void *workspace, size_t workspace_bytes, void *stream)
{
    if (!one_source(keys)) return KRUL_EINVAL;
    return run_all_pairs(shape, q, keys->dense, keys->strided, keys->paged, pair_score_all, pair_dist_all,
                         head_score_all, workspace, workspace_bytes, static_cast<hipStream_t>(stream));
}

size_t krul_all_pairs_workspace(const krul_shape_t *shape, size_t max_bytes)
{
    return all_pairs_workspace(shape, max_bytes);
}

int krul_all_pairs_similarity(const krul_shape_t *shape, const void *q, const void *k,
                              float *pair_score_all, float *pair_dist_all, float *head_score_all,
                              void *workspace, size_t workspace_bytes, void *stream)
{
    return run_all_pairs(shape, q, k, nullptr, nullptr, pair_score_all, pair_dist_all, head_score_all, workspace,
                         workspace_bytes, static_cast<hipStream_t>(stream));
}

int krul_select_pairs_all(const float *score, int32_t closer_is_smaller, const uint8_t *eligible,
                          int32_t batch, int32_t n_layers, int32_t n_select,
                          int32_t *out_pairs, int32_t *out_count, void *stream)
{
    if (!score || !out_count || batch <= 0 || n_layers < 2 || n_select < 0 || n_select > n_layers / 2 ||
        (n_select > 0 && !out_pairs))
        return KRUL_EINVAL;
    if (((uintptr_t)score | (uintptr_t)out_pairs | (uintptr_t)out_count) & 3) return KRUL_EINVAL;
    if (n_layers > 1024) return KRUL_EUNSUPPORTED;   // (n_select rounds over n_layers^2 entries)
    const hipError_t e = launch_select_all(score, closer_is_smaller, eligible, batch, n_layers, n_select, out_pairs,
                                           out_count, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? KRUL_OK : KRUL_ELAUNCH;
}

int krul_pair_similarity_select(const krul_shape_t *shape, const void *q, const void *k,
                                const uint8_t *eligible, int32_t n_select,
                                float *pair_score, float *head_score, float *pair_dist,
                                int32_t *out_pairs, int32_t *out_count,
                                void *workspace, size_t workspace_bytes, void *stream,
                                void *event_begin, void *event_end)
{
    if (!shape || !out_count || n_select < 0 || n_select > shape->n_layers / 2 || (n_select > 0 && !out_pairs))
        return KRUL_EINVAL;
    if (((uintptr_t)out_pairs | (uintptr_t)out_count) & 3) return KRUL_EINVAL;
    const SelectArgs sel = {eligible, n_select, out_pairs, out_count};
    return run_similarity(shape, q, k, pair_score, head_score, pair_dist, false, 0.f, nullptr, nullptr,
                          workspace, workspace_bytes, stream, event_begin, event_end, false, nullptr, nullptr, &sel);
}

int krul_pair_similarity_paged(const krul_shape_t *shape, const void *q, const krul_k_pages_t *k_pages,
                               float *pair_score, float *head_score, float *pair_dist,
                               void *workspace, size_t workspace_bytes, void *stream)
{
    if (!k_pages) return KRUL_EINVAL;
    return run_similarity(shape, q, nullptr, pair_score, head_score, pair_dist, false, 0.f, nullptr, nullptr,
                          workspace, workspace_bytes, stream, nullptr, nullptr, false, nullptr, k_pages);
}

int krul_pair_similarity_accumulate(const krul_shape_t *shape, const void *q, const void *k,
                                    float *head_sum, float *head_dist_sum,
                                    void *workspace, size_t workspace_bytes, void *stream)
{
    return run_similarity(shape, q, k, nullptr, head_sum, head_dist_sum, false, 0.f, nullptr, nullptr,
                          workspace, workspace_bytes, stream, nullptr, nullptr, true);
}

int krul_pair_similarity_accumulate_in_place(const krul_shape_t *shape, const void *q, const krul_keys_t *keys,
                                             float *head_sum, float *head_dist_sum,
                                             void *workspace, size_t workspace_bytes, void *stream)
{
    if (!one_source(keys)) return KRUL_EINVAL;
    return run_similarity(shape, q, keys->dense, nullptr, head_sum, head_dist_sum, false, 0.f, nullptr, nullptr,
                          workspace, workspace_bytes, stream, nullptr, nullptr, true, keys->strided, keys->paged);
}

int krul_pair_similarity_ir_in_place(const krul_shape_t *shape, const void *q, const krul_keys_t *keys, float gamma,
                                     float *pair_score, float *head_score, float *pair_dist,
                                     float *ir_mass, uint8_t *eligible,
                                     void *workspace, size_t workspace_bytes, void *stream)
{
    if (!one_source(keys)) return KRUL_EINVAL;
    return run_similarity(shape, q, keys->dense, pair_score, head_score, pair_dist, true, gamma, ir_mass, eligible,
                          workspace, workspace_bytes, stream, nullptr, nullptr, false, keys->strided, keys->paged);
}

int krul_pair_scores_from_sums(const float *head_sum, const float *head_dist_sum,
                               int32_t batch, int32_t n_layers, int32_t n_q_heads, float n_tokens,
                               float *pair_score, float *head_score, float *pair_dist, void *stream)
{
    if (!head_sum || !pair_score || batch <= 0 || n_layers < 2 || n_q_heads <= 0 || !(n_tokens > 0.f) ||
        !isfinite(n_tokens) || (pair_dist && !head_dist_sum))
        return KRUL_EINVAL;
    if (((uintptr_t)head_sum | (uintptr_t)head_dist_sum | (uintptr_t)pair_score | (uintptr_t)head_score |
         (uintptr_t)pair_dist) & 3)
        return KRUL_EINVAL;
    const hipError_t e = launch_scores_from_sums(head_sum, head_dist_sum, batch * (n_layers - 1), n_q_heads,
                                                 1.0f / n_tokens, pair_score, head_score, pair_dist,
                                                 static_cast<hipStream_t>(stream));
    return e == hipSuccess ? KRUL_OK : KRUL_ELAUNCH;
}

size_t krul_pair_similarity_ir_workspace(const krul_shape_t *shape)
{
    Plan pl;
    if (make_plan(shape, &pl, true) != KRUL_OK) return 0;
    return pl.total_bytes > pl.fallback_bytes ? pl.total_bytes : pl.fallback_bytes;
}

int krul_pair_similarity_ir(const krul_shape_t *shape, const void *q, const void *k, float gamma,
                            float *pair_score, float *head_score, float *pair_dist,
                            float *ir_mass, uint8_t *eligible,
                            void *workspace, size_t workspace_bytes, void *stream)
{
    return run_similarity(shape, q, k, pair_score, head_score, pair_dist, true, gamma, ir_mass, eligible,
                          workspace, workspace_bytes, stream, nullptr, nullptr);
}

int krul_select_pairs(const float *pair_score, const uint8_t *eligible,
                      int32_t batch, int32_t n_layers, int32_t n_select,
                      int32_t *out_pairs, int32_t *out_count, void *stream)
{
    if (!pair_score || !out_count || batch <= 0 || n_layers < 2 || n_select < 0 ||
        n_select > n_layers / 2 || (n_select > 0 && !out_pairs))
        return KRUL_EINVAL;
    if (((uintptr_t)pair_score | (uintptr_t)out_pairs | (uintptr_t)out_count) & 3) return KRUL_EINVAL;
    if (n_layers > 4096) return KRUL_EUNSUPPORTED;
    const hipError_t e = launch_select(pair_score, eligible, batch, n_layers, n_select, out_pairs,
                                       out_count, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? KRUL_OK : KRUL_ELAUNCH;
}

int32_t krul_n_select_from_ratio(int32_t n_layers, float r_l)
{
    if (n_layers < 2 || !(r_l > 0.f)) return 0;
    const double want = ceil((double)n_layers * (double)r_l / 2.0 - 1e-9);
    const int32_t cap = n_layers / 2;
    return want > cap ? cap : (int32_t)want;
}

const char *krul_strerror(int status)
{
    switch (status) {
    case KRUL_OK: return "ok";
    case KRUL_EINVAL: return "invalid argument";
    case KRUL_EDTYPE: return "unknown dtype";
    case KRUL_EWORKSPACE: return "workspace missing, misaligned or too small";
    case KRUL_ELAUNCH: return "kernel launch failed";
    case KRUL_EUNSUPPORTED: return "no kernel for this shape";
    case KRUL_ESCRATCH: return "the problem needs more scratch memory than the library's built-in area holds";
    default: return "unknown status";
    }
}

}  // extern "C"
