// C-ABI entry points of libvispec_verify: host-side argument checks, launch planning and
// kernel enqueues. Nothing here allocates device memory or synchronises.
#include <math.h>
#include <string.h>

#include <atomic>

#include "vs_internal.h"

namespace {

using namespace vs;

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
inline bool is_pow2(int32_t x) { return x > 0 && (x & (x - 1)) == 0; }
inline bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

} // namespace

namespace vs {
// Is the current device one this library's kernels were written for? Asked once per device
// and remembered; called after the argument checks and before the first enqueue.
int32_t check_device() {
    constexpr int kMaxDevices = 64;
    static std::atomic<int> known[kMaxDevices]; // 0 = not asked yet, 1 = gfx950, -1 = something else
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) {
        (void)hipGetLastError();
        return VS_ERR_NO_DEVICE;
    }
    if (dev < kMaxDevices) {
        const int k = known[dev].load(std::memory_order_relaxed);
        if (k != 0) return k > 0 ? VS_OK : VS_ERR_NO_DEVICE;
    }
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) {
        (void)hipGetLastError();
        return VS_ERR_NO_DEVICE;
    }
    const bool ok = strncmp(prop.gcnArchName, "gfx950", 6) == 0;
    if (dev < kMaxDevices) known[dev].store(ok ? 1 : -1, std::memory_order_relaxed);
    return ok ? VS_OK : VS_ERR_NO_DEVICE;
}
} // namespace vs

namespace {

// of this thread's next launches (vs_internal_set_merge_wait)
thread_local uint32_t merge_wait = 2000;

struct Plan {
    int32_t impl, rpw, waves, row_groups, rows, rows_pad, num_splits, keys_per_split, total_wgs, schedule;
    int32_t own_tiles;  // every wave has key tiles of its own (attention_mfma_rows.hip): row blocks per workgroup, else 0
    int32_t bal_chunks; // balanced schedule: shares per (KV head, row group); num_splits = slots per KV head
    int32_t f32_rows; // fp32 storage: query rows per workgroup
    int32_t rounds; // loop schedule on the LDS-resident kernel's form: splits in rounds of 128 keys
    int32_t res_rb; // resident schedule: row blocks per workgroup (4, 2 or 1)
};
bool merges_inside(const vs_attn_desc* d, const Plan& pl);
int filling_splits(int wgs, int tiles);
int pipe_splits(const vs_attn_desc* d, Plan pl, int nrb, int waves, int tiles);

// Shape / dtype / layout checks that need no device. Returns VS_OK or a vs_error.
int32_t check_desc(const vs_attn_desc* d, int tree = 1) {
    if (!d) return VS_ERR_NULL;
    if (d->B < 1 || d->T < 1 || d->T > VS_MAX_TREE || d->Hq < 1 || d->Hkv < 1 || d->Hq % d->Hkv != 0)
        return VS_ERR_SHAPE;
    if (d->d != 64 && d->d != 128) return VS_ERR_SHAPE;
    if ((int64_t)d->B * d->Hkv > kMaxGridY) return VS_ERR_SHAPE; // one grid row per (sequence, KV head) in the combine
    // query rows are counted in 32 bits, up to a whole row block (q and out of this many would not fit the card)
    if ((int64_t)d->T * d->Hq > (0x7fffffff - kRowBlock) / d->B) return VS_ERR_SHAPE;
    if (d->max_prefix_len < 0) return VS_ERR_SHAPE;
    if (!(d->softmax_scale > 0.f) || !isfinite(d->softmax_scale)) return VS_ERR_SHAPE;
    if (d->dtype != VS_BF16 && d->dtype != VS_F32) return VS_ERR_DTYPE;
    if (d->impl != VS_IMPL_AUTO && d->impl != VS_IMPL_GENERIC && d->impl != VS_IMPL_MFMA) return VS_ERR_SHAPE;
    if (d->impl == VS_IMPL_MFMA && d->dtype != VS_BF16) return VS_ERR_DTYPE;
    if (d->num_splits < 0 || d->rows_per_wave < 0 || d->rows_per_wave > 2) return VS_ERR_SHAPE;
    if (d->waves_per_group != 0 && d->waves_per_group != 1 && d->waves_per_group != 2 && d->waves_per_group != 4 &&
        d->waves_per_group != 8)
        return VS_ERR_SHAPE;
    if (d->schedule != VS_SCHED_AUTO && d->schedule != VS_SCHED_LOOP && d->schedule != VS_SCHED_PIPELINED &&
        d->schedule != VS_SCHED_RESIDENT && d->schedule != VS_SCHED_BALANCED)
        return VS_ERR_SHAPE;
    if (d->schedule == VS_SCHED_RESIDENT && (d->rows_per_wave == 2 || (d->waves_per_group != 0 && d->waves_per_group != 8)))
        return VS_ERR_SHAPE; // eight waves, one row block each
    if (d->schedule == VS_SCHED_BALANCED) {
        // a lane per sequence and per share; num_splits, when given, is the number of shares
        if (d->B > kBalMaxSeqs || d->num_splits > kBalMaxChunks) return VS_ERR_SHAPE;
        if (d->impl == VS_IMPL_GENERIC || d->dtype != VS_BF16) return VS_ERR_SHAPE;
    }
    if (d->schedule == VS_SCHED_PIPELINED || d->schedule == VS_SCHED_BALANCED) {
        // the pipelined kernel exists for one row block per wave and four or eight waves
        if (d->rows_per_wave == 2) return VS_ERR_SHAPE;
        if (d->waves_per_group != 0 && d->waves_per_group != 4 && d->waves_per_group != 8) return VS_ERR_SHAPE;
    }
    if (d->stride_head < 0 || d->stride_tok < d->d) return VS_ERR_LAYOUT;
    const int64_t need = (int64_t)d->max_prefix_len + (tree ? d->T : 0);
    if (!tree && d->max_prefix_len < 1) return VS_ERR_SHAPE;
    if (d->paged) {
        if (!is_pow2(d->block_size) || d->block_size < 16) return VS_ERR_LAYOUT;
        if (d->max_blocks < 1 || d->num_blocks < 1 || d->stride_block < 0) return VS_ERR_LAYOUT;
        if (!d->block_table) return VS_ERR_NULL;
        if (need > (int64_t)d->max_blocks * d->block_size) return VS_ERR_LAYOUT;
    } else {
        if (d->stride_seq < 0 || d->capacity < 1) return VS_ERR_LAYOUT;
        if (need > d->capacity) return VS_ERR_LAYOUT;
    }
    const bool mfma = d->impl == VS_IMPL_MFMA || (d->impl == VS_IMPL_AUTO && d->dtype == VS_BF16);
    if (mfma) {
        // token offsets inside one (sequence, KV head) slice are kept in 32 bits
        if (d->stride_tok >= ((int64_t)1 << 30)) return VS_ERR_LAYOUT; // (the product below would wrap for some)
        const int64_t span = d->paged ? (int64_t)d->block_size * d->stride_tok : need * d->stride_tok;
        if (span >= ((int64_t)1 << 30)) return VS_ERR_LAYOUT;
        // 16-byte vector loads of 8 bf16
        if (d->stride_head % 8 || d->stride_tok % 8 || (d->paged ? d->stride_block % 8 : d->stride_seq % 8))
            return VS_ERR_LAYOUT;
    }
    return VS_OK;
}

Plan plan_kernel(const vs_attn_desc* d, int tree) {
    Plan pl{};
    const int group = d->Hq / d->Hkv;
    pl.rows = d->T * group;
    pl.rows_pad = (pl.rows + kRowBlock - 1) / kRowBlock * kRowBlock;
    pl.impl = d->impl == VS_IMPL_AUTO ? (d->dtype == VS_BF16 ? VS_IMPL_MFMA : VS_IMPL_GENERIC) : d->impl;
    if (pl.impl == VS_IMPL_GENERIC) {
        // fp32 storage: eight waves share eight rows, or four where that keeps to one workgroup per CU (2 x 31
        // nodes, 8 / 2 heads of 128 channels, 600 keys: 124 workgroups of four rows 12 us, 62 of eight 19 us; with
        // more workgroups than CUs the second read of K and V costs more: 280 of four 26.8, 140 of eight 25.0 us);
        // bf16 storage: a wave per row
        const bool f32 = d->dtype == VS_F32;
        pl.f32_rows = (int64_t)d->B * d->Hkv * ((pl.rows + 3) / 4) <= kNumCUs ? 4 : 8;
        pl.rpw = 0;
        pl.waves = f32 ? 8 : 1;
        pl.row_groups = f32 ? (pl.rows + pl.f32_rows - 1) / pl.f32_rows : 1;
        pl.num_splits = 1;
        pl.keys_per_split = 0;
        pl.total_wgs = f32 ? d->B * d->Hkv * pl.row_groups : d->B * d->T * d->Hq;
        return pl;
    }
    const int nrb = pl.rows_pad / kRowBlock;
    const int tiles = ((int64_t)d->max_prefix_len + (tree ? d->T : 0) + kIterKeys - 1) / kIterKeys;
    const int units0 = d->B * d->Hkv;
    // Which kernel: the first that applies (the figures stand at each predicate; a "unit" is a (sequence, KV head)).
    //  * one row block, and some launches of two: key tiles of the wave's own (own_ok)
    //  * long batches whose sequences may differ in length: balanced shares (balanced_ok, bal_capped, rnd_fills)
    //  * short sequences and, below twelve units, up to 2048 keys: a split's keys resident in LDS (resident_ok)
    //  * up to four row blocks, or few units: splits of any length in rounds of 128 keys (rounds_ok)
    //  * twelve units and more: the software-pipelined kernel, one row block per wave, the rows split over row groups of
    //    eight (or four) waves, and key splits only when units x row groups leave CUs empty
    //  * the straight loop: AUTO without other knobs reaches it only with fewer than twelve units of more than 256 workgroups' rows
    // A caller's schedule is taken as it is. With other knobs set AUTO leaves out own tiles and rounds; rows_per_wave = 2 or a wave
    // count that the pipelined kernel does not have mean the straight loop: one row block per wave unless told otherwise,
    // up to four waves for small launches and eight for large ones.
    const bool big = units0 >= kManyUnits;
    int rpw = d->rows_per_wave, waves = d->waves_per_group, splits = d->num_splits;
    const bool pipe_ok = (rpw == 0 || rpw == 1) && (waves == 0 || waves == 4 || waves == 8);
    const bool many = units0 >= 12; // enough (sequence, KV head) units for the pipelined kernel, see below
    // Below twelve units the LDS-resident kernel for up to 2048 keys, as long as all its workgroups (up to 96 KB of LDS each: one
    // per CU) run at once: splits of two 64-key tiles when that fits, else three (28 / 4 heads, 60 nodes, 1696 keys, every
    // layer cold in the caches: 14 splits of 128 keys 15.8 us, 10 of 192 16.7, with a combine kernel behind both). For 5000
    // keys and more its 192-key limit forces too many partial results.
    const int res_rg = (nrb + 3) / 4;
    // Short sequences: one split where it is at most the kernel's 192 keys, then splits of 64 keys where those find a CU
    // each (with few splits the merge's items queue up in few waves: 1 x 60 nodes, 28 / 4 heads, 400 keys in splits of 128 12.3 us, of
    // 64 9.3; 650 keys 11.0 / 9.8; 2 x 17 nodes, 1400 keys 11.5 / 10.7), and then for any number of units (4 x 14 nodes,
    // 120 keys: rounds 11.7, one split 9.7; 12 x 62 nodes, 76 keys: pipelined 14.8, one split 11.0).
    // Four tiles (193 .. 256 keys) of twelve units or more stay one split too, as two rounds (below): their sums then remain fp32
    // up to the one final rounding. Splits store bf16 partial rows - relative error of N(0, 1) inputs 2.6e-3 in four splits
    // of 64 keys, 2.2e-3 in one - and are hardly faster: 28 / 4 heads, 190 .. 240 keys, us in one split / in four (one of
    // the pipelined kernel's): 3 x 60 nodes 11.4 / 11.6 (16.6), 16 x 14 nodes 11.2 / 12.1 (13.3); 32 / 8 heads of 64, 2 x 31 nodes
    // 8.1 / 7.9 (9.7), 16 x 31 8.9 / 11.6 in two (10.6).
    const bool one_split = many && tiles == 4;
    const int res_short = tiles <= 3 ? 1 : (tiles <= 32 && !one_split && (int64_t)units0 * res_rg * tiles <= kNumCUs ? tiles : 0);
    const int res_tps = res_short ? tiles / res_short : (int64_t)units0 * res_rg * ((tiles + 1) / 2) <= kNumCUs ? 2 : 3; // 64-key tiles per split
    const int res_splits = splits > 0 ? splits : (tiles + res_tps - 1) / res_tps;
    const bool resident_ok = (!many || (res_short && splits <= 0)) && nrb >= 2 && tiles <= 32 && (rpw == 0 || rpw == 1) && (waves == 0 || waves == 8) &&
                             (splits <= 0 || (tiles + splits - 1) / splits <= kResidentMaxKeys / kIterKeys) &&
                             (int64_t)units0 * res_rg * res_splits <= kNumCUs;
    // Twelve units: from there on the pipelined kernel beats the straight loop (us per call, loop / pipelined, 28 / 4 heads, 60 nodes,
    // 1696 keys: 2 sequences 21.7 / 23.3, 3: 26.3 / 24.9, 4: 28.6 / 26.9, 8: 39.9 / 31.4, 11: 50.9 / 39.9).
    // Balanced shares instead of equal splits per sequence: for batches whose sequences may differ in
    // length (the host only knows the longest allowed one). As many workgroups as the CUs hold at once
    // (one of eight waves, two of four). Taken when the launch would need key splits to fill those
    // places anyway, or when whole sequences would make more than one round and less than two - shares
    // then replace a second, partly filled round of workgroups of unequal length - and a share would
    // be 32 steps of 64 keys if every sequence had the longest allowed length (reading the lengths and
    // cutting the shares costs each kernel a dependent load and a few microseconds).
    // Paged batches, one layer, planner's other choice / balanced shares, lengths drawn from 1024 .. 8192
    // unless stated. 28 / 4 heads, 16 sequences: 138 / 118, 135 / 107, 138 / 106, 127 / 96 us; all
    // 4600 keys: 93 / 98; all 8000: 150 / 156; 256 .. 2048 keys: 50 / 57; 32 sequences: 242 / 192;
    // 40: 279 / 226, all 3000 keys 202 / 162; 64: 418 / 340, all 3000 keys 227 / 237. 32 / 32 heads,
    // 4 sequences: 120 / 77; 8: 237 / 168; 12: 262 / 201; 24: 422 / 361; 32: 518 / 487, and 32 folded layers
    // of 3136 keys 308 / 334.
    // (Both with a combine kernel behind them; shares now merge their own pieces and take 0.90 of that.)
    // A launch that is one full round of whole sequences is left alone: unequal lengths would gain there too (32 x 60 nodes, 28 / 4
    // heads, 1000 .. 8000 keys 210 / 152), equal and short ones lose (all of 1000 44 / 48, 3000 112 / 114), and the
    // host cannot tell which it has - such callers ask for VS_SCHED_BALANCED themselves. Two rounds or more are left alone as
    // well: nothing is gained (64 x 1000 .. 8000 317 / 321, all of 3000 220 / 218) and 32 / 32 heads lose 5 - 15 %.
    const int bal_waves = waves ? waves : (nrb > 4 ? 8 : 4);
    const int bal_rg = (nrb + bal_waves - 1) / bal_waves;
    const int bal_places = kNumCUs * (bal_waves == 8 ? 1 : 2);
    const int bal_w_auto = bal_places / (d->Hkv * bal_rg) > kBalMaxChunks ? kBalMaxChunks : bal_places / (d->Hkv * bal_rg);
    const int bal_wgs = units0 * bal_rg;
    const bool balanced_ok = many && pipe_ok && splits <= 0 && d->B >= 2 && d->B <= kBalMaxSeqs &&
                             (bal_wgs * 32 < bal_places * 25 || (bal_wgs > bal_places && bal_wgs < 2 * bal_places)) &&
                             bal_w_auto >= 2 && (int64_t)d->B * tiles >= 32 * (int64_t)bal_w_auto;
    // Rounds: the resident kernel's form (keys split among the waves too) on splits of any length, 128 keys in LDS at
    // a time. Where a unit's rows are at most one workgroup (two to four row blocks) and all workgroups run at
    // once, or too few units for the pipelined kernel: us per call, pipelined with its combine kernel / rounds
    //   4 x 16 nodes, 28 / 4 heads, 1300 keys 16.7 / 11.4; 16 x the same, up to 8191 keys 68.3 / 57.2
    //   8 x 31 nodes, 32 / 8 heads of 64, up to 2047 keys 18.1 / 16.6; 4 x 60 nodes, 32 / 32 heads, 3400 keys 51.2 / 47.6
    // and straight loop / rounds 2 x 60 nodes, 28 / 4 heads, 1696 keys 17.6 / 14.2, one of 6684 keys 25.2 / 18.4.
    // More workgroups than CUs: 16 x 60 nodes, 32 / 32 heads, 1000 keys 61.4 / 64.1. One sequence of many KV heads
    // with two row blocks of 128 channels: 700 keys 15.8 / 10.6, 1300 keys 15.9 / 12.5, 3136 keys 18.9 / 20.1.
    const int rnd_rb = nrb >= 3 ? 4 : 2;
    const int rnd_wgs = units0 * ((nrb + rnd_rb - 1) / rnd_rb);
    // With few KV heads the 64 shares do not fill the places, and the kernels that split the keys among the waves take
    // over: us per call, shares / they: 64 x 30 nodes, 8 / 2 heads, 1000 .. 7999 keys 188 / 98; 64 x 14, 8 / 1 heads
    // 176 / 56; 64 x 16, 28 / 4 heads, 8000 keys 278 / 221, 1024 .. 8191 keys 197 / 175; 20 x 13, 4096 .. 8191 keys 89 / 71.
    // - as long as they find a place for two splits of every sequence, or a whole one fills the chip. In between, us per call,
    // whole sequences / five splits of each / shares: 40 x 18 nodes, 28 / 4 heads, 1024 .. 8191 keys 162 / 132 / -; 36 x 18, 687 .. 5500
    // - / 89 / 68, 2750 .. 5500 - / 101 / 91, all of 5500 - / 112 / 118; 33 x 11, 1000 .. 8000 - / 121 / 95, all of 8000 - / 132 / 122;
    // 52 x 11, 4000 .. 8000 - / 181 / 161; 58 x 18, 1000 .. 8000 - / 181 / 154, all of 8000 - / 241 / 241; and from 240 workgroups on 62 x 18, 400 .. 3200
    // 79 / - / 96, 1000 .. 8000 168 / - / 153, all of 8000 216 / - / 236.
    // (More than four row blocks have no rounds, and the pipelined kernel's splits are no choice for them, though faster where shares fill at
    // most half of the CUs - us per call, shares / splits: 8 / 1 heads, 56 x 29 nodes, 7025 keys 141.6 / 58.1; 50 x 51, 694 .. 5554 72.6 / 70.4 -:
    // with about as many shares as sequences most of those are one piece, fp32 up to the final rounding, and every split is a bf16 partial row.
    // Relative error against 64 bits, 40 drawn calls of them, shares / splits: mean 2.77e-3 / 2.80e-3, at most 2.54e-3 / 2.74e-3 (62 x 62
    // nodes, 8 / 2 heads, 331 .. 2652 keys).)
    const bool bal_capped = bal_w_auto * d->Hkv * bal_rg < bal_places * 7 / 8;
    const bool rnd_fills = 2 * rnd_wgs <= kNumCUs || rnd_wgs >= 240;
    const bool knobs = d->schedule != VS_SCHED_AUTO || rpw != 0 || waves != 0 || splits > 0;
    const bool rounds_ok = !knobs && nrb >= 2 && rnd_wgs <= kNumCUs && (!many || one_split || (nrb <= 4 && (nrb > 2 || d->B > 1 || d->d == 64 || tiles <= 24)));
    // One row block: tiles of the wave's own (attention_mfma_rows.hip), for any number of units: splits of at least 192
    // keys while CUs are free (28 / 4 heads, 4 nodes: 700 keys in one split 9.7 us, in four 8.8; 400 keys 8.2 / 9.1 in
    // three); past one workgroup of eight waves per CU whole sequences, two workgroups of four waves (32 x 20
    // nodes, 32 / 32 heads, 818 keys: pipelined 90, these 81 us). Two row blocks of 128 channels: the rounds' finer
    // splits win while there are CUs for them (2 x 9 nodes, 1700 keys 9.8 / 12.6 us), from splits of 1024 keys on, and
    // for one split of at most 320 keys, the waves' own tiles do (16 x 9 nodes, up to 8191 keys 47.8 / 43.2; 200 keys 11.1 / 8.9).
    const bool own_ok = !knobs && (nrb == 1 || (nrb == 2 && d->d == 128 && units0 <= kNumCUs && (!balanced_ok || bal_capped) &&
                                                ((many && (int64_t)units0 * tiles >= 16 * kNumCUs) || tiles <= 5)));
    pl.schedule = d->schedule != VS_SCHED_AUTO ? d->schedule
                  : own_ok                     ? VS_SCHED_LOOP
                  : balanced_ok && !(bal_capped && rounds_ok && rnd_fills) ? VS_SCHED_BALANCED
                  : many && resident_ok        ? VS_SCHED_RESIDENT
                  : many && rounds_ok          ? VS_SCHED_LOOP
                  : many && pipe_ok            ? VS_SCHED_PIPELINED
                  : resident_ok                ? VS_SCHED_RESIDENT
                                               : VS_SCHED_LOOP;
    if (pl.schedule == VS_SCHED_BALANCED) {
        pl.rpw = 1;
        pl.waves = bal_waves;
        pl.row_groups = bal_rg;
        pl.bal_chunks = splits > 0 ? splits : (bal_w_auto < 1 ? 1 : bal_w_auto);
        pl.num_splits = pl.bal_chunks + d->B; // partial-result slots per KV head
        pl.keys_per_split = 0;                // shares are measured at run time
        pl.total_wgs = pl.bal_chunks * d->Hkv * pl.row_groups;
        return pl;
    }
    if (pl.schedule == VS_SCHED_RESIDENT) {
        // eight waves = res_rb row blocks x 8 / res_rb key parts; a split holds at most
        // kResidentMaxKeys keys (three 64-key tiles)
        pl.rpw = 1;
        pl.waves = 8;
        pl.res_rb = nrb >= 3 ? 4 : nrb;
        pl.row_groups = (nrb + pl.res_rb - 1) / pl.res_rb;
        const int max_tiles = kResidentMaxKeys / kIterKeys;
        if (splits <= 0) splits = res_splits;
        int tps = (tiles + splits - 1) / splits;
        if (tps > max_tiles) tps = max_tiles;
        if (tps < 1) tps = 1;
        pl.keys_per_split = tps * kIterKeys;
        pl.num_splits = (tiles + tps - 1) / tps;
        pl.total_wgs = units0 * pl.row_groups * pl.num_splits;
        return pl;
    }
    if (pl.schedule == VS_SCHED_LOOP && own_ok && units0 <= kNumCUs) {
        // ... in the resident kernel where the splits fit it and all run at once: one split of up to 256 keys, or (where own
        // tiles would be split too) splits of 64, 128 or 192. us per call, own tiles / resident, 28 / 4 heads unless stated:
        //   one split: 4 x 3 nodes, 60 keys 6.1 / 4.9, 150 keys 6.6 / 6.2; 4 x 8 nodes (two row blocks), 60 keys 8.4 / 6.0, 150 keys 9.1 / 7.2
        //   one row block, split: 1 x 3, 600 keys 9.0 in three / 7.5 in ten of 64; 4 x 3, 1200 10.4 / 9.0 in ten of 128;
        //     16 x 3, 600 11.4 / 10.4 in four of 192; 32 / 8 heads of 64, 4 x 6, 600 8.3 / 7.4 in five of 128
        // From seventeen splits on a merge takes a second trip to memory (0.55 us); 128 keys a split cost 0.2 us over 64, 192 0.7.
        // (Own tiles keep one row block over 256 keys, a tile for every wave: paged 6.6 / 6.9; and splits of 192 beyond sixteen: 7 x 3
        // nodes, 8 / 2 heads, 3152 keys 11.5 / 11.7.)
        int tps = tiles <= 3 || (tiles == 4 && nrb == 2) ? tiles : 0;
        float best = INFINITY;
        for (int t = 1; t <= 3 && tiles > 8; ++t) {
            const int n = (tiles + t - 1) / t;
            const float cost = (t == 1 ? 0.f : t == 2 ? 0.2f : 0.7f) + (n > 16 ? 0.55f : 0.f);
            if (n <= (t == 3 ? 16 : kMergeMaxSplits) && units0 * n <= kNumCUs && cost < best) {
                best = cost;
                tps = t;
            }
        }
        if (tps > 0) {
            pl.rounds = 1;
            pl.rpw = 1;
            pl.waves = 8;
            pl.res_rb = nrb;
            pl.row_groups = 1;
            pl.keys_per_split = tps * kIterKeys;
            pl.num_splits = (tiles + tps - 1) / tps;
            pl.total_wgs = units0 * pl.num_splits;
            return pl;
        }
    }
    if (pl.schedule == VS_SCHED_LOOP && own_ok) {
        // One short split of two row blocks: a workgroup for each where both find a CU (smaller launches keep the plan they had). us per call, both blocks in one / one each: 16 x 9
        // nodes, 28 / 4 heads, 291 keys 9.3 / 6.6; 25 x 9, 290 keys, paged 9.9 / 7.0; 3 x 40, 32 / 32 heads, 250 keys 9.0 / 6.5. (Long sequences are read
        // twice then, and few of them at a time keep half as many bytes in flight: 30 x 9, 600 .. 5000 keys, cold 47.2 / 52.5.)
        pl.own_tiles = nrb == 2 && tiles <= 5 && units0 >= 16 && 2 * units0 <= kNumCUs ? 1 : nrb;
        pl.rpw = 1;
        pl.row_groups = nrb / pl.own_tiles;
        pl.waves = units0 > kNumCUs ? 4 : 8;
        splits = tiles <= 8 ? 1 : tiles / 3;
        if (splits > kNumCUs / (units0 * pl.row_groups)) splits = kNumCUs / (units0 * pl.row_groups);
        if (splits > kMergeMaxSplits) splits = kMergeMaxSplits;
        if (splits < 1) splits = 1;
        const int tps = (tiles + splits - 1) / splits;
        pl.keys_per_split = tps * kIterKeys;
        pl.num_splits = (tiles + tps - 1) / tps;
        pl.total_wgs = units0 * pl.row_groups * pl.num_splits;
        return pl;
    }
    if (pl.schedule == VS_SCHED_LOOP && rounds_ok) {
        pl.rounds = 1;
        pl.rpw = 1;
        pl.waves = 8;
        pl.res_rb = rnd_rb;
        pl.row_groups = (nrb + pl.res_rb - 1) / pl.res_rb;
        splits = kNumCUs / (units0 * pl.row_groups);
        const int most = one_split ? 1 : (tiles + 1) / 2;
        if (splits > most) splits = most;
        if (splits > kMergeMaxSplits) splits = kMergeMaxSplits;
        if (splits < 1) splits = 1;
        const int tps = (tiles + splits - 1) / splits;
        pl.keys_per_split = tps * kIterKeys;
        pl.num_splits = (tiles + tps - 1) / tps;
        pl.total_wgs = units0 * pl.row_groups * pl.num_splits;
        return pl;
    }
    if (pl.schedule == VS_SCHED_PIPELINED) {
        rpw = 1;
        if (!waves) waves = nrb > 4 ? 8 : 4;
        if (splits <= 0) splits = pipe_splits(d, pl, nrb, waves, tiles);
    } else {
        if (!rpw) rpw = 1;
        if (!waves) {
            const int need1 = (nrb + rpw - 1) / rpw;
            const int cap = (big && nrb > 4) ? kMaxWaves : 4;
            waves = 1;
            while (waves < need1 && waves < cap) waves *= 2;
        }
    }
    pl.rpw = rpw;
    pl.waves = waves;
    const int need = (nrb + pl.rpw - 1) / pl.rpw;
    pl.row_groups = (need + pl.waves - 1) / pl.waves;
    const int units = units0 * pl.row_groups;
    if (splits <= 0) {
        // large: fill the CUs once. Small launches are latency-bound: the write-back of the
        // partial results at the end of the kernel (about 0.2 us per split for a C3-sized
        // launch) and the combine grow with the split count, the loop (about 2 us per 64 keys
        // with one wave per SIMD) with the keys per split; measured optima were 3 iterations
        // of 64 keys per split for short sequences and 8 for long ones, with at most one
        // workgroup per CU (two C3 sequences: 7 splits = 224 workgroups 21.7 us, 10 splits = 320
        // workgroups 25.1 us).
        if (big) {
            splits = kNumCUs / units;
        } else {
            const int iters = tiles <= 32 ? 3 : (tiles <= 64 ? 5 : 8);
            splits = (tiles + iters - 1) / iters;
            const int cap = kNumCUs / units; // one workgroup per CU: a second one on some CUs makes those the tail
            if (splits > cap) splits = cap;
        }
        const int max_splits = (tiles + 1) / 2;
        if (splits > max_splits) splits = max_splits;
    }
    if (splits < 1) splits = 1;
    if (splits > tiles) splits = tiles;
    if (splits > 64) splits = 64; // more splits than this only add partial-result traffic
    const int tiles_per_split = (tiles + splits - 1) / splits;
    pl.keys_per_split = tiles_per_split * kIterKeys;
    pl.num_splits = (tiles + tiles_per_split - 1) / tiles_per_split;
    pl.total_wgs = units * pl.num_splits;
    return pl;
}

// rows of partial results: every (sequence, KV head) has num_splits slots; the balanced schedule has
// num_splits slots per KV head for the whole batch
size_t partial_rows(const vs_attn_desc* d, const Plan& pl) {
    return (size_t)(pl.bal_chunks > 0 ? 1 : d->B) * d->Hkv * pl.num_splits * pl.rows_pad;
}

// Splits merged by their own workgroups instead of a combine kernel: they wait for each other, so only where
// all of them run at once (given an idle device; with a busy one the wait is bounded). Few splits of many rows stay with
// the combine kernel, which spreads them over the whole chip: with six items for a wave (merge_splits)
// 2 splits of 192 rows took 19.2 us against 18.0.
// A workgroup of the pipelined kernel has up to eight row blocks and often few splits, so that its waves have several items, more
// than they take at once; the merge then only pays where most of the chip takes part in it. us per call, inside / combine
// kernel (sequences x nodes, keys, splits x workgroups; 28 / 4 heads of 128 channels unless stated):
//   from seven splits on: 3 x 35, 2019, 9 x 108 19.7 / 20.9; 3 x 27, 4036, 16 x 192 19.7 / 23.0; 3 x 60, 3136, 10 x 240 22.4 / 25.5;
//     32 / 8 heads of 64, 2 x 35, 1770, 8 x 128 13.9 / 15.9
//   fewer, on 11/16 of the CUs: 9 x 22, 148 .. 1186, 5 x 180 20.2 / 21.2; 5 x 60, 1000, 5 x 200 21.6 / 21.8; 8 x 35, 1247, 6 x 192 20.9 / 21.6; 8 x 60,
//     3136, 4 x 256 36.5 / 40.8; 9 x 36 (40 / 8 heads), 2166, 3 x 216 34.1 / 37.2; but 8 x 39, 85 .. 684, 3 x 192 21.9 / 21.1;
//     on fewer: 3 x 60, 1000, 5 x 120 20.3 / 19.5; 4 x 60, 1000, 5 x 160 20.8 / 20.1; 3 x 60, 1400, 6 x 144 20.4 / 20.1; 5 x 46 (28 / 4
//     heads of 64), 919, 4 x 160 17.1 / 16.6
//   two and three with at most three items already on 9/16 (heads of 64): 11 x 48 (32 / 8), 1744, 2 x 176 26.8 / 27.8; 6 x 50 (32 / 8),
//     261 .. 523, 3 x 144 14.9 / 15.3; on fewer: 5 x 44 (28 / 4), 650, 3 x 120 16.1 / 15.6; 2 x 52 (32 / 8), 527, 3 x 48 16.0 / 15.0
bool merges_inside(const vs_attn_desc* d, const Plan& pl) {
    const int blocks = pl.rows_pad / kRowBlock, in_group = (blocks + pl.row_groups - 1) / pl.row_groups;
    const int items = in_group * (d->d / 8), takers = pl.num_splits * pl.waves;
    const bool few_items = pl.num_splits <= 3 && items <= 3 * takers;
    const bool pipelined = pl.schedule == VS_SCHED_PIPELINED && (pl.num_splits >= 7 || pl.total_wgs >= kNumCUs * (few_items ? 9 : 11) / 16);
    return (pl.schedule == VS_SCHED_RESIDENT || pipelined || pl.rounds || pl.own_tiles) && pl.num_splits > 1 &&
           pl.num_splits <= kMergeMaxSplits && pl.total_wgs <= kNumCUs && items <= 4 * takers &&
           pl.rows_pad <= (1 << 16); // offsets inside a row group's partial results are 32 bits wide
}

// Key splits that fill the CUs with `wgs` workgroups each, of four iterations or more; launches that fill 200 CUs with whole sequences stay whole.
int filling_splits(int wgs, int tiles) {
    const int n = wgs >= 200 ? 1 : kNumCUs / wgs, most = (tiles + 3) / 4;
    return n < most ? n : most;
}

// Key splits of the pipelined kernel, where a caller names none: as many as fill the CUs, or with eight waves of 128 channels whole sequences, where
// a model of the kernel's time (3 % rms of 394 timings of 12 .. 200 units x row groups, 5 .. 60 iterations, 1 .. 20 splits) says that
// the iterations saved are not worth the merge. us per call, 28 / 4 heads, filling / whole: 24 x 25 nodes, 61 .. 490 keys 2 21.9 / 19.6; 10 x 64, 25 ..
// 203 keys 2 19.4 / 15.1; 22 x 35, 615 keys 2 26.7 / 23.2. Over 9241 drawn calls that it takes 0.83 of the time, eight of them 1.01 -
// 1.02. 64 channels lose (16 x 40, 48 .. 388 keys 2 14.1 / 15.1); of four waves two workgroups share a CU.
// Never more splits: finer ones were faster (12 x 21 nodes, 481 keys 2 17.1 / 4 13.4), but the shorter sequences of a ragged batch, one piece
// and so fp32 up to the final rounding in a coarser split, are then bf16 partial rows. Relative error against 64 bits, 40 drawn
// calls each, filling / so: whole 2.68e-3 / 2.30e-3; finer ones 2.76e-3 / 2.77e-3, at worst 2.17e-3 / 2.59e-3 (2 x 36 nodes, 32 / 8 heads
// of 64, 68 .. 548 keys, 3 / 5 resident splits).
int pipe_splits(const vs_attn_desc* d, Plan pl, int nrb, int waves, int tiles) {
    pl.schedule = VS_SCHED_PIPELINED;
    pl.waves = waves;
    pl.row_groups = (nrb + waves - 1) / waves;
    const int wgs = d->B * d->Hkv * pl.row_groups, filling = filling_splits(wgs, tiles);
    if (waves == 4 || d->d != 128 || filling == 1) return filling;
    pl.num_splits = filling;
    pl.total_wgs = filling * wgs;
    const auto loop = [&](int n) { return (tiles + n - 1) / n * (1.2f + 0.28f * n * wgs / kNumCUs); }; // us: iterations take longer with all CUs at work
    const float mb = (float)filling * (d->B * d->Hkv) * pl.rows_pad * d->d * 2e-6f;                    // of partial rows
    const float split = 8.f + loop(filling) + (merges_inside(d, pl) ? 0.9f + 0.35f * mb : 2.1f + 0.48f * mb);
    return 8.f + loop(1) < 0.93f * split ? 1 : filling; // whole ones have to bring more than the model is good for (0.95: up to 1.05 of the time)
}

size_t workspace_bytes(const vs_attn_desc* d, const Plan& pl) {
    if (pl.impl != VS_IMPL_MFMA || pl.num_splits <= 1) return 0;
    const size_t prow = partial_rows(d, pl);
    return align_up(prow * d->d * sizeof(uint16_t)) + align_up(prow * 2 * sizeof(float)) +
           (pl.bal_chunks > 0 ? align_up(kBalMaxChunks * sizeof(int32_t)) : 0) + // (unused: the size that callers know)
           (merges_inside(d, pl) ? align_up((size_t)d->B * d->Hkv * pl.row_groups * kGateWords * sizeof(uint64_t)) : 0);
}

// How the resident kernel cuts a launch. Its eight waves are row blocks x key parts, so with fewer row blocks a wave has fewer
// tiles one after the other, and taking up to four times the workgroups for the same rows costs nothing while CUs are idle.
// us per call, 28 / 4 heads (1 to 4 sequences of 16 to 60 nodes, 100 .. 1700 keys), by row blocks of a workgroup (1, 2, 4) and
// 64-key tiles of a split; a call that is one split takes 2.0 less, heads of 64 channels 1.0 less in nearly the same order.
constexpr float kResidentCost[3][4] = {{6.5f, 6.95f, 7.5f, 8.1f}, {7.1f, 7.6f, 8.8f, 9.25f}, {8.1f, 8.9f, 10.7f, INFINITY}};
float resident_cost(int row_blocks, int tps, int n) { return kResidentCost[row_blocks / 2][tps - 1] - (n == 1 ? 2.f : 0.f); }

// The kernel and its cut as plan_kernel has them, or (AUTO without other knobs) the resident kernel's cheapest cut into no more
// splits - a split's rows are rounded once more than the sums - whose workgroups all run at once. us per call before / with it:
//   one split: 1 x 60 nodes, 28 / 4 heads, 130 keys 7.1 / 4.9, 4 x 60, 190 keys 9.0 / 5.7; 8 x 31, 32 / 8 heads of 64, 90 keys 5.6 / 4.4
//   fewer row blocks: 1 x 25, 28 / 4, 325 keys, six splits 8.0 / 6.1; 1 x 42, 1291 keys, 21 / 11 splits 8.3 / 7.5; 8 x 29, 8 / 2, 410 keys 7.8 / 7.1
//   fewer than the rounds of 128 keys had: 1 x 33, 8 / 2, 2025 keys 9.8 / 8.0; 2 x 29, 1911 .. 3822 keys, 31 splits 9.6 / 8.4
//   in place of the pipelined kernel: 4 x 21, 28 / 4, 741 keys, three splits 15.9 / 8.2; 6 x 36, 32 / 8, 297 keys 15.0 / 11.3; 8 x 34, 32 / 8 heads of
//     64, 240 keys 12.0 / 8.8
// Of some 110 shapes drawn from the changed calls the slowest stayed within 1 % of what it was, and the gain is a little larger with K and
// V cold in the caches. Up to 64 tiles, as far as was measured; twelve units and more up to 24 (from there on the rule for rounds ends too).
// RESIDENT by name, with no number of splits or with the one that AUTO reports, is AUTO's plan where that is RESIDENT too: the number
// of row blocks is no knob, and a caller who asks for the plan that was reported gets it.
Plan make_plan(const vs_attn_desc* d, int tree = 1) {
    if (d->schedule == VS_SCHED_RESIDENT) {
        vs_attn_desc any = *d;
        any.schedule = VS_SCHED_AUTO;
        any.num_splits = any.rows_per_wave = any.waves_per_group = 0;
        const Plan pl = make_plan(&any, tree);
        if (pl.schedule == VS_SCHED_RESIDENT && (d->num_splits == 0 || d->num_splits == pl.num_splits)) return pl;
    }
    const Plan base = plan_kernel(d, tree);
    const int nrb = base.rows_pad / kRowBlock;
    const int tiles = ((int64_t)d->max_prefix_len + (tree ? d->T : 0) + kIterKeys - 1) / kIterKeys;
    const int units = d->B * d->Hkv;
    const bool knobs = d->schedule != VS_SCHED_AUTO || d->rows_per_wave != 0 || d->waves_per_group != 0 || d->num_splits > 0;
    if (base.impl != VS_IMPL_MFMA || knobs || base.schedule == VS_SCHED_BALANCED || nrb < 2 || (int64_t)units * nrb > 4 * kNumCUs || tiles > (units < 12 ? 64 : 24))
        return base;
    int allowed = base.num_splits;
    if (base.schedule == VS_SCHED_PIPELINED) { // whole sequences of it where splits of this one are the faster ones: 10.1 us instead of 14 and the like
        const int n = filling_splits(units * base.row_groups, tiles), tps = (tiles + n - 1) / n;
        allowed = (tiles + tps - 1) / tps;
    }
    // (the pipelined kernel, the loops and longer rounds cost more than any of these)
    const float keep = 0.95f; // another number of splits has to bring more than the table is good for
    const bool same_kernel = base.res_rb > 0 && base.keys_per_split <= resident_max_keys(base.res_rb);
    float best = same_kernel ? keep * resident_cost(base.res_rb, base.keys_per_split / kIterKeys, base.num_splits) : INFINITY;
    Plan pl = base;
    for (int rb = 1; rb <= 4; rb *= 2) {
        const int groups = (nrb + rb - 1) / rb;
        const int most = kNumCUs / (units * groups) < allowed ? kNumCUs / (units * groups) : allowed;
        for (int tps = 1; tps <= resident_max_keys(rb) / kIterKeys && tps <= tiles; ++tps) {
            if (tps * most < tiles) continue;
            const int n = (tiles + tps - 1) / tps;
            const float cost = (n == allowed ? keep : 1.f) * resident_cost(rb, tps, n);
            if (!(cost < best)) continue;
            Plan c = base;
            c.schedule = base.schedule == VS_SCHED_LOOP ? VS_SCHED_LOOP : VS_SCHED_RESIDENT;
            c.rounds = base.schedule == VS_SCHED_LOOP;
            c.own_tiles = 0;
            c.rpw = 1;
            c.waves = 8;
            c.res_rb = rb;
            c.row_groups = groups;
            c.keys_per_split = tps * kIterKeys;
            c.num_splits = n;
            c.total_wgs = units * groups * n;
            if (n > 1 && !merges_inside(d, c)) continue;
            best = cost;
            pl = c;
        }
    }
    return pl;
}

// K and V as data that is read once (nt loads), where one workgroup alone reads a tile: kernels without row groups that share it, and a contiguous
// cache in which no two rows are the same memory. Sequences that share a prompt's rows read them from the caches, which such loads
// pass by, and a block table, of which the host knows nothing, may have it so: us per call, plain / such loads, all
// sequences on the same rows: 64 x 4 nodes, 28 / 4 heads, 8000 keys paged 56 / 90, half of the keys 121 / 130, contiguous with a sequence stride of 0 53 / 85;
// 64 x 9, 1024 .. 8191 keys paged 73 / 92; 8 x 60 nodes, 32 / 32 heads, 1024 .. 8191 keys paged 105 / 119. (Paged caches without common blocks gain
// as much as contiguous ones do; such launches go without.)
// Such loads come faster from memory and leave less of their data in the caches: faster for who finds nothing there, as the layers of a model, each with
// a cache of its own, do; not always for who goes over one layer again and again that the 256 MB cache in front of the memory would have held - least so
// where CUs are idle and each of the others waits for its own loads. Time relative to plain loads, over other data each time / over the
// same, 30379 drawn calls on contiguous caches, by the megabytes of K and V up to the longest allowed prefix; filled: all but a tenth of the CUs' places
// taken in the last round, 99 in 100 calls over the same data in brackets:
//   own tiles of one row block, filled 20 .. 40 0.95 / 0.98 (1.05), .. 96 0.93 / 0.94 (1.04), .. 256 0.91 / 0.99 (1.15), .. 512 0.90 / 0.94 (1.12), above 0.89 / 0.89;
//   not filled .. 96 0.94 / 0.97 (1.08), .. 256 0.91 / 1.03 (1.22), .. 512 0.89 / 0.95 (1.16), above 0.89 / 0.88;
//   of two row blocks, filled 128 .. 256 0.92 / 1.00 (1.10), .. 512 0.91 / 0.95 (1.13), above 0.91 / 0.91; not filled .. 256 0.93 / 1.04 (1.18);
//   four waves of the pipelined kernel, filled .. 256 0.98 / 1.00 (1.09), .. 512 0.92 / 0.96 (1.06), .. 768 0.91 / 0.90, above 0.89 / 0.89; not filled, above 768 0.92 / 0.91.
// (Two row groups of eight waves, which share what they read, 1.03 / 1.04.) So what is too large for any cache, and of the rest what repeats
// no slower; of two row blocks, whose repetition takes 1.00 (1.12 where all are half as long as allowed and half of the splits have no keys), all that fills
// the CUs. All that the rule takes 0.906 / 0.908, 39 of 8124 over 1.05 of the same data's time. us per call: 64 x 4 nodes, 28 / 4 heads, 8000 keys 184 / 162;
// 4 x 60 nodes, 32 / 32 heads, 2880 .. 3392 keys, one layer of 32 45.1 / 40.7; 8 x 60, 1024 .. 8191 keys 159 / 139; 20 x 60, 2000 keys 155 / 132
bool reads_once(const vs_attn_desc* d, const Plan& pl, int tree) {
    const bool four = (pl.schedule == VS_SCHED_PIPELINED || pl.schedule == VS_SCHED_BALANCED) && pl.waves == 4;
    if (d->paged || pl.row_groups != 1 || !(pl.own_tiles || four)) return false;
    const int64_t keys = (int64_t)d->max_prefix_len + (tree ? d->T : 0);
    if (!rows_apart(d->d, keys, d->stride_tok, d->Hkv, d->stride_head, d->B, d->stride_seq)) return false;
    const double mb = (double)d->B * d->Hkv * keys * d->d * 4e-6;
    const int places = kNumCUs * (pl.waves == 8 ? 1 : 2), rounds = (pl.total_wgs + places - 1) / places;
    const bool filled = pl.total_wgs >= 0.9 * rounds * places;
    return mb >= (filled ? 512 : 768) || (filled && ((pl.own_tiles == 1 && mb >= 40 && mb < 96) || (pl.own_tiles == 2 && mb >= 128)));
}

int32_t draft_chunks(int32_t V, int32_t vec) { return (int32_t)(((int64_t)V + vec * kDraftVec - 1) / (vec * kDraftVec)); }
// Chunks of 8192 logits; of 10240 or 12288 where those of 8192 are more workgroups than there are CUs and these are not: the CUs with
// two of them hold up the sequence's last part. us, three levels and the selection, chunks of 8192 / chosen so:
//   2 x 8 x 152064 34.6 / 33.2, 3 x 8 x 98304 32.1 / 31.9, 5 x 8 x 60000 31.1 / 30.4, 8 x 8 x 36000 31.4 / 30.6, 8 x 8 x 45000 32.1 / 31.8,
//   1 x 16 x 180000 52.7 / 48.3
// (So the order of a row's sums, and with it the last bits of its scores, depends on the number of rows in the call, which the header says.)
int32_t draft_vec(int32_t V, int64_t rows) {
    for (int32_t vec = 4; vec <= 6; ++vec)
        if (rows * draft_chunks(V, vec) <= kNumCUs) return vec;
    return 4;
}
int32_t accept_chunks(int32_t V) { return (V + kAcceptChunk - 1) / kAcceptChunk; }

} // namespace

extern "C" {

void vs_internal_set_merge_wait(uint32_t ticks) { merge_wait = ticks; }
int32_t vs_internal_reads_once(const vs_attn_desc* desc, int32_t tree) {
    const int32_t rc = check_desc(desc, tree);
    return rc != VS_OK ? rc : reads_once(desc, make_plan(desc, tree), tree);
}

int32_t vs_version(void) { return VS_VERSION; }

const char* vs_strerror(int32_t err) {
    switch (err) {
    case VS_OK: return "ok";
    case VS_ERR_NULL: return "a required pointer is NULL";
    case VS_ERR_SHAPE: return "unsupported or inconsistent shape";
    case VS_ERR_DTYPE: return "unsupported dtype";
    case VS_ERR_WORKSPACE: return "workspace missing or too small";
    case VS_ERR_HIP: return "HIP runtime error at launch";
    case VS_ERR_LAYOUT: return "unsupported strides, alignment or paging parameters";
    case VS_ERR_NO_DEVICE: return "no usable gfx950 device";
    default: return "unknown error";
    }
}

const char* vs_status_string(int32_t code) {
    switch (code) {
    case VS_STATUS_OK: return "ok";
    case VS_STATUS_BAD_ROOT: return "parent[0] is not -1";
    case VS_STATUS_BAD_PARENT: return "a parent index is outside [0, i)";
    case VS_STATUS_BAD_PREFIX: return "prefix_len outside the cache or the host bound";
    case VS_STATUS_BAD_BLOCK: return "a block-table entry is outside the pool";
    case VS_STATUS_BAD_PATH: return "accepted path is not the root followed by increasing node ids";
    case VS_STATUS_BAD_CANDIDATE: return "a candidate's parent is not an earlier candidate, or a child outscores its parent";
    default: return "unknown status";
    }
}

int32_t vs_tree_validate_host(const int32_t* parent, int32_t T) {
    if (!parent) return VS_ERR_NULL;
    if (T < 1 || T > VS_MAX_TREE) return VS_ERR_SHAPE;
    return validate_tree_host(parent, T);
}

int32_t vs_tree_mask_build(const int32_t* parent, int32_t B, int32_t T, uint64_t* mask, int32_t* depth,
                           int32_t* status, void* stream) {
    if (!parent || !mask || !depth) return VS_ERR_NULL;
    if (B < 1 || T < 1 || T > VS_MAX_TREE) return VS_ERR_SHAPE;
    if (const int32_t dc = check_device()) return dc;
    return launch_tree_mask(parent, B, T, mask, depth, status, (hipStream_t)stream) == hipSuccess ? VS_OK
                                                                                                    : VS_ERR_HIP;
}

int32_t vs_attention_plan(const vs_attn_desc* desc, vs_attn_plan* plan) {
    if (!plan) return VS_ERR_NULL;
    const int32_t rc = check_desc(desc);
    if (rc != VS_OK) return rc;
    const Plan pl = make_plan(desc);
    plan->impl = pl.impl;
    plan->num_splits = pl.bal_chunks > 0 ? pl.bal_chunks : pl.num_splits;
    plan->keys_per_split = pl.keys_per_split;
    plan->row_groups = pl.row_groups;
    plan->waves_per_group = pl.waves;
    plan->rows_per_wave = pl.rpw;
    plan->workgroups = pl.total_wgs;
    plan->combine = (pl.impl == VS_IMPL_MFMA && pl.num_splits > 1) ? 1 : 0;
    plan->schedule = pl.schedule;
    return VS_OK;
}

size_t vs_attention_workspace_bytes(const vs_attn_desc* desc) {
    if (check_desc(desc) != VS_OK) return 0;
    return workspace_bytes(desc, make_plan(desc));
}

namespace {
// Shared by the two attention entry points. tree = 1: the T queries are tree nodes whose own
// K/V sit behind the prefix; tree = 0: T learnable queries over the prefix alone.
int32_t enqueue_attention(const vs_attn_desc* desc, int tree, const void* q, const void* k_cache, const void* v_cache,
                          const int32_t* prefix_len, const int32_t* tree_parent, const uint64_t* tree_mask, void* out,
                          int32_t* status, void* workspace, size_t workspace_bytes_given, void* stream) {
    const int32_t rc = check_desc(desc, tree);
    if (rc != VS_OK) return rc;
    Plan pl = make_plan(desc, tree);
    // (a finer cut has more gates, 256 bytes each: with less scratch than it asks for a call runs on the other one's)
    if (workspace_bytes_given < workspace_bytes(desc, pl)) pl = plan_kernel(desc, tree);
    if (pl.impl == VS_IMPL_MFMA && !(aligned16(q) && aligned16(k_cache) && aligned16(v_cache) && aligned16(out)))
        return VS_ERR_LAYOUT;
    const size_t need = workspace_bytes(desc, pl);
    if (need > 0 && (!workspace || workspace_bytes_given < need || ((uintptr_t)workspace & (kAlign - 1))))
        return VS_ERR_WORKSPACE;
    if (const int32_t dc = check_device()) return dc;

    AttnParams p{};
    p.q = q;
    p.k = k_cache;
    p.v = v_cache;
    p.out = out;
    p.prefix_len = prefix_len;
    p.parent = tree_parent;
    p.tree_mask = tree_mask;
    p.block_table = desc->paged ? desc->block_table : nullptr;
    p.status = status;
    p.B = desc->B;
    p.T = desc->T;
    p.tree_keys = tree ? desc->T : 0;
    p.Hq = desc->Hq;
    p.Hkv = desc->Hkv;
    p.d = desc->d;
    p.group = desc->Hq / desc->Hkv;
    p.inv_group = 1.f / (float)p.group;
    p.node_stride = (int64_t)(desc->Hq - p.group) * desc->d;
    p.row_skip = desc->Hq - p.group;
    p.rows = pl.rows;
    p.rows_pad = pl.rows_pad;
    p.max_prefix_len = desc->max_prefix_len;
    p.paged = desc->paged ? 1 : 0;
    p.block_size = desc->paged ? desc->block_size : 1;
    p.block_shift = 0;
    while ((1 << p.block_shift) < p.block_size) ++p.block_shift;
    p.max_blocks = desc->max_blocks;
    p.num_blocks = desc->num_blocks;
    p.capacity = desc->capacity;
    p.stride_seq = desc->stride_seq;
    p.stride_block = desc->stride_block;
    p.stride_head = desc->stride_head;
    p.stride_tok = desc->stride_tok;
    p.scale = desc->softmax_scale;
    p.scale_log2 = desc->softmax_scale * 1.4426950408889634f;
    p.num_splits = pl.num_splits;
    p.keys_per_split = pl.keys_per_split;
    p.row_groups = pl.row_groups;
    p.rows_per_group = pl.f32_rows ? pl.f32_rows : (pl.res_rb ? pl.res_rb : pl.own_tiles ? pl.own_tiles : pl.waves * pl.rpw) * kRowBlock;
    p.total_wgs = pl.total_wgs;
    if (pl.num_splits > 0 && pl.row_groups > 0) {
        p.by_splits = fast_div_by(pl.num_splits);
        p.by_groups = fast_div_by(pl.row_groups);
        p.by_heads = fast_div_by(desc->Hkv);
    }
    p.bal_chunks = pl.bal_chunks;
    if (pl.bal_chunks > 0) {
        p.by_shares = fast_div_by(pl.bal_chunks);
        if (pl.bal_chunks % desc->B == 0) p.bal_per_seq = fast_div_by(pl.bal_chunks / desc->B);
    }
    // A launch of more whole sequences than run at once hands out the longest first (a lane per sequence), unless even the longest is
    // so short that the wait for all lengths costs more than it brings. us per call, longest first / in order:
    // pipelined kernel, 28 / 4 heads, 60 nodes, 64 sequences, all of 100 keys 41.6 / 36.1, 250 51.8 / 46.3, 500 65.0 / 60.0, 1000 93.2 / 89.1;
    // 1/8 .. 1 of 100 38.8 / 33.3, 250 42.7 / 40.5, 500 51.1 / 50.4, 1000 69.1 / 71.5, 2000 105.6 / 120.6; 40 sequences, 1/8 .. 1 of 500
    // 41.8 / 41.1, 1000 54.4 / 65.8; 20 of 32 / 32 heads, 1/8 .. 1 of 250 32.2 / 33.2, 500 39.1 / 42.0, 1000 57.5 / 61.6, all of 500 54.2 / 53.0
    // own tiles: 64 x 20 nodes, 32 / 32 heads, 30 .. 249 keys 56 / 45
    const int64_t by_length_from = pl.schedule == VS_SCHED_PIPELINED ? 768 : 1024; // longest allowed prefix
    p.by_length = (pl.schedule == VS_SCHED_PIPELINED || pl.own_tiles) && desc->max_prefix_len >= by_length_from && pl.num_splits == 1 &&
                  desc->B >= 2 && desc->B <= kBalMaxSeqs && pl.total_wgs > kNumCUs * (pl.waves == 8 ? 1 : 2) &&
                  !(pl.schedule == VS_SCHED_PIPELINED && pipe_three_per_cu(desc->d, pl.waves, pl.total_wgs));
    p.once = reads_once(desc, pl, tree);
    if (need > 0) {
        const size_t prow = partial_rows(desc, pl);
        p.part_o = (uint16_t*)workspace;
        p.part_ml = (float*)((char*)workspace + align_up(prow * desc->d * sizeof(uint16_t)));
        char* behind = (char*)p.part_ml + align_up(prow * 2 * sizeof(float));
        if (merges_inside(desc, pl)) p.gates = (uint64_t*)behind;
        p.crowd = pl.num_splits >= 28 && pl.total_wgs >= 224 && (pl.rounds || (pl.own_tiles == 1 && pl.waves == 8)); // why there: attn_mfma_common.h
        p.merge_wait = merge_wait;
    }
    hipStream_t s = (hipStream_t)stream;
    hipError_t e;
    if (pl.impl == VS_IMPL_GENERIC) {
        e = desc->dtype == VS_F32 ? launch_attention_f32(p, s) : launch_attention_generic(p, s);
    } else {
        e = (pl.schedule == VS_SCHED_PIPELINED || pl.schedule == VS_SCHED_BALANCED) ? launch_attention_mfma_pipe(p, pl.rpw, pl.waves, s)
            : pl.own_tiles ? launch_attention_mfma_rows(p, pl.waves, s)
            : pl.rounds ? launch_attention_mfma_rounds(p, pl.res_rb, s)
            : pl.schedule == VS_SCHED_RESIDENT ? launch_attention_mfma_resident(p, pl.res_rb, s)
                                               : launch_attention_mfma(p, pl.rpw, pl.waves, s);
        if (e == hipSuccess && pl.num_splits > 1 && !p.gates && pl.bal_chunks == 0) e = launch_attention_combine(p, desc->dtype, s);
    }
    return e == hipSuccess ? VS_OK : VS_ERR_HIP;
}
} // namespace

int32_t vs_tree_verify_attention(const vs_attn_desc* desc, const void* q, const void* k_cache,
                                 const void* v_cache, const int32_t* prefix_len, const int32_t* tree_parent,
                                 const uint64_t* tree_mask, void* out, int32_t* status, void* workspace,
                                 size_t workspace_bytes_given, void* stream) {
    if (!desc || !q || !k_cache || !v_cache || !prefix_len || !tree_parent || !out) return VS_ERR_NULL;
    return enqueue_attention(desc, 1, q, k_cache, v_cache, prefix_len, tree_parent, tree_mask, out, status, workspace,
                             workspace_bytes_given, stream);
}

size_t vs_compress_attention_workspace_bytes(const vs_attn_desc* desc) {
    if (check_desc(desc, 0) != VS_OK) return 0;
    return workspace_bytes(desc, make_plan(desc, 0));
}

int32_t vs_compress_attention(const vs_attn_desc* desc, const void* q, const void* k, const void* v,
                              const int32_t* kv_len, void* out, int32_t* status, void* workspace,
                              size_t workspace_bytes_given, void* stream) {
    if (!desc || !q || !k || !v || !kv_len || !out) return VS_ERR_NULL;
    return enqueue_attention(desc, 0, q, k, v, kv_len, nullptr, nullptr, out, status, workspace, workspace_bytes_given,
                             stream);
}

size_t vs_accept_workspace_bytes(int32_t B, int32_t T, int32_t V) {
    if (B < 1 || T < 1 || T > VS_MAX_TREE || V < 1) return 0;
    const size_t n = (size_t)B * T * accept_chunks(V);
    return align_up(n * sizeof(float)) + align_up(n * sizeof(int32_t));
}

int32_t vs_tree_accept(const float* logits, int64_t ld_logits, int32_t V, const int32_t* draft_tokens,
                       const int32_t* parent, int32_t B, int32_t T, int32_t* accepted_len, int32_t* path,
                       int32_t* bonus_token, int32_t* row_argmax, int32_t* status, void* workspace,
                       size_t workspace_bytes_given, void* stream) {
    if (!logits || !draft_tokens || !parent || !accepted_len || !path || !bonus_token) return VS_ERR_NULL;
    if (B < 1 || T < 1 || T > VS_MAX_TREE || V < 1 || ld_logits < V) return VS_ERR_SHAPE;
    if ((int64_t)B * T * accept_chunks(V) > kMaxGridX) return VS_ERR_SHAPE; // one workgroup per (row, chunk)
    const size_t need = vs_accept_workspace_bytes(B, T, V);
    if (!workspace || workspace_bytes_given < need || ((uintptr_t)workspace & (kAlign - 1))) return VS_ERR_WORKSPACE;
    if (const int32_t dc = check_device()) return dc;
    AcceptParams p{};
    p.logits = logits;
    p.ld = ld_logits;
    p.V = V;
    p.draft = draft_tokens;
    p.parent = parent;
    p.B = B;
    p.T = T;
    p.accepted_len = accepted_len;
    p.path = path;
    p.bonus = bonus_token;
    p.row_argmax = row_argmax;
    p.status = status;
    return launch_accept(p, workspace, (hipStream_t)stream) == hipSuccess ? VS_OK : VS_ERR_HIP;
}

size_t vs_accept_sample_workspace_bytes(int32_t B, int32_t T, int32_t V) {
    if (B < 1 || T < 1 || T > VS_MAX_TREE || V < 1 || accept_chunks(V) > 2 * kMaxSampleChunks) return 0;
    const size_t n = (size_t)B * T * accept_chunks(V);
    return 2 * align_up(n * sizeof(float));
}

int32_t vs_tree_accept_sample(const float* logits, int64_t ld_logits, int32_t V, float temperature,
                              const int32_t* draft_tokens, const int32_t* parent, const float* u_accept,
                              const float* u_bonus, int32_t B, int32_t T, int32_t* accepted_len, int32_t* path,
                              int32_t* bonus_token, int32_t* status, void* workspace, size_t workspace_bytes_given,
                              void* stream) {
    if (!logits || !draft_tokens || !parent || !u_accept || !u_bonus || !accepted_len || !path || !bonus_token)
        return VS_ERR_NULL;
    if (B < 1 || T < 1 || T > VS_MAX_TREE || V < 1 || ld_logits < V) return VS_ERR_SHAPE;
    if (accept_chunks(V) > 2 * kMaxSampleChunks || (int64_t)B * T * accept_chunks(V) > kMaxGridX) return VS_ERR_SHAPE;
    if (!(temperature > 0.f) || !(temperature < INFINITY)) return VS_ERR_SHAPE;
    const size_t need = vs_accept_sample_workspace_bytes(B, T, V);
    if (!workspace || workspace_bytes_given < need || ((uintptr_t)workspace & (kAlign - 1))) return VS_ERR_WORKSPACE;
    if (const int32_t dc = check_device()) return dc;
    SampleParams p{};
    p.logits = logits;
    p.ld = ld_logits;
    p.V = V;
    p.draft = draft_tokens;
    p.parent = parent;
    p.u_accept = u_accept;
    p.u_bonus = u_bonus;
    p.B = B;
    p.T = T;
    p.accepted_len = accepted_len;
    p.path = path;
    p.bonus = bonus_token;
    p.status = status;
    p.k_log2 = 1.4426950408889634f / temperature;
    return launch_accept_sample(p, workspace, (hipStream_t)stream) == hipSuccess ? VS_OK : VS_ERR_HIP;
}

size_t vs_draft_expand_workspace_bytes(int32_t B, int32_t F, int32_t V, int32_t K) {
    if (B < 1 || F < 1 || F > VS_MAX_TREE || K < 1 || K > kMaxDraftK || F * K > kMaxDraftCand || V < K) return 0;
    const size_t n = (size_t)B * F * accept_chunks(V); // (what it was with 4096-float chunks; half of it is used)
    return 2 * align_up(n * sizeof(float)) + 2 * align_up(n * K * sizeof(float)) + (size_t)B * kArrivalWords * sizeof(uint64_t);
}

int32_t vs_draft_expand(const float* logits, int64_t ld_logits, int32_t V, const float* cum_in,
                        const int32_t* frontier_cand, int32_t B, int32_t F, int32_t K, int32_t cand_base,
                        int32_t cand_capacity, int32_t* cand_token, float* cand_score, int32_t* cand_parent,
                        int32_t* next_frontier_cand, float* next_cum, void* workspace, size_t workspace_bytes_given,
                        void* stream) {
    if (!logits || !cand_token || !cand_score || !cand_parent || !next_frontier_cand || !next_cum) return VS_ERR_NULL;
    if (B < 1 || F < 1 || F > VS_MAX_TREE || K < 1 || K > kMaxDraftK || F * K > kMaxDraftCand) return VS_ERR_SHAPE;
    if (V < K || ld_logits < V || (int64_t)B * F * accept_chunks(V) > kMaxGridX) return VS_ERR_SHAPE;
    if (cand_base < 0 || cand_capacity < 1 || (int64_t)cand_base + (int64_t)F * K > cand_capacity) return VS_ERR_SHAPE;
    const size_t need = vs_draft_expand_workspace_bytes(B, F, V, K);
    if (!workspace || workspace_bytes_given < need || ((uintptr_t)workspace & (kAlign - 1))) return VS_ERR_WORKSPACE;
    if (const int32_t dc = check_device()) return dc;
    DraftExpandParams p{};
    p.logits = logits;
    p.ld = ld_logits;
    p.V = V;
    p.cum_in = cum_in;
    p.frontier_cand = frontier_cand;
    p.B = B;
    p.F = F;
    p.K = K;
    p.cand_base = cand_base;
    p.cand_capacity = cand_capacity;
    p.cand_token = cand_token;
    p.cand_score = cand_score;
    p.cand_parent = cand_parent;
    p.next_frontier_cand = next_frontier_cand;
    p.next_cum = next_cum;
    p.vec = draft_vec(V, (int64_t)B * F);
    p.chunks = draft_chunks(V, p.vec);
    p.by_chunks = fast_div_by(p.chunks);
    p.by_F = fast_div_by(F);
    p.by_K = fast_div_by(K);
    const size_t n = (size_t)B * F * p.chunks;
    char* w = (char*)workspace;
    p.part_ms = (uint64_t*)w;
    w += align_up(n * sizeof(uint64_t));
    p.part_top = (uint64_t*)w;
    w += align_up(n * K * sizeof(uint64_t));
    p.arrivals = (uint64_t*)w;
    return launch_draft_expand(p, (hipStream_t)stream) == hipSuccess ? VS_OK : VS_ERR_HIP;
}

int32_t vs_draft_tree_build(const int32_t* cand_token, const float* cand_score, const int32_t* cand_parent, int32_t B,
                            int32_t M, int32_t cand_capacity, int32_t N, const int32_t* root_token, int32_t* parent,
                            int32_t* draft_tokens, int32_t* node_cand, int32_t* num_nodes, int32_t* status,
                            void* stream) {
    if (!cand_token || !cand_score || !cand_parent || !parent || !draft_tokens || !node_cand || !num_nodes)
        return VS_ERR_NULL;
    if (B < 1 || M < 1 || M > kMaxDraftTotal || cand_capacity < M || N < 1 || N > VS_MAX_TREE - 1) return VS_ERR_SHAPE;
    if (const int32_t dc = check_device()) return dc;
    DraftBuildParams p{};
    p.cand_token = cand_token;
    p.cand_score = cand_score;
    p.cand_parent = cand_parent;
    p.root_token = root_token;
    p.B = B;
    p.M = M;
    p.N = N;
    p.cand_capacity = cand_capacity;
    p.parent = parent;
    p.tokens = draft_tokens;
    p.node_cand = node_cand;
    p.num_nodes = num_nodes;
    p.status = status;
    return launch_draft_tree_build(p, (hipStream_t)stream) == hipSuccess ? VS_OK : VS_ERR_HIP;
}

int32_t vs_tree_kv_commit(const vs_kv_desc* d, void* k_cache, void* v_cache, const int32_t* prefix_len,
                          const int32_t* path, const int32_t* accepted_len, int32_t* new_prefix_len,
                          int32_t* status, void* stream) {
    if (!d || !k_cache || !v_cache || !prefix_len || !path || !accepted_len || !new_prefix_len) return VS_ERR_NULL;
    if (d->B < 1 || d->T < 1 || d->T > VS_MAX_TREE || d->Hkv < 1 || d->d < 1 || d->num_layers < 1) return VS_ERR_SHAPE;
    if (d->dtype != VS_BF16 && d->dtype != VS_F32) return VS_ERR_DTYPE;
    const int64_t eb = d->dtype == VS_BF16 ? 2 : 4;
    if (d->stride_head < 0 || d->stride_tok < d->d || d->stride_layer < 0) return VS_ERR_LAYOUT;
    if (d->paged) {
        if (!is_pow2(d->block_size) || d->block_size < 16) return VS_ERR_LAYOUT;
        if (d->max_blocks < 1 || d->num_blocks < 1 || d->stride_block < 0) return VS_ERR_LAYOUT;
        if (!d->block_table) return VS_ERR_NULL;
        if (d->T > (int64_t)d->max_blocks * d->block_size) return VS_ERR_LAYOUT;
    } else {
        if (d->stride_seq < 0 || d->capacity < d->T) return VS_ERR_LAYOUT;
    }
    // rows move in 16-byte pieces
    if ((d->d * eb) % 16 || (d->stride_tok * eb) % 16 || (d->stride_head * eb) % 16 || (d->stride_layer * eb) % 16 ||
        ((d->paged ? d->stride_block : d->stride_seq) * eb) % 16)
        return VS_ERR_LAYOUT;
    if (!aligned16(k_cache) || !aligned16(v_cache)) return VS_ERR_LAYOUT;
    if (new_prefix_len == prefix_len) return VS_ERR_LAYOUT;
    if ((((int64_t)d->num_layers * 2 * d->Hkv * (d->d * eb / 16)) + 255) / 256 > 0x7fffffffLL || d->B > kMaxGridY) return VS_ERR_SHAPE;
    if (const int32_t dc = check_device()) return dc;
    CommitParams p{};
    p.k = k_cache;
    p.v = v_cache;
    p.prefix_len = prefix_len;
    p.path = path;
    p.accepted_len = accepted_len;
    p.block_table = d->paged ? d->block_table : nullptr;
    p.new_prefix_len = new_prefix_len;
    p.status = status;
    p.B = d->B;
    p.T = d->T;
    p.Hkv = d->Hkv;
    p.chunks_per_row = (int32_t)(d->d * eb / 16);
    p.items_per_seq = (int64_t)d->num_layers * 2 * d->Hkv * p.chunks_per_row;
    p.by_chunks = fast_div_by(p.chunks_per_row);
    p.by_heads = fast_div_by(d->Hkv);
    p.paged = d->paged ? 1 : 0;
    p.block_size = d->paged ? d->block_size : 1;
    p.block_shift = 0;
    while ((1 << p.block_shift) < p.block_size) ++p.block_shift;
    p.max_blocks = d->max_blocks;
    p.num_blocks = d->num_blocks;
    p.capacity = d->capacity;
    p.stride_layer_bytes = d->stride_layer * eb;
    p.stride_seq_bytes = d->stride_seq * eb;
    p.stride_block_bytes = d->stride_block * eb;
    p.stride_head_bytes = d->stride_head * eb;
    p.stride_tok_bytes = d->stride_tok * eb;
    return launch_kv_commit(p, (hipStream_t)stream) == hipSuccess ? VS_OK : VS_ERR_HIP;
}


} // extern "C"
