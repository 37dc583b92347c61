// Which kernel variant and work split a call takes: rules over sizes and measured times, host code only (no
// HIP header, so that they can be compiled and looked at without a device).
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <utility>
#include <vector>

namespace ttt {

// what the rules read of an attention call (a slice of the batch)
struct CallShape {
    int T, step_begin, n_steps, G, hkv;
    int n_docs;
    const int32_t* cu_host;   // n_docs + 1 entries, first entry = cu_base
    int cu_base;
};

// ------------------------------------------------------------------------------------------------
// Forward
// ------------------------------------------------------------------------------------------------
// How the waves of a workgroup share its work: eight waves (or four) with 32 rows each, or two key groups that
// take every second key tile of the same rows.
enum FwdSplit { kFwdEightWaves, kFwdFourWaves, kFwdTwoKeyGroups };

// Rows of the diagonal keys through LDS: up to three blocks behind the tile stages, if the LDS for one block at least is to
// be had without a workgroup less on the compute unit.  Fragment loads from global memory instead touch 32 rows each and
// wait (forward and backward of the last of twelve steps, 512 tokens: 12/2 heads, 64 or 128 rows 81.7 -> 69.0 us; 8/2 heads of
// 64, 32 rows 48.9 -> 44.3).  16-bit; a workgroup of `waves` waves in `key_groups` groups covers `rows` rows, `per_cu` of
// them share a compute unit.
struct DiagSlots {
    int rows, slots;   // rows copied of a block (whole copies of the workgroup), blocks; or 0, 0
};
constexpr int fwd_lds_max(int per_cu) { return 160 * 1024 / per_cu / 1024 * 1024; }
constexpr int fwd_lds_tiles(int head_dim, int elem_bytes, int key_groups) { return 4 * key_groups * 64 * head_dim * elem_bytes; }   // two stages of K and V
inline DiagSlots fwd_diag_slots(int head_dim, int waves, int key_groups, int per_cu, int rows) {
    const int copied = std::max(rows, waves * 64 * 16 / (head_dim * 2)), slot = 2 * copied * head_dim * 2;
    const int tiles = fwd_lds_tiles(head_dim, 2, key_groups), slots = std::min(3, (fwd_lds_max(per_cu) - tiles) / slot);
    return slots > 0 && slot <= tiles ? DiagSlots{copied, slots} : DiagSlots{0, 0};
}

// Which work split ends first: one key group (all eight waves share a 64-key tile) or two (each tile pair's tiles go
// to the two halves of the workgroup, which covers half as many rows).  Two groups halve the longest
// workgroup -- a causal launch of one step at 2048 tokens is one workgroup per compute unit, and ends with the
// one that has all the keys -- but copy every tile for half as many waves and pay set-up, merge and epilogue
// twice as often.  Estimate per split: the longest workgroup, or the work of all over the compute units,
// whichever is more.  Measured (16-bit, head_dim 128, us): a workgroup 3, a tile 1.55 while the device is not
// full and 1.85 when it is, a tile pair 2.0 and 2.2; a diagonal key through LDS 1.6 and 0.9, straight from global memory
// 4.0 and 2.1, a fifth more when the device is full (slopes over steps 1 to 12 of 512 ... 2048 tokens, 32/8, 16/8, 12/2
// and 16/16 heads: 1.0 ... 1.5 and 0.7 ... 0.85, 4.0 and 2.1; the prices are those that choose best).  Over 8371 shapes of 128 ...
// 8192 tokens, twelve head geometries, steps 0 to 11, the choice takes 1.0048 of the better one in the mean, less than 1.153 in 99
// of 100 (1.0054 and 1.173 with 2.0 and 1.3 for a key, and twice that unless a workgroup of one group has 64 rows).  One step,
// 32/8 heads: 1024 tokens 30 -> 22 us, 2048 60 -> 50, 3000 98 (114 with two groups); all seven steps at 2048 293 (373).
inline bool two_key_groups_end_first(const CallShape* calls, int n_calls, int pack_log2, int n_cu) {
    const int rows = (8 * 32) >> pack_log2;      // of a workgroup with one key group
    auto per_tile = [&](const CallShape& a) { return (int64_t)a.hkv * (a.G >> pack_log2) * a.n_steps; };
    int64_t tiles_all = 0;
    for (int i = 0; i < n_calls; ++i) tiles_all += (int64_t)(calls[i].T + rows - 1) / rows * per_tile(calls[i]);
    if (tiles_all > 6 * n_cu) return false;   // many rounds: the work decides
    double est[2];
    for (int ks = 1; ks <= 2; ++ks) {
        const int r = rows / ks;
        const bool through_lds = fwd_diag_slots(128, 8, ks, 1, r).slots > 0;
        const double diag = ks == 1 ? (through_lds ? 1.6 : 4.0) : through_lds ? 0.9 : 2.1;
        double longest = 0., work = 0.;
        for (int i = 0; i < n_calls; ++i) {
            const CallShape& a = calls[i];
            const double j_mean = a.step_begin + 0.5 * (a.n_steps - 1), j_max = a.step_begin + a.n_steps - 1;
            int doc = 0;
            int64_t steps = 0, n = 0, most = 0;
            for (int row = 0; row < a.T; row += r, ++n) {
                while (doc + 1 < a.n_docs && a.cu_host[doc + 1] - a.cu_base <= row) ++doc;
                const int64_t tiles = std::min(row + r - 1, a.T - 1) / 64 - (a.cu_host[doc] - a.cu_base) / 64 + 1;
                const int64_t s = (tiles + ks - 1) / ks;
                steps += s;
                most = std::max(most, s);
            }
            longest = std::max(longest, 3. + most * (ks == 1 ? 1.55 : 2.0) + j_max * diag);
            work += (n * (3. + j_mean * 1.2 * diag) + steps * (ks == 1 ? 1.85 : 2.2)) * (double)per_tile(a) / n_cu;
        }
        est[ks - 1] = std::max(longest, work);
    }
    return est[1] < 0.97 * est[0];
}

// The longest and all of what the tiles of `rows` rows of a slice see, in groups of `per` key blocks of `keys` keys.
struct KeyCount {
    int64_t tiles = 0, blocks = 0, groups = 0;
    int64_t longest = 0, longest_cut = 0;   // groups of one tile; of one with a document start inside a wave's 32 rows
};
inline KeyCount count_keys(const CallShape& a, int rows, int keys, int per) {
    KeyCount n;
    int doc = 0;
    for (int row = 0; row < a.T; row += rows) {
        while (doc + 1 < a.n_docs && a.cu_host[doc + 1] - a.cu_base <= row) ++doc;
        const int64_t blocks = std::min(row + rows - 1, a.T - 1) / keys - (a.cu_host[doc] - a.cu_base) / keys + 1, groups = (blocks + per - 1) / per;
        ++n.tiles;
        n.blocks += blocks;
        n.groups += groups;
        n.longest = std::max(n.longest, groups);
        for (int d = doc + 1; d < a.n_docs && a.cu_host[d] - a.cu_base < row + rows; ++d)
            if (a.cu_host[d] - a.cu_base < a.T && (a.cu_host[d] - a.cu_base) % 32 != 0) n.longest_cut = std::max(n.longest_cut, groups);
    }
    return n;
}

// The same choice for head_dim 64, whose workgroups leave room for others on their compute unit: eight waves in 128
// registers (two workgroups per unit), four waves and half the rows (three per unit), or two key groups
// (one per unit).  Long workgroups want splitting, by keys while there are few of them; many short ones want the fewest
// passes over the keys.  Two lines, at one and three of the largest workgroups per unit and 1024-token documents, say which, unless
// another split is estimated to take 0.98 of that one's time or less.  A split is estimated as its longest workgroup, or the work
// of all over the compute units (what each costs of its own counts more where they make no whole rounds) and a part of the longest one (how unevenly they end),
// whichever is more, by prices (us) fitted to 3000 launches of 40 ... 9000 tokens, timed in graphs (one launch after another
// the shortest are as long as their submission): seven head geometries, one document or many, first step 0 to 10, one to nine steps.
// A document that starts inside a wave's 32 rows masks every key tile of the one before it (4463 tokens and one more, 8/2 heads, one step: 58.7 us
// with four waves in one document, 96.7 in two), and diagonal keys cost more the fewer of their LDS slots there are.
// Over 1400 others the choice takes 1.008 of the best of the three in the mean, the lines alone 1.059; 15 launches in 1000 are more than
// 3 % slower than by the lines, 1.12 at most (28 by the estimates alone, which take 1.007).  566 tokens in two documents, 24/8
// heads, the last of eleven steps: 23 -> 17 us; 65, 64/4, nine steps from the tenth on: 22 -> 16.
// Beyond sixteen of the largest workgroups per unit (more than were measured) the fewest passes over the keys.
struct Fwd64Prices {
    double own, tile, diag;                  // the longest workgroup: of its own, per key tile (or pair of them), per diagonal key
    double wg, wg_tile, wg_diag;             // the work: per workgroup, its tiles, its diagonal keys
    double base, uneven, rounds;             // of the launch; of the longest workgroup; of what the last round leaves idle
    double masked;                           // per key tile of a workgroup with a document start inside a wave's rows
    double from_memory, one_slot, idle;      // diagonal keys that do not go through LDS, or through one slot: more, by; less for waves without rows, by
};
inline FwdSplit work_split_64(const CallShape* calls, int n_calls, int pack_log2, int n_cu) {
    constexpr Fwd64Prices kPrices[] = {   // in the order of FwdSplit
        {0.12, 1.19, 0.69, 2.54, 0.95, 0.46, 4.57, 0.34, 0.35, 0.36, 1.55, 0.34, 0.42},
        {0.62, 0.80, 0.51, 1.26, 0.50, 0.27, 3.74, 0.36, 0.57, 0.43, 0.95, 0.34, 0.33},
        {1.66, 1.23, 0.53, 4.14, 1.30, 0.47, 3.24, 0.03, 0.79, 0.39, 0., 0., 0.},
    };
    int64_t n_wgs = 0;
    int longest_doc = 0;
    for (int i = 0; i < n_calls; ++i) {
        const CallShape& a = calls[i];
        n_wgs += (int64_t)((a.T + (256 >> pack_log2) - 1) / (256 >> pack_log2)) * a.hkv * (a.G >> pack_log2) * a.n_steps;
        for (int r = 0; r < a.n_docs; ++r) longest_doc = std::max(longest_doc, a.cu_host[r + 1] - a.cu_host[r]);
    }
    if (n_wgs > 16 * (int64_t)n_cu) return kFwdEightWaves;
    const bool is_long = longest_doc >= 1024;
    const FwdSplit line = is_long && n_wgs <= n_cu                                    ? kFwdTwoKeyGroups
                          : n_wgs <= n_cu || (is_long && n_wgs <= 3 * (int64_t)n_cu) ? kFwdFourWaves
                                                                                     : kFwdEightWaves;
    double us[3];
    for (FwdSplit split : {kFwdEightWaves, kFwdFourWaves, kFwdTwoKeyGroups}) {
        const Fwd64Prices& p = kPrices[split];
        const int waves = split == kFwdFourWaves ? 4 : 8, groups = split == kFwdTwoKeyGroups ? 2 : 1, per_cu = split == kFwdEightWaves ? 2 : split == kFwdFourWaves ? 3 : 1;
        const int rows = (waves / groups * 32) >> pack_log2;
        const int slots = fwd_diag_slots(64, waves, groups, per_cu, rows).slots;
        double longest = 0., each = 0., tiles = 0., n = 0.;
        for (int i = 0; i < n_calls; ++i) {
            const CallShape& a = calls[i];
            const KeyCount keys = count_keys(a, rows, 64, groups);
            const double full = std::min(1., (double)a.T / rows), busy = 1. - p.idle * (1. - full), per_tile = (double)a.hkv * (a.G >> pack_log2) * a.n_steps;
            const double diag = busy * (1. + (slots == 0 ? p.from_memory * full : slots == 1 ? p.one_slot : 0.));
            const double chain = std::max(p.tile * keys.longest, (p.tile + p.masked) * keys.longest_cut);
            longest = std::max(longest, p.own + busy * chain + diag * p.diag * (a.step_begin + a.n_steps - 1));
            each += per_tile * keys.tiles * (p.wg + diag * p.wg_diag * (a.step_begin + 0.5 * (a.n_steps - 1)));
            tiles += per_tile * busy * keys.groups * p.wg_tile;
            n += per_tile * keys.tiles;
        }
        const double rounds = n / n_cu;
        if (rounds > 1.) each *= 1. + p.rounds * (std::ceil(rounds) / rounds - 1.);
        us[split] = p.base + std::max(longest, p.uneven * longest + (each + tiles) / n_cu);
    }
    const FwdSplit best = (FwdSplit)(std::min_element(us, us + 3) - us);
    return us[best] < 0.98 * us[line] ? best : line;
}

// The forward's split, and how many heads of a kv group share a workgroup (its log2).
struct FwdPlan {
    FwdSplit split;
    int pack_log2;
};

// One launch serves `n_calls` slices of a batch, all of one head geometry.
inline FwdPlan plan_fwd(const CallShape* calls, int n_calls, bool is_bf16, int head_dim, int n_cu) {
    const int G = calls[0].G;
    // as many heads of a kv group per workgroup as divide the group, at most 4
    int pack_log2 = 0;
    while ((2 << pack_log2) <= 4 && G % (2 << pack_log2) == 0) ++pack_log2;
    if (is_bf16 && head_dim == 128)
        return FwdPlan{two_key_groups_end_first(calls, n_calls, pack_log2, n_cu) ? kFwdTwoKeyGroups : kFwdEightWaves, pack_log2};
    if (is_bf16) return FwdPlan{work_split_64(calls, n_calls, pack_log2, n_cu), pack_log2};
    if (head_dim == 64) {
        // fp32 matrix instructions are slow and a short launch lasts as long as one wave's key tiles: two key groups
        // (LDS for one workgroup per compute unit) while every workgroup still gets a unit of its own (128 tokens, 4/4
        // heads, three steps 20 -> 13 us; 700 tokens, 8/1 heads, one step 56 -> 37)
        const int pack = std::min(pack_log2, 1);   // two waves per key group
        const int rows = (2 * 32) >> pack;
        int64_t n = 0;
        for (int i = 0; i < n_calls; ++i)
            n += (int64_t)((calls[i].T + rows - 1) / rows) * calls[i].hkv * (G >> pack) * calls[i].n_steps;
        if (n <= n_cu) return FwdPlan{kFwdTwoKeyGroups, pack};
    }
    return FwdPlan{kFwdFourWaves, pack_log2};
}
inline FwdPlan plan_fwd(const CallShape& a, bool is_bf16, int head_dim, int n_cu) { return plan_fwd(&a, 1, is_bf16, head_dim, n_cu); }

struct F32FwdPrices {
    double own, chain, diag;                  // the longest workgroup: of its own, per group of key blocks, per diagonal key
    double base, tile, block, tile_diag;      // the work: of the launch, per row tile, per key block, per diagonal key of a tile
};

// Whether an fp32 forward takes its operands straight from memory (ttt_fwd_f32_kernel: 32 rows of one head per workgroup, eight waves
// that take the key blocks in turn) or through LDS tiles, as `tiled` says.  Each is estimated as its longest workgroup, or
// the work of all over the compute units, by prices (us) fitted to 2863 launches of 32 ... 2500 tokens, eight head geometries, one step or up to
// eight at once: in the mean the lower estimate takes 1.003 / 1.002 of the better one (head_dim 64 / 128), tiles alone 1.35 / 1.96,
// memory alone 1.030 / 1.013.  Few or long workgroups want the first, many rounds of the device with four heads to a tile the second.
// Beyond those sizes tiles are better than estimated by a few percent (8963 tokens, 64/4 heads of 64, one step 5995 against 6393 us), so
// memory has to be estimated at 0.95: over 1100 launches of 150 ... 16384 tokens 0.878 / 0.767 of the time of tiles in the mean, 11 of them more than
// 3 % slower (0.876 / 0.762 and 87 by the lower estimate).
// kv_st: elements from row to row, a multiple of 8; a lane's place in a row or the fourth after it is a 32-bit byte offset.
inline bool fwd_f32_direct(const CallShape* calls, int n_calls, int head_dim, int n_cu, const FwdPlan& tiled, int64_t kv_st) {
    if (kv_st >= (int64_t)1 << 28) return false;
    const bool d64 = head_dim == 64;
    const F32FwdPrices m = d64 ? F32FwdPrices{5.2, 5.0, 0.19, 6.0, 5.2, 0.62, 0.33} : F32FwdPrices{3.2, 11.7, 0.54, 10.2, 8.3, 1.43, 0.87};
    const F32FwdPrices t = d64 ? F32FwdPrices{6.4, 5.1, 1.08, 8.3, 5.8, 5.26, 2.1} : F32FwdPrices{9.5, 11.8, 3.4, 19.8, 9.6, 12.3, 4.6};
    const int groups = tiled.split == kFwdTwoKeyGroups ? 2 : 1, rows = (128 / groups) >> tiled.pack_log2;
    double m_long = 0., m_work = 0., t_long = 0., t_work = 0.;
    for (int i = 0; i < n_calls; ++i) {
        const CallShape& a = calls[i];
        const double heads = (double)a.hkv * a.G * a.n_steps, j_max = a.step_begin + a.n_steps - 1, j_mean = a.step_begin + 0.5 * (a.n_steps - 1);
        const KeyCount nm = count_keys(a, 32, 32, 8), nt = count_keys(a, rows, 64, groups);
        m_long = std::max(m_long, m.own + m.chain * nm.longest + m.diag * j_max);
        m_work += heads * (nm.tiles * (m.tile + m.tile_diag * j_mean) + nm.blocks * m.block);
        t_long = std::max(t_long, t.own + t.chain * nt.longest + t.diag * j_max);
        t_work += heads / (1 << tiled.pack_log2) * (nt.tiles * (t.tile + t.tile_diag * j_mean) + (groups == 1 ? nt.groups * t.block : 0.));
    }
    return std::max(m_long, m.base + m_work / n_cu) < 0.95 * std::max(t_long, t.base + t_work / n_cu);
}

// ------------------------------------------------------------------------------------------------
// Work split of the 16-bit backward launch: 32-row query blocks per dK/dV chunk and ways to split the
// (step, head) list, chosen by a model of the launch.
//
// One workgroup fills a compute unit.  Measured on MI355X (chunk size x split swept at 512 ... 16384
// tokens, all steps and one step per call, five head geometries): a dK/dV unit = (128-key tile, chunk,
// split) costs about 1.9 us per step (one 32-row query block per wave group and (step, head) pair) plus
// about 13 us of its own (workgroup launch, the K_0/V_0 tile and first query block arriving, the flush
// of its sums through LDS and fp32 atomics), an empty unit (a tile that no row of the chunk sees) about
// 1 us; a dQ tile costs about 5 us per 128-key tile, 1.7 per diagonal key and 8 of its own; with
// head_dim 64 the streaming parts take 0.6 of that.  The model deals the units of one XCD in launch order
// to its compute units (each to the one that frees up first); over the sweeps its choice is 1.1 % slower
// than the best one on average and 5 % at most (the dK/dV units dealt alone, with 512 ... 2048-row
// chunks: 6 % and 17 %).  Long lists stop at 1024-row chunks: the model does not see HBM traffic, and
// with longer chunks the units of one XCD no longer stream the same Q / dO rows together (4096 tokens, all
// steps, dK/dV units alone: 2.6 GB fetched with 2048 rows, 0.9 with 512).  1024 rows already cost some of it:
// one launch fetches 2.9 GB there against 1.9 with 512, and at 2 x 8192 tokens, 64/4 heads 58 against 39 GB,
// where a forward and backward with 512 would be 0.7 and 1.1 % faster (4382 against 4414 us, 64.2 against 64.9
// ms).  Over 90 shapes of 768 ... 16384 tokens for which the two limits choose differently the backward takes 0.89 to
// 1.22 times as long with 512 at most, 1.004 in the geometric mean, so the line stays here -- but for long lists of
// two to four kv heads in a batch of 2048 tokens or more whose longest document has at least 1280: 512.  Over 476 such shapes
// for which the limits choose differently (12/2, 32/2, 12/3, 24/3, 32/4, 64/4 heads, 3 to 12 steps, up to 8192 tokens)
// the backward takes 0.80 to 1.06 times as long, 0.984 in the mean; 2 x 8192 tokens, 64/4 heads, with the forward 63.3 -> 62.7
// ms.  Elsewhere, from 2048 tokens on: shorter documents 1.02 (longest below 512) and 0.994, five to seven heads 0.997 with a
// document of 1280 and 1.000 in all, eight 1.011, 9 to 20 1.003, one 0.78 to 1.16 and 0.993 in the mean.
// ------------------------------------------------------------------------------------------------
struct DkvPlan {
    int chunk_blocks, n_split;
};

inline int64_t dkv_units_of(int T, int n_tiles, int chunk_blocks) {
    const int n_chunks = (T + chunk_blocks * 32 - 1) / (chunk_blocks * 32);
    int64_t n = 0;
    for (int ch = 0; ch < n_chunks; ++ch) n += std::min(n_tiles, (ch + 1) * chunk_blocks / 4);
    return n;
}

// Steps per (step, head) pair of one unit: its 32-row query blocks (from the tile's first row, or the chunk's, to the
// last row that sees the tile's last key), two at a time.  0: no row of the chunk sees the tile.
inline int dkv_unit_steps(int tile, int q_end, int chunk, int chunk_blocks) {
    const int first = std::max(tile * 4, chunk * chunk_blocks);
    const int n = std::min((q_end - 1) / 32, (chunk + 1) * chunk_blocks - 1) - first + 1;
    return n > 0 ? (n + 1) / 2 : 0;
}

// the share of one XCD of a launch part: unit number u of every kv head, in launch order (decode_block)
template <typename F> void for_units_of_an_xcd(int hkv, int64_t n_units, F&& f) {
    if (hkv % 8 == 0) {
        for (int64_t u = 0; u < n_units; ++u)
            for (int hp = 0; hp < hkv / 8; ++hp) f(u);
    } else if (8 % hkv == 0) {
        for (int64_t u = 0; u < n_units; u += 8 / hkv) f(u);
    } else {
        for (int64_t id = 0; id < n_units * hkv; id += 8) f(id / hkv);
    }
}

// Planning is on the caller's thread, and a packed batch has a new layout every iteration: what is counted per chunk
// size has a closed form per key tile, and units are listed only for options that are dealt, at most kMaxDealt in
// all; a launch with more is judged by its bound, to which it is then close (the choices at 128 ... 16384 tokens are
// those of dealing every option, up to 131072 tokens within 0.04 % by the model).  Seven calls of one step each,
// fresh layout of documents of 256 ... 4096 tokens, 32/8 heads: 16384 tokens 0.17 ms, 65536 1.1, 524288 1.3 (lists of
// all units per call: 0.36, 5.2 and 590).
//
// other_us: what the other slices of the same launch take of an XCD's compute units, in all; it is taken to fill them evenly.
// limit: only options that end sooner count.  only: this one counts.
struct BwdPrices {   // us
    float step, unit, empty;        // of a dK/dV unit: per step, of its own; one that no row sees
    float tile, diag, own;          // of a dQ tile: per 128-key tile, per diagonal key, of its own
    float later, later_pair;        // of a workgroup of the later blocks: of its own, per (step, head) pair; 0: not counted
    float flush;                    // of 256 units' sums: the rate of the atomics, all compute units together
};
struct BwdDeal {
    DkvPlan plan;
    double us;   // when the last compute unit ends, by the prices; < 0: no option ends before `limit`
};
constexpr int kDiagRegBlocks = 7, kDiagRegBlocksF32 = 3;   // later blocks whose rows and gradients fit a lane's registers
inline int diag_passes(const CallShape& a, int per_pass) { return std::max(1, (a.step_begin + a.n_steps - 2 + per_pass) / per_pass); }

inline BwdDeal deal_bwd(const CallShape& a, int n_cu, double other_us, const BwdPrices& price, int q_rows, bool short_launch,
                        int later_rows = 1, double limit = -1., const DkvPlan* only = nullptr) {
    const int T = a.T, n_jh = a.n_steps * a.G;
    const int n_tiles = (T + 127) / 128, n_tiles_q = (T + q_rows - 1) / q_rows;
    const float kStepUs = price.step, kUnitUs = price.unit, kEmptyUs = price.empty;
    const float kTileUs = price.tile, kDiagUs = price.diag, kQUs = price.own;
    const int kMaxDealt = short_launch ? 6144 : 12288;
    const int cus = std::max(1, n_cu / 8);
    const double share = (double)a.hkv / 8.;   // heads per XCD
    // document of token i, asked for rising i
    int doc = 0;
    auto doc_of = [&](int i) {
        while (doc + 1 < a.n_docs && a.cu_host[doc + 1] - a.cu_base <= i) ++doc;
        return doc;
    };
    // last query row (+1) that sees the last key of each tile: the end of that key's document
    std::vector<int> q_end(n_tiles), q_keys(n_tiles_q);
    for (int t = 0; t < n_tiles; ++t) q_end[t] = a.cu_host[doc_of(std::min(t * 128 + 127, T - 1)) + 1] - a.cu_base;
    doc = 0;
    double keys = 0.;
    for (int t = 0; t < n_tiles_q; ++t) {
        q_keys[t] = std::min((t + 1) * q_rows - 1, T - 1) / 128 - (a.cu_host[doc_of(t * q_rows)] - a.cu_base) / 128 + 1;
        keys += q_keys[t];
    }
    // the dQ tiles of one XCD in launch order
    const double n_dq = share * n_tiles_q * n_jh;
    const double dq_work = n_dq * (kQUs + (a.step_begin + 0.5 * (a.n_steps - 1)) * kDiagUs) + share * n_jh * keys * kTileUs;
    std::vector<float> dq;
    if (n_dq <= kMaxDealt)
        for_units_of_an_xcd(a.hkv, (int64_t)n_tiles_q * n_jh, [&](int64_t unit) {
            const int u = (int)unit, js = u / a.G % a.n_steps, t = n_tiles_q - 1 - u / n_jh;
            dq.push_back(kQUs + q_keys[t] * kTileUs + (a.step_begin + js) * kDiagUs);
        });
    const bool later = price.later > 0.f && a.step_begin + a.n_steps > 1;   // the later blocks' workgroups of one XCD
    const int n_later = later ? (int)(((int64_t)T * a.hkv + later_rows - 1) / later_rows * diag_passes(a, kDiagRegBlocks) + 7) / 8 : 0;
    const float later_us = price.later + price.later_pair * (float)n_jh;
    struct Option {
        int cb, ns;
        double flush;   // the atomics of all units
        double bound;   // about when the best schedule ends: the longest unit, or the work over the compute units
        double dealt;   // units and dQ tiles of one XCD
    };
    int longest_doc = 0;
    for (int r = 0; r < a.n_docs; ++r) longest_doc = std::max(longest_doc, a.cu_host[r + 1] - a.cu_host[r]);
    const bool few_heads = !short_launch && n_jh > 16 && a.hkv > 1 && a.hkv < 5 && T >= 2048 && longest_doc >= 1280;
    std::vector<Option> options;
    for (int log2_cb = 3; log2_cb <= 7; ++log2_cb) {
        const int cb = 1 << log2_cb;
        if (only && cb != only->chunk_blocks) continue;
        if (cb > 32 && n_jh > 8) break;
        if (cb > 16 && few_heads) break;
        if (cb > 8 && cb * 16 >= T) break;    // one chunk covers everything already
        // A tile is seen from the chunk of its own first row to that of its last row's block: the first of these
        // chunks and the last are partial, those between are whole.
        double blocks = 0., used = 0.;
        int most = 0;
        for (int t = 0; t < n_tiles; ++t) {
            const int c0 = t * 4 >> log2_cb, c1 = (q_end[t] - 1) >> (5 + log2_cb);
            const int s0 = dkv_unit_steps(t, q_end[t], c0, cb), s1 = c1 > c0 ? dkv_unit_steps(t, q_end[t], c1, cb) : 0;
            const int whole = std::max(0, c1 - c0 - 1);
            blocks += s0 + s1 + (double)whole * (cb / 2);
            used += c1 - c0 + 1;
            most = std::max({most, s0, s1, whole > 0 ? cb / 2 : 0});
        }
        const int64_t units = dkv_units_of(T, n_tiles, cb);
        for (int ns : {1, 2, 3, 4, 6, 8, 12, 16, 24}) {
            if (only && ns != only->n_split) continue;
            if (ns > 8 && !short_launch) break;
            if (ns > n_jh || units * ns * a.hkv > 0x7fffffff) break;   // (more workgroups than a grid has)
            const double work = share * (blocks * n_jh * kStepUs + ns * (used * kUnitUs + ((double)units - used) * kEmptyUs));
            const double longest = (double)((n_jh + ns - 1) / ns) * most * kStepUs + kUnitUs;
            const double flush = price.flush * used * ns * a.hkv / 256.;
            options.push_back(Option{cb, ns, flush, flush + std::max(longest, (work + dq_work + other_us + n_later * later_us) / cus),
                                     share * (double)units * ns + n_dq + n_later});
        }
    }
    std::sort(options.begin(), options.end(), [](const Option& x, const Option& y) { return x.bound < y.bound; });
    DkvPlan best{16, 1};
    if (!options.empty()) best = DkvPlan{options[0].cb, options[0].ns};
    double best_us = -1., dealt = 0.;
    if (limit >= 0.) {
        best_us = limit;
        best = DkvPlan{0, 0};
    }
    std::vector<float> free_at;
    std::vector<int> steps;
    for (const Option& o : options) {
        if (best_us >= 0. && o.bound >= best_us) break;
        if ((dealt += o.dealt) > kMaxDealt) {
            if (best_us < 0.) best_us = o.bound;
            break;
        }
        steps.clear();
        const int n_chunks = (T + o.cb * 32 - 1) / (o.cb * 32);
        for (int ch = 0; ch < n_chunks; ++ch)
            for (int t = 0; t < std::min(n_tiles, (ch + 1) * o.cb / 4); ++t) steps.push_back(dkv_unit_steps(t, q_end[t], ch, o.cb));
        free_at.assign(cus, (float)(other_us / cus));
        float finish = 0.f;
        auto deal = [&](float us) {   // to the compute unit that frees up first: the root of a heap, which then sinks
            const float t = free_at[0] + us;
            finish = std::max(finish, t);
            int i = 0;
            for (int c = 1; c < cus; c = 2 * i + 1) {
                if (c + 1 < cus && free_at[c + 1] < free_at[c]) ++c;
                if (!(free_at[c] < t)) break;
                free_at[i] = free_at[c];
                i = c;
            }
            free_at[i] = t;
        };
        const int n = (int)steps.size();
        for_units_of_an_xcd(a.hkv, (int64_t)n * o.ns, [&](int64_t u) {
            const int sp = (int)u / n, n2 = steps[(int)u % n];
            deal(n2 > 0 ? (float)((n_jh - sp + o.ns - 1) / o.ns * n2) * kStepUs + kUnitUs : kEmptyUs);
        });
        for (float us : dq) deal(us);
        for (int i = 0; i < n_later; ++i) deal(later_us);
        if (best_us < 0. || finish + o.flush < best_us) {
            best_us = finish + o.flush;
            best = DkvPlan{o.cb, o.ns};
        }
    }
    return BwdDeal{best, best.n_split > 0 ? best_us : -1.};
}

inline DkvPlan plan_dkv_split(const CallShape& a, int head_dim, int n_cu, double other_us = 0.) {
    const float stream = head_dim == 64 ? 0.6f : 1.f;
    return deal_bwd(a, n_cu, other_us, BwdPrices{1.9f * stream, 13.f, 1.f, 5.f * stream, 1.7f * stream, 8.f, 0.f, 0.f, 0.f}, 256, false).plan;
}

// Where the later blocks' dK, dV of the 16-bit backward are made: in the preprocess launch, together with D (true), or as the
// last workgroups of the streaming launch, whose tail they fill while the preprocess only makes D.  The second
// way reads dO once more and is the better one (forward and backward, 256 ... 8192 tokens in one document or many, one
// step a call: 2 to 27 % up to 2048 tokens, 0 to 2 % beyond; all steps in one call, up to 512 tokens: 3 to 40 %)
// except for sweeps over many (step, head) pairs that also fill the device: there one unit is as long as a
// dQ tile and leaves a tail of its own (all steps, 7 to 12 of 32/8 heads: 0 to 2.7 % slower from 1024 tokens on).
inline bool diag_blocks_apart(const CallShape* calls, int n_calls, int head_dim, int n_cu) {
    int64_t all = 0;
    for (int i = 0; i < n_calls; ++i) {
        const CallShape& a = calls[i];
        const int64_t n_pairs = (int64_t)a.n_steps * a.G;
        const int64_t units = (int64_t)a.T * a.hkv * head_dim / (8 * 512) * diag_passes(a, kDiagRegBlocks);   // 512 threads, 8 elements each
        if (n_pairs > 16 && a.step_begin + a.n_steps > 1) all += units * n_pairs;
    }
    return all > 20 * (int64_t)n_cu;
}
inline bool diag_blocks_apart(const CallShape& a, int head_dim, int n_cu) { return diag_blocks_apart(&a, 1, head_dim, n_cu); }

// What a slice takes of one XCD's compute units by the model above, us in all: its documents one by one, half of each key
// tile's rows below the diagonal.
inline double bwd_slice_us(const CallShape& a, int head_dim) {
    const double stream = head_dim == 64 ? 0.6 : 1., pairs = (double)a.n_steps * a.G;
    double units = 0., steps = 0., keys = 0.;
    for (int r = 0; r < a.n_docs; ++r) {
        const double n = a.cu_host[r + 1] - a.cu_host[r], tiles = n / 128. + 0.5;
        units += tiles * (n / 2048. + 1.);
        steps += tiles * (n / 128. + 0.5);
        keys += (n / 256. + 0.5) * (n / 256. + 1.);
    }
    return a.hkv / 8. * (steps * pairs * 1.9 * stream + units * 13. + keys * pairs * 5. * stream +
                         ((double)a.T / 256. + 1.) * pairs * (8. + 1.7 * stream * (a.step_begin + 0.5 * (a.n_steps - 1))));
}

// Short launches of one slice: prices of their own, and dQ tiles of 256 rows or of 128 whose keys two halves of the workgroup share
// (two key groups: half as long a chain of key tiles and diagonal keys).  A launch that leaves compute units idle, or ends with
// a few long tiles, gains from them; the work of all is less without.
// The prices are fitted to all splits (chunk size, list split up to 24, key groups) of 2097 launches of up to 1600 dQ tiles: 64 ...
// 4096 tokens in one document or many, seven head geometries, one step a call (the first to the ninth) or two to eight at once.
// Whole backward over the best split of each, in the mean, head_dim 128 / 64: 1.023 / 1.027; with the prices above and one key group 1.128 / 1.105,
// with the best split of one key group 1.047 / 1.038.  The best one by these prices was 0.95 of the split by the prices above in the mean,
// and more than 3 % slower in seven launches of a hundred, mostly with several steps (fewer rounds of longer units, and closer to each other).
// There the split by the prices above stays unless two key groups, or with head_dim 128 another split with one, are estimated at 0.91
// of it.  1500 other launches, timed in graphs, take 0.938 / 0.959 of the time by the prices above in the mean (head_dim 128 / 64);
// 20 and 23 in a thousand are more than 3 % slower, 1.17 and 1.15 at most.
// 1320 tokens, 8/1 heads of 64, the last of eight steps, forward and backward 63.9 -> 50.9 us; 493 tokens, 12/2 heads, five steps one
// by one 200 -> 179.  Launches of several slices keep the prices above (1154 tokens in eight slices: 3 % slower with these).
constexpr int kShortLaunchTiles = 1600, kShortLaunchTokens = 4096;
inline BwdPrices short_launch_prices(int head_dim, int dq_groups) {
    if (head_dim == 64)
        return dq_groups == 2 ? BwdPrices{1.19f, 8.7f, 1.05f, 1.15f, 0.30f, 9.6f, 7.2f, 0.08f, 0.3f} : BwdPrices{1.19f, 8.7f, 1.05f, 2.65f, 0.85f, 5.1f, 7.2f, 0.08f, 0.3f};
    return dq_groups == 2 ? BwdPrices{1.59f, 11.5f, 2.5f, 2.17f, 0.81f, 8.7f, 8.4f, 0.33f, 3.1f} : BwdPrices{1.59f, 11.5f, 2.5f, 4.16f, 1.64f, 5.5f, 8.4f, 0.33f, 3.1f};
}
struct ShortPlan {
    int dq_groups;   // 0: not a short launch
    DkvPlan kv;
};
inline ShortPlan plan_short_bwd(const CallShape& a, int head_dim, int n_cu) {
    ShortPlan best{0, {}};
    if (a.T > kShortLaunchTokens || (int64_t)((a.T + 255) / 256) * a.n_steps * a.G * a.hkv > kShortLaunchTiles) return best;
    const int later_rows = 512 / (head_dim / 8);
    double limit = -1.;
    int64_t most = INT64_MAX;   // workgroups of the launch
    auto workgroups = [&](const DkvPlan& p, int q_rows) {
        const int64_t later = ((int64_t)a.T * a.hkv + later_rows - 1) / later_rows * diag_passes(a, kDiagRegBlocks);
        return later + dkv_units_of(a.T, (a.T + 127) / 128, p.chunk_blocks) * p.n_split * a.hkv + (int64_t)((a.T + q_rows - 1) / q_rows) * a.n_steps * a.G * a.hkv;
    };
    if (a.n_steps > 1) {
        const DkvPlan first = plan_dkv_split(a, head_dim, n_cu);   // the split that another one has to beat
        limit = 0.91 * deal_bwd(a, n_cu, 0., short_launch_prices(head_dim, 1), 256, true, later_rows, -1., &first).us;
        // While it has a compute unit for every workgroup, so has the other one: a second round starts when all of the first one end,
        // which the prices do not tell (666 tokens, 8/1 heads, four steps 45 -> 61 us; such launches 1.11 of the time in the mean, with one step 0.86)
        if (workgroups(first, 256) <= n_cu) most = n_cu;
        best = ShortPlan{1, first};
        if (limit < 0.) return best;
    }
    for (int groups = a.n_steps > 1 && head_dim == 64 ? 2 : 1; groups <= 2; ++groups) {
        const BwdDeal d = deal_bwd(a, n_cu, 0., short_launch_prices(head_dim, groups), 256 / groups, true, later_rows, limit);
        if (d.us < 0. || workgroups(d.plan, 256 / groups) > most) continue;
        limit = d.us;
        best = ShortPlan{groups, d.plan};
    }
    return best;
}

// The plans of the slices that share a launch; returns the key groups of its dQ tiles.  They depend on the document structure, the
// steps, the heads and the device, and are kept for the last 64 launches: a batch of more runs of documents than that would push out its own
// entries, and those of every other call, if each slice had one (153 runs of documents of 20 to 200 tokens, 32/8 heads, up to
// seven steps: 0.5 ms of planning in each call with the same batch, 0.07 so, most of it the caller's).
inline int plan_dkv_launch(const CallShape* calls, int n_calls, int head_dim, int n_cu, DkvPlan* plans) {
    struct Key {
        int64_t tokens;
        int n_calls, n_docs, step_begin, n_steps, G, hkv, head_dim, n_cu;   // (documents and steps of all slices together)
        uint64_t hash;
        bool operator==(const Key& o) const {
            return tokens == o.tokens && n_calls == o.n_calls && n_docs == o.n_docs && step_begin == o.step_begin && n_steps == o.n_steps &&
                   G == o.G && hkv == o.hkv && head_dim == o.head_dim && n_cu == o.n_cu && hash == o.hash;
        }
    };
    Key key{0, n_calls, 0, calls[0].step_begin, 0, calls[0].G, calls[0].hkv, head_dim, n_cu, 1469598103934665603ull};
    auto add = [&](int x) { key.hash = (key.hash ^ (uint64_t)(uint32_t)x) * 1099511628211ull; };
    for (int i = 0; i < n_calls; ++i) {
        const CallShape& a = calls[i];
        key.tokens += a.T;
        key.n_docs += a.n_docs;
        key.n_steps += a.n_steps;
        add(a.n_steps);
        for (int r = 0; r <= a.n_docs; ++r) add(a.cu_host[r] - a.cu_base);
    }
    static std::mutex mu;
    struct Made {
        Key key;
        int dq_groups;
        std::vector<DkvPlan> kv;
    };
    static std::vector<Made> cache;
    {
        std::lock_guard<std::mutex> lock(mu);
        for (const Made& e : cache)
            if (e.key == key) {
                std::copy(e.kv.begin(), e.kv.end(), plans);
                return e.dq_groups;
            }
    }
    const ShortPlan one = n_calls == 1 ? plan_short_bwd(calls[0], head_dim, n_cu) : ShortPlan{0, {}};
    const int dq_groups = std::max(1, one.dq_groups);
    if (one.dq_groups > 0) {
        plans[0] = one.kv;
    } else {
        std::vector<double> us(n_calls, 0.);
        double all_us = 0.;
        for (int i = 0; n_calls > 1 && i < n_calls; ++i) all_us += us[i] = bwd_slice_us(calls[i], head_dim);
        for (int i = 0; i < n_calls; ++i) plans[i] = plan_dkv_split(calls[i], head_dim, n_cu, all_us - us[i]);
    }
    Made made{key, dq_groups, std::vector<DkvPlan>(plans, plans + n_calls)};
    std::lock_guard<std::mutex> lock(mu);
    if (cache.size() >= 64) cache.erase(cache.begin());
    cache.push_back(std::move(made));
    return dq_groups;
}

// Whether a slice has a backward launch of its own.  Slices that share a launch fill each other's tails and save launches, but
// workgroups that start one by one, as others end, no longer stream the same Q / dO rows together.  So a slice that takes the
// device more than a millisecond is alone (forward and backward, 16384 tokens in nine slices of up to twelve steps,
// 32/8 heads: 12133 us with a launch per slice, 11965 so, 12300 at 0.2 ms, 12030 at 2; all in one 12450; 8192
// tokens in documents of 100 to 500, up to seven steps 2171 -> 1461, 8/2 heads of 64 1321 -> 471 at any of these lines).
inline bool bwd_slice_alone(const CallShape& a, int head_dim, int n_cu) {
    return bwd_slice_us(a, head_dim) > 1000. * std::max(1, n_cu / 8);
}

// The fp32 backward with operands straight from memory (ttt_bwd_f32_kernel): ways to split the (step, head, query block) items of a
// 32-key unit.  Estimated as the longest chain of a wave, or the work of all over the compute units and 0.15 of that chain (how
// unevenly they end), by prices (us) fitted to all splits of the 2863 launches of fwd_f32_direct: 1.013 / 1.011 of the best split in the mean
// (head_dim 64 / 128).  Slices that share a launch count each other's dQ tiles and later blocks as work.
struct F32BwdPrices {
    double unit, step, tile, group, diag;                        // the chains: a unit and four of its items, a dQ tile, four of its key blocks, a diagonal key
    double later, unit_work, step_work, tile_work, group_work, diag_work;
};
inline F32BwdPrices f32_bwd_prices(int head_dim) {
    return head_dim == 64 ? F32BwdPrices{1.35, 5.1, 1.45, 3.75, 0.31, 0.91, 4.9, 0.25, 2.9, 8.05, 0.78}
                          : F32BwdPrices{0.95, 11.5, 0.82, 9.3, 0.68, 2.0, 8.8, 0.1, 1.1, 18.2, 1.8};
}
// per key tile of 32: the query blocks that see it
inline std::vector<int> f32_query_blocks(const CallShape& a) {
    std::vector<int> n((a.T + 31) / 32);
    int doc = 0;
    for (int t = 0; t < (int)n.size(); ++t) {
        const int last = std::min(t * 32 + 31, a.T - 1);
        while (doc + 1 < a.n_docs && a.cu_host[doc + 1] - a.cu_base <= last) ++doc;
        n[t] = (a.cu_host[doc + 1] - a.cu_base - 1) / 32 - t + 1;
    }
    return n;
}
inline double f32_bwd_dq_work(const CallShape& a, int head_dim, const KeyCount& n) {
    const F32BwdPrices p = f32_bwd_prices(head_dim);
    const double heads = (double)a.hkv * a.G * a.n_steps, later = a.step_begin + a.n_steps > 1 ? (double)a.T * a.hkv * head_dim / 2048. * a.n_steps * a.G : 0.;
    return heads * (n.tiles * (p.tile_work + p.diag_work * (a.step_begin + 0.5 * (a.n_steps - 1))) + n.groups * p.group_work) + later * p.later;
}
inline int f32_direct_split(const CallShape& a, int head_dim, int n_cu, const KeyCount& keys, double dq_work) {
    const F32BwdPrices p = f32_bwd_prices(head_dim);
    const std::vector<int> blocks = f32_query_blocks(a);
    const int64_t n_jh = (int64_t)a.n_steps * a.G;
    const double dq_chain = p.tile + p.group * keys.longest + p.diag * (a.step_begin + a.n_steps - 1);
    int best = 1;
    double best_us = -1.;
    for (int ns : {1, 2, 3, 4, 6, 8, 12, 16, 24}) {
        if (ns > 4 * n_jh || (int64_t)blocks.size() * ns * a.hkv > 0x7fffffff) break;
        int64_t steps = 0, longest = 0;
        for (int b : blocks) {
            const int64_t s = (n_jh * b + 4 * ns - 1) / (4 * ns);
            steps += s;
            longest = std::max(longest, s);
        }
        const double work = ((double)blocks.size() * p.unit_work + steps * p.step_work) * ns * a.hkv + dq_work;
        const double chain = std::max(p.unit + p.step * longest, dq_chain), us = std::max(chain, work / n_cu + 0.15 * chain);
        if (best_us < 0. || us < best_us) {
            best_us = us;
            best = ns;
        }
    }
    return best;
}
inline void plan_dkv_f32_direct(const CallShape* calls, int n_calls, int head_dim, int n_cu, int* n_split) {
    std::vector<KeyCount> keys(n_calls);
    double dq_work = 0.;
    for (int i = 0; i < n_calls; ++i) {
        keys[i] = count_keys(calls[i], 32, 32, 4);
        dq_work += f32_bwd_dq_work(calls[i], head_dim, keys[i]);
    }
    for (int i = 0; i < n_calls; ++i) n_split[i] = f32_direct_split(calls[i], head_dim, n_cu, keys[i], dq_work);
}
// Over 1100 launches of 150 ... 16384 tokens operands from memory take 0.863 / 0.855 of the time of tiles through LDS
// (ttt_bwd_main_f32_kernel) in the mean (head_dim 64 / 128; 444 tokens, 8/2 heads of 128, the last of seven steps 129 -> 63 us), but tiles are
//  - 5 to 13 % faster with head_dim 128, 512 tokens or more in a document and work for many rounds of the device (2000 tokens, 32/8 heads,
//    two steps 2391 against 2610 us);
//  - 3 to 14 % faster where a unit of 32 keys has one (step, head) pair and diagonal keys beside, and there are many units: few
//    items share what a unit costs of its own (head_dim 64, 16/16 heads, a later step: 7658 tokens in documents of 114 in the mean 363 against
//    394 us; with documents of 3000 and more the items of a unit are many, and 0.98).
// Elsewhere 20 of the launches are more than 3 % slower than with tiles, 1.15 at most.
// q_st, kv_st: elements from row to row; the 32 rows of a block are told apart by 32-bit byte offsets.
inline bool bwd_f32_direct(const CallShape* calls, int n_calls, int head_dim, int64_t q_st, int64_t kv_st) {
    if (std::max(q_st, kv_st) >= (int64_t)1 << 25) return false;
    int64_t tiles = 0;
    int longest = 0;
    bool one_pair = calls[0].step_begin > 0;
    for (int i = 0; i < n_calls; ++i) {
        const CallShape& a = calls[i];
        tiles += (int64_t)((a.T + 31) / 32) * a.hkv * a.G * a.n_steps;
        one_pair = one_pair && a.G * a.n_steps == 1;
        for (int r = 0; r < a.n_docs; ++r) longest = std::max(longest, a.cu_host[r + 1] - a.cu_host[r]);
    }
    if (one_pair && tiles >= 800 && (head_dim == 128 || longest < 2500)) return false;
    return head_dim == 64 || tiles < 1500 || longest < 512;
}

// The fp32 backward with tiles in LDS: ways to split the (step, head) list of a 128-key tile.
inline int plan_dkv_split_f32(const CallShape& a) {
    const int n_jh = a.n_steps * a.G, n_tiles = (a.T + 127) / 128;
    int n_split = 1;
    while (n_split < n_jh && (int64_t)n_tiles * a.hkv * n_split < 2048) ++n_split;
    return n_split;
}

// ------------------------------------------------------------------------------------------------
// Projections
// ------------------------------------------------------------------------------------------------
// The tiles a call can be cut into, and what they were measured to take (us; sweeps over 16 to 8192 tokens, hidden_in
// 64 to 8192, 2048 to 9216 features): `round` once per round of the device (first copies, epilogue), and per
// 64-column slice `t1` with one workgroup on every compute unit, `lo` in the limit of few workgroups (copies and
// clock are shared), and `t2` with two side by side on one unit.  With weights that are in no cache model and measurement
// differ by 5 % (256 x 256) to 15 % (64 x 64; rms over 120 shapes).
struct QkvTile {
    int mt, nt, per_cu;
    int max_group;     // token tiles of one feature tile that are dealt to an XCD together, at most
    bool by_xcd;       // long workgroups, one to a compute unit: the XCD that gets the most tiles sets the rounds
    double round, lo, t1, t2;
};
constexpr QkvTile kQkvTiles[] = {
    {256, 256, 1, 4, true, 8., 0.95, 1.55, 0.},
    {128, 128, 2, 8, false, 5., 0.57, 0.57, 1.03},
    {128, 128, 1, 8, true, 4., 0.44, 0.55, 0.},
    {128, 64, 1, 8, false, 3., 0.30, 0.37, 0.},
    {64, 64, 2, 8, false, 3., 0.18, 0.18, 0.36},
    {64, 32, 2, 8, false, 2., 0.17, 0.17, 0.28},
    {32, 32, 2, 8, false, 2., 0.14, 0.14, 0.22},
};
constexpr int kQkvTileKinds = sizeof(kQkvTiles) / sizeof(kQkvTiles[0]);
constexpr double kQkvLaunchUs = 3.;

// Tiles of the XCD that gets the most: groups of m_per token tiles (the last of a feature tile is smaller) go to the eight
// XCDs in turn.
inline int64_t qkv_xcd_tiles(int64_t m, int64_t n, int m_per) {
    const int64_t groups = (m + m_per - 1) / m_per, most = (groups * n + 7) / 8;
    // an odd number of groups brings every XCD its share of the smaller ones
    return most * m_per - (groups % 2 ? most / groups * (groups * m_per - m) : 0);
}

// How many token tiles go together: as many as the kind allows in equal groups; fewer of the largest tiles where that saves
// a round of the device (253 of them in groups of four are 36 on one XCD of 32 compute units: 2772 tokens, hidden_in 7040,
// 5888 features took two rounds for one).  Groups without a remainder only: the empty workgroups of the others take a
// compute unit each before the last tiles of an XCD get one (2283 tokens, hidden_in 2752, 6912 features, 243 tiles: groups
// of three, 33 on one XCD, 131 us, of two 142, one by one 87).  Smaller tiles lose more by sharing less of an L2 (539 tokens, hidden_in 2304,
// 7168 features 39 us in groups of five, 47 in groups of three).
inline int qkv_group(const QkvTile& v, int64_t m, int64_t n, int n_cu) {
    const int64_t slots = std::max(1, n_cu / 8);
    auto rounds = [&](int per) { return (qkv_xcd_tiles(m, n, per) + slots - 1) / slots; };
    const int64_t groups = (m + v.max_group - 1) / v.max_group;
    int best = (int)((m + groups - 1) / groups);
    if (v.mt == 256)
        for (int per = best - 1; per >= 1; --per)
            if (m % per == 0 && rounds(per) < rounds(best)) best = per;
    return best;
}

// estimated time of m x n tiles: full rounds of the device and a last one, as full as it is
inline double qkv_cost(const QkvTile& v, int64_t m, int64_t n, int n_cu, int slices) {
    const int64_t slots = (int64_t)n_cu * v.per_cu;
    const int64_t tiles = v.by_xcd ? 8 * qkv_xcd_tiles(m, n, qkv_group(v, m, n, n_cu)) : m * n, rest = tiles % slots;
    const double full = v.round + slices * (v.per_cu == 2 ? v.t2 : v.t1);
    double us = kQkvLaunchUs + (double)(tiles / slots) * full;
    if (rest > n_cu) us += full;
    else if (rest > 0) us += v.round + slices * (v.lo + (v.t1 - v.lo) * (double)rest / (double)n_cu);
    return us;
}

// One kind of tile for all features, or the full rounds of a large kind and the rest of the features with
// another, whichever is estimated shortest: 4096 tokens x 6144 features are 16 x 24 of the largest tiles =
// one and a half rounds of 256 compute units (371 us at hidden_in 8192), or 16 x 16 of them and 32 x 16 of
// 128 x 128, two to a unit (356 us).  largest_fits: the largest kind may be used.
struct QkvPlan {
    int first, second;   // kinds (places in kQkvTiles); second = -1: one launch
    int f_first;         // features of the first launch
};

inline QkvPlan plan_qkv(int64_t tokens, int hidden_in, int features, bool largest_fits, int n_cu) {
    const int slices = hidden_in / 64, kinds = largest_fits ? 0 : 1;
    auto row_tiles = [&](const QkvTile& t) { return (tokens + t.mt - 1) / t.mt; };
    auto cost = [&](const QkvTile& t, int f) { return qkv_cost(t, row_tiles(t), (f + t.nt - 1) / t.nt, n_cu, slices); };
    QkvPlan plan{-1, -1, features};
    double best = 0.;
    for (int t = kinds; t < kQkvTileKinds; ++t) {
        const double c = cost(kQkvTiles[t], features);
        if (plan.first < 0 || c < best) {
            best = c;
            plan.first = t;
        }
    }
    for (int t = kinds; t < 2; ++t) {
        const QkvTile& large = kQkvTiles[t];
        const int64_t slots = (int64_t)n_cu * large.per_cu, m = row_tiles(large);
        const int64_t rounds = m * ((features + large.nt - 1) / large.nt) / slots;
        int64_t n = rounds * slots / m;
        while (n > 0 && qkv_xcd_tiles(m, n, qkv_group(large, m, n, n_cu)) > rounds * slots / 8) --n;   // the fullest XCD, too
        const int64_t f = n * large.nt;
        if (f <= 0 || f >= features) continue;
        const double head = cost(large, (int)f);
        for (int u = kinds; u < kQkvTileKinds; ++u) {
            if (u == t) continue;   // two launches of one kind gain nothing (6322 tokens, hidden_in 5376, 7040 features 495 us, 507)
            const double c = head + cost(kQkvTiles[u], features - (int)f);
            if (c < best) {
                best = c;
                plan = QkvPlan{t, u, (int)f};
            }
        }
    }
    return plan;
}

}  // namespace ttt
