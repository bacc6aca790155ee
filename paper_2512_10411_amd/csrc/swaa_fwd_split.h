// Split keys of the pipelined forward kernel: the plan, and what a workgroup computes.
//
// A chunk of new tokens against a long cache, or single generated tokens in a serving batch, gives
// the forward kernel few row tiles with many keys each: 512 rows on 32 heads are 128 workgroups of
// a chip that runs 512 at once, and one generated token on a 12k-token cache is 375 halves of 32
// keys in a row for one workgroup while the others are long done.  The tiles of a sequence are then
// cut along the keys into n workgroups, each of which leaves its unnormalised O, its softmax
// reference and its row sums in the workspace, and swaa_fwd_merge_kernel adds them up.
//
// How many splits each sequence gets follows from a cost model in units of one half (the time a
// workgroup needs for 32 keys with a second one on its compute unit, 0.83 us measured):
//   * 64 candidates for the longest split, L = h_max / 1 .. h_max / 64 (at least kSplitMinHalves),
//     one per lane; a sequence whose tiles visit h halves gets ceil(h / L) splits;
//   * m = (total + start-up) / 512 is the time of a chip kept full.  A unit (workgroup) alone on
//     its compute unit runs 1 / kSplitAloneRate as fast: up to 256 units all of them are alone, above
//     the longest one shares its unit for about m and is alone for the rest;
//   * above 512 units the chip also works through the total, kSplitFull slower than m says, and the
//     last units run out a share of an average one late;
//   * sequences of one or two row tiles (generated tokens) read their keys for nobody else: HBM
//     delivers 350 halves (16 KiB each) in the time of one, and 0.3 of the shorter of the two times shows;
//   * where a sequence's rows fit one column tile (swaa_fwd_few_rows.h) the four waves share the keys: a half
//     costs kSplitFewRate, a workgroup kSplitFewStart outside its loop;
//   * a workgroup costs kSplitStart halves outside its loop, and splitting at all the merge kernel
//     (kSplitMerge) and the traffic of the partial results (64 KiB per unit).
// The constants are a fit to 70 batches of 1-34 sequences (100-2048 new rows beside 0-31 generated
// tokens, caches of 2-30k tokens, 8-40 heads) at 4-11 plans each: the plan it picks costs 1.1-1.7 % more than
// the best of them on average (3.2 % with the first model, which took the longest split for the time
// below 512 units, did not know HBM's rate and split batches that fill the chip).  The terms of few rows, and of
// HBM beside them, are a fit to 230 batches of 7 or 31 generated tokens beside chunks at 81 plans each.  Over 500 other
// batches (3-60 sequences of 1-4 rows beside 0-3 chunks, 8-40 heads on 2-8) the plan is 1.7 % behind the best of its candidates
// on average, 30 % the worst; against row tiles they take 0.837 of the time, ten more than 1.02 (the worst 1.12).
// The lengths of a packed batch are known on the device only: there every workgroup works the plan
// out for itself (batches of at most 64 sequences: one per lane).  Measured, binary16 and pages of
// 16 tokens, 32 heads on 8: 512 rows on 24k tokens, full attention, 364 -> 207 us (four splits,
// 196 + 9 us; 128 workgroups before); 23 generated tokens on caches of 1-12k tokens beside a chunk
// of 999 rows on a 2k window 213 -> 139 us in row tiles, 118 with the few rows of a token in one column tile.
// Calls that the plan leaves whole on the host (prompts on themselves, short windows, chunks that
// fill the chip) launch the same kernels as without a workspace: the split kernel takes about 4 us more
// for the same plan (the plan itself, also in the workgroups that it then has no work for, and a merge without
// work: 31 generated tokens on 3k tokens beside a chunk of 256 rows, 8 heads on 8, 77.5 us without a workspace, 81.5
// with one, 80.6 since the launch follows a closer bound and the plan's sums no longer cross LDS).
// So do batches of chunks with little to gain (whole_batch), if the number of packed rows shows on the
// host that they are that; the device follows the same rule, so that the results do not depend on
// whether the caller states that number.
#ifndef SWAA_FWD_SPLIT_H_
#define SWAA_FWD_SPLIT_H_

#include "swaa_common.h"

namespace swaa {

constexpr int kSplitMaxBatch = 64;   // one sequence per lane
constexpr int kSplitMinHalves = 16;  // no split shorter than this many halves
constexpr int kSplitUnits = 1024;    // most partial results a packed batch may leave (64 KiB each)
constexpr float kSplitResident = 512.f, kSplitAlone = 256.f, kSplitAloneRate = 0.65f;
constexpr float kSplitStart = 8.f, kSplitMerge = 8.f, kSplitTraffic = 0.015f, kSplitFull = 1.1f, kSplitTail = 0.5f;
constexpr float kSplitMemory = 1.f / 350.f, kSplitOverlap = 0.3f;
constexpr float kSplitFewRate = 0.65f, kSplitFewStart = 12.f;  // a workgroup of few rows (swaa_fwd_few_rows.h)

// Halves a row tile at positions [a, b] visits (as the kernel's prologue counts them).
__host__ __device__ inline int tile_halves(int a, int b, int W, int S) {
    const int band_lo = a - W + 1 > 0 ? a - W + 1 : 0;
    const int lo = band_lo >> 5, hi = b >> 5;
    const int sink_keys = S < band_lo ? S : band_lo;
    const int sinks = (sink_keys + 31) >> 5;
    return (sinks < lo ? sinks : lo) + hi - lo + 1;
}

// A sequence whose rows fit one column tile of a KV head: a single tile, see swaa_fwd_few_rows.h.
__host__ __device__ inline bool few_rows(const FwdParams &p, int nq) { return p.G * nq <= 32; }

// What a sequence brings to the plan.
struct SplitSeq {
    int tiles;    // row tiles per (sequence, KV head)
    int halves;   // visited by the last, longest of them
    int cost;     // what that takes, in halves of a row tile
    int average;  // the same of a tile on average
    float start;  // what a workgroup costs outside its loop
    bool whole;   // never split: prompt and generated rows mixed, whose tiles differ too much
};
__host__ __device__ inline SplitSeq split_seq(const FwdParams &p, int nq, int nk, int n_prompt) {
    SplitSeq s{0, 0, 0, 0, kSplitStart, true};
    if (nq <= 0) return s;
    constexpr int r1 = kFwdWgRows, r2 = r1 / 2, r4 = r1 / 4;  // (the rows of p's plan; known here, so no divisions)
    s.tiles = p.n4 * ((nq + r4 - 1) / r4) + p.has2 * ((nq + r2 - 1) / r2) + p.has1 * ((nq + r1 - 1) / r1);
    const int r = p.n4 ? r4 : p.has2 ? r2 : r1;
    const int first = nk - nq;
    const bool some = n_prompt < nk, all = n_prompt <= first;  // generated rows
    if (few_rows(p, nq)) {
        s.tiles = 1;
        s.halves = tile_halves(first, nk - 1, some ? nk : p.W, p.S);
        s.cost = s.average = (int)((float)s.halves * kSplitFewRate) + 1;
        s.start = kSplitFewStart;
        s.whole = false;
        return s;
    }
    s.halves = s.cost = tile_halves(nk - (r < nq ? r : nq), nk - 1, some ? nk : p.W, p.S);
    const int h0 = tile_halves(first, first + (r < nq ? r : nq) - 1, all ? nk : p.W, p.S);
    s.average = (h0 + s.halves + 1) / 2;
    s.whole = some && !all;
    return s;
}

// Candidate i for the longest split, h_max / (i + 1) rounded up; rcp: about 1 / (i + 1).  (An approximate quotient
// will do: every workgroup comes to the same, and nobody else needs it.  Candidate 0 is the exception: it is the one
// plan that splits nothing, and so fits every workspace.)
__host__ __device__ inline int split_length(int h_max, int i, float rcp) {
    const int L = i == 0 ? h_max : (int)((float)(h_max + i) * rcp);
    return L > kSplitMinHalves ? L : kSplitMinHalves;
}

// Splits of a sequence whose tiles visit h halves, for splits of at most L; rcp = 1 / L.  (Rounded
// down instead of up where the product comes out just below a whole number: no matter, the same
// expression is used for the plan and for the work list.)
__host__ __device__ inline int split_count(int h, int L, float rcp) {
    const int n = (int)((float)(h + L - 1) * rcp);
    return n < 1 ? 1 : n;
}
// Predicted time of a plan, in halves.  starts: of all units together; longest: with its own.  memory: halves read
// from HBM by sequences of one or two row tiles, over all KV heads.
__host__ __device__ inline float split_time(float units, float split_units, float starts, float longest, float total, float memory) {
    const float l = longest, m = (total + starts) * (1.f / kSplitResident);
    float t = kSplitAloneRate * l;
    if (units > kSplitAlone) t += (1.f - kSplitAloneRate) * (l < m ? l : m);
    if (units > kSplitResident) {
        const float full = kSplitFull * m + kSplitTail * total / units;
        t = t > full ? t : full;
    }
    const float read = memory * kSplitMemory;
    t = t > read ? t + kSplitOverlap * read : read + kSplitOverlap * t;
    return split_units > 0.f ? t + kSplitMerge + kSplitTraffic * split_units : t;
}

// A batch in which every sequence brings at least `least` rows, with at least `units` row tiles (times KV heads):
// stays whole where the split kernel does not win its overhead back.  From 64 rows on a sequence is
// taken for a chunk of a prompt, whose rows see the window.  The more tiles there are, the longer the windows
// (h halves) for which that holds; from 400 tiles on there are enough for any.  Measured, whole / as planned (us;
// 32 heads on 8, binary16, pages of 16; bfloat16, pages of 64 and contiguous keys alike):
//    64 tiles   window 1250 28.6 / 29.3   1500 33.2 / 30.0   2048 38.7 / 31.6
//    96         window 1250 28.8 / 32.4   1500 33.2 / 34.3   1750 36.7 / 36.1   2500 47.6 / 41.0
//   128         window 1500 33.2 / 36.7   2048 39.1 / 40.1   2500 47.7 / 43.9   3000 53.4 / 46.2
//   160         window 2048 39.6 / 44.4   2500 48.0 / 49.1   3000 54.3 / 52.8   4096 68.6 / 61.5
//   192         window 2500 50.4 / 52.9   3000 57.8 / 61.7   4096 74.9 / 74.9   6000 104 / 97.7
//   240         window 3000 58.2 / 60.9   4096 76.0 / 82.2   6000 109 / 110     8192 144 / 141
//   304         window 3000 84.2 / 88.4   8192 201 / 206     24k, full attention 546 / 476
// Groups of fewer than four heads share less, and their tiles of 64 or 128 positions take longer (8 heads on 8,
// 112 tiles: window 1250 35.6 / 35.2, 1500 38.8 / 36.1).  Fewer tiles gain on every window that is long enough to be
// split (16 tiles: window 700 20.7 / 23.6, 1250 28.4 / 24.0).  (These are chunks on 12k tokens.)  With full
// attention, and on caches shorter than a long window, the tiles differ, by sequence and along its rows, and splits
// even them out: three chunks of 735 rows, 276 tiles, on 3-6k tokens 113 / 109; two of 339, 224 tiles, window 4096, on
// 3-10k tokens 81.0 / 75.5.  So the rule ends at windows of 3000.
__host__ __device__ inline bool whole_batch(const FwdParams &p, int least, int units) {
    if (least < 64) return false;
    if (units >= 400 && p.Hkv * split_seq(p, least, p.Nk, p.Nk).tiles >= 64) return true;
    const int h = tile_halves(p.Nk - 32, p.Nk - 1, p.W, p.S);
    if (units < 64) return h <= 2 * kSplitMinHalves;
    if (p.n4 == 0 || p.W >= p.Nk) return h <= (units < 160 ? 42 : 72);
    return h <= (units < 160 ? 42 + (units - 64) * 9 / 20 : 100);
}
// Row tiles (times KV heads) of a batch of so many rows: no fewer than one sequence with all of them has.
__host__ __device__ inline int least_units(const FwdParams &p, int rows) { return p.Hkv * split_seq(p, rows, rows, 0).tiles; }

// First of a sequence's units that die xcd takes (up to the next die's): an eighth of them.  Where they do not divide by
// eight, which dies get one more follows from the units of the sequences ahead, so that over the batch all get as
// many.  (Chunks of a rounded-up eighth left the last dies with nothing in every sequence: 64 generated tokens on 6000
// keys, four KV heads, took 204 us with their units on four dies, and 135 on eight.)
__host__ __device__ inline unsigned die_share(unsigned units, unsigned ahead, unsigned xcd) {
    return (xcd * units + ahead % kXcds) / kXcds;
}

// Which unit of a die's list is workgroup `rank`: the at-th of few rows, or of row tiles?  Row tiles compute and few rows
// read, so that they take turns and neither is left alone with the chip -- the other way round every 32 ranks,
// so that the two workgroups of a compute unit, ranks r and r + 32 (of the first 64), are one of each.  When less than 32
// of a kind are left (or were there), first what there is of it: turns to the end would put two row tiles
// on a compute unit while few rows have others to themselves (31 tokens beside two chunks of 1588 rows, 8 heads on 8, 184 us
// in row tiles for all; 205 with turns to the end, 187 so).  Against row tiles, 280 batches: 15.7 % faster on average,
// six slower by more than 2 %; with turns to the end 14.7 % and 14.
__host__ __device__ inline void unit_of_rank(unsigned rank, unsigned n_rows, unsigned n_few, bool &few, unsigned &at) {
    const unsigned turns = n_rows < n_few ? n_rows : n_few, paired = turns / 32 * 64;
    if (rank < paired) {
        few = ((rank ^ (rank >> 5)) & 1u) != 0;
        at = rank >> 1;
        return;
    }
    const unsigned done = paired / 2, rel = rank - paired, first = turns - done;
    few = (rel < first) == (n_few <= n_rows);
    at = rel < first ? done + rel : rank - turns;
}

// A batch of few rows on whole keys, `units` (times KV heads) of about one length: do row tiles, which are as many where the
// heads of a group share one, run them faster?  Two workgroups of few rows on a compute unit read no more than one alone
// does (32 KB/us), two of row tiles 37, and from 257 units on the doubled ones are the time, until all are.  Row tiles / few
// rows (us; 32 heads on 8, bfloat16, caches that no cache of the chip has seen; pages of 16 and other groups alike):
//    units    256          272          288          320          352          384          448          512
//    1504     41.0 / 39.0  46.2 / 52.2  47.5 / 52.8  50.5 / 54.2  53.8 / 56.3  56.6 / 57.9  64.1 / 63.8  72.3 / 72.1
//    4000     96.9 / 96.5   110 / 130    114 / 132    123 / 136    131 / 141    140 / 145    161 / 162    183 / 185
//    16000     349 / 354    407 / 491    423 / 497    455 / 507    490 / 523    522 / 543    602 / 608    687 / 690
// In drawn batches the two are even from 377 units on, and in any number where the lengths differ by a factor of four, so
// that the longest ones are the time (272 units on 2-9k keys: 0.97).
__host__ __device__ inline bool few_in_row_tiles(const FwdParams &p, unsigned units) {
    return p.n4 + p.has2 + p.has1 == 1 && units > 256 && units <= 376;
}

// Does such a batch stay whole because its units have a compute unit each, and most of those have one?  Splits share
// compute units, which read no more for it; the model, whose row tiles do, splits from about 13000 keys on.  Whole / the best
// of two to eight splits / row tiles (us; 13440 keys, 16 heads on 4; 2500 to 24000 keys and 32 heads on 8 alike):
//    units    128              144              160              176              192              208              240
//             163 / 158 / 164  171 / 180 / 189  184 / 198 / 207  200 / 217 / 222  219 / 237 / 260  239 / 251 / 267  277 / 285 / 283
// Up to 160 it depends on where the keys lie (144 units on 10270 keys, packed: 160 / 151).
__host__ __device__ inline bool few_stay_whole(unsigned units) { return units > 160 && units <= 256; }

// Is the only sequence of a batch as long as the host's bounds on its lengths (bound_splits), or up to a sixteenth shorter?  Bounds
// may be far above the lengths (a captured graph is launched for the longest cache that it will meet), and the host's split count is
// then too high, or too low where there are fewer rows than it reckons with.  The host's count / the device's plan (us;
// binary16, 32 heads on 8, full attention; rows and keys, of their bounds where those differ):
//    1 row on 600 keys of 32768 24.9 / 12.3   64 on 1000 of 32768 28.1 / 20.4     64 on 16384 of 32768 41.7 / 36.4
//    64 rows of 512 on 32768 keys 114 / 57.4  64 of 512 on 131072 503 / 171       1 on 4000 of 8192 18.8 / 19.7
//    1 on 7936 of 8192 24.1 / 26.7 (the plan's own time in front of the first key)
__host__ __device__ inline bool as_the_bounds_say(const FwdParams &p, int nq, int cost) {
    return nq == p.Nq && cost <= p.bound_cost && 16 * cost >= 15 * p.bound_cost;  // (at most 2^26 halves and one)
}

// One workgroup's share of the keys.
struct SplitItem {
    int n, s;       // the sequence's splits (0: none, and few rows on a row tile all the same), and which of them this is
    unsigned slot;  // partial result (n >= 2)
};

// Sequence `lane` of the batch (0 rows and keys beyond its end): rows, keys, prompt length, and first row along the row axes.
struct SplitLengths {
    int nq, nk, np, q0, k0;
};
__device__ __forceinline__ SplitLengths split_lengths(const FwdParams &p, int lane) {
    // (a lane beyond the batch reads the last sequence's, so that all loads go out together and none waits for a branch)
    const int b = min(lane, p.B - 1);
    int q0 = 0, q1 = p.Nq, k0 = 0, k1 = p.Nk, np = p.P;
    if (p.cu_q) {
        q0 = p.cu_q[b];
        q1 = p.cu_q[b + 1];
    }
    if (p.cu_k) {
        k0 = p.cu_k[b];
        k1 = p.cu_k[b + 1];
    }
    if (p.n_prompts) np = p.n_prompts[b];
    asm volatile("" : "+v"(q0), "+v"(q1), "+v"(k0), "+v"(k1), "+v"(np));
    SplitLengths s{q1 - q0, k1 - k0, max(np, 0), q0, k0};
    s.nq = max(0, min(min(s.nq, p.Nq), s.nk));
    s.nk = min(s.nk, p.Nk);
    s.nq = min(s.nq, s.nk);
    if (lane >= p.B) s.nq = s.nk = s.np = 0;
    return s;
}
// Sequence b of them as seq_geom describes it, without a second trip to memory; false if it has no rows.
__device__ __forceinline__ bool split_geom(const FwdParams &p, const SplitLengths &s, int b, SeqGeom &g) {
    g.nq = (int)wave_read_lane((unsigned)s.nq, b);
    g.nk = (int)wave_read_lane((unsigned)s.nk, b);
    g.n_prompt = (int)wave_read_lane((unsigned)s.np, b);
    g.q_row0 = (int)wave_read_lane((unsigned)s.q0, b);
    g.q_batch = p.cu_q ? 0 : b;
    g.k_row0 = p.block_table ? 0 : (int)wave_read_lane((unsigned)s.k0, b);  // (a paged cache: the offsets only give the lengths)
    g.k_batch = p.cu_k || p.block_table ? 0 : b;
    return g.nq > 0;
}

// Row tile `t` of a (sequence, KV head) pair with nq query rows (the order of decode_work).
__device__ __forceinline__ void split_tile(const FwdParams &p, int nq, unsigned t, WorkItem &w) {
    constexpr unsigned r1 = kFwdWgRows, r2 = r1 / 2, r4 = r1 / 4;
    const unsigned nt4 = ((unsigned)nq + r4 - 1) / r4, nt2 = ((unsigned)nq + r2 - 1) / r2, nt1 = ((unsigned)nq + r1 - 1) / r1;
    if (t < (unsigned)p.n4 * nt4) {
        const unsigned g = t / nt4;
        w.hpb = 4;
        w.h0 = 4 * (int)g;
        w.pt = (int)(nt4 - 1 - (t - g * nt4));
        return;
    }
    t -= (unsigned)p.n4 * nt4;
    if (p.has2 && t < nt2) {
        w.hpb = 2;
        w.h0 = 4 * p.n4;
        w.pt = (int)(nt2 - 1 - t);
        return;
    }
    if (p.has2) t -= nt2;
    w.hpb = 1;
    w.h0 = p.G - 1;
    w.pt = (int)(nt1 - 1 - t);
}

// Sum and largest of x over the 64 lanes (the data-parallel-primitive steps of wave_inclusive_scan).
__device__ __forceinline__ unsigned wave_max(unsigned x) {
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false));
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false));
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false));
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false));
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false));
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false));
    return wave_read_lane(x, 63);
}
__device__ __forceinline__ float wave_sum(float x) {
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x111, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x112, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x114, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x118, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x142, 0xa, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x143, 0xc, 0xf, false));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

// The work list with split keys: sequence after sequence, every sequence's units cut into eight
// contiguous chunks, one per die (die_share); inside a sequence by KV head, then
// split, then row tile, so that the workgroups side by side on a die read the same keys.  scratch:
// 4 KiB of LDS of a workgroup of four waves, free again after the caller's next barrier.
__device__ __forceinline__ bool decode_work_split(const FwdParams &p, uint32_t scratch, WorkItem &w, SplitItem &si, SeqGeom &sg) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned xcd = blockIdx.x % kXcds, rank = blockIdx.x / kXcds;
    const SplitLengths lengths = split_lengths(p, lane);
    const int nq = lengths.nq;
    const SplitSeq me = split_seq(p, nq, lengths.nk, lengths.np);
    const int items = me.tiles * p.Hkv;
    int n = 1;
    bool few_even = true;  // few rows only, of about one length: the average is 0.8 of the longest and more
    if (p.split_keys != 1) {
        n = p.split_keys;  // (-1: one)
    } else if (p.bound_splits > 1 && as_the_bounds_say(p, (int)wave_read_lane((unsigned)nq, 0), (int)wave_read_lane((unsigned)me.cost, 0))) {
        n = p.bound_splits;
    } else {
        // the model's terms of candidate `lane`, summed over the sequences: wave w takes every fourth
        const int splittable = me.whole ? 0 : me.cost;
        int h_max = splittable, rows = nq, least = nq > 0 ? nq : p.Nq;
        float total = (float)items * (float)me.average;
        float memory = me.tiles <= 2 ? (float)(p.Hkv * me.halves) : 0.f;
        h_max = (int)wave_max((unsigned)h_max);
        total = wave_sum(total);
        memory = wave_sum(memory);
        rows = (int)wave_read_lane(wave_inclusive_scan((unsigned)rows), 63);
        least = 0x7fffffff - (int)wave_max((unsigned)(0x7fffffff - least));
        const int L = split_length(h_max, lane, __builtin_amdgcn_rcpf((float)(lane + 1)));
        const float rcp = 1.f / (float)L;
        float units = 0.f, split_units = 0.f, starts = 0.f, longest = 0.f;
        for (int b = wave; b < p.B; b += 4) {
            const int it = __builtin_amdgcn_readlane(items, b), h = __builtin_amdgcn_readlane(me.cost, b);
            const int c = __builtin_amdgcn_readlane(splittable, b) ? split_count(h, L, rcp) : 1;
            const float u = (float)(it * c);
            units += u;
            split_units += c > 1 ? u : 0.f;
            const float start = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(me.start), b));
            starts += u * start;
            longest = fmaxf(longest, it ? (float)h * __builtin_amdgcn_rcpf((float)c) + start : 0.f);
        }
        typedef float __attribute__((address_space(3))) *LdsFloats;
        const LdsFloats mine = (LdsFloats)(uintptr_t)(scratch + (uint32_t)(wave * 1024 + lane * 4));
        mine[0] = units;
        mine[64] = split_units;
        mine[128] = longest;
        mine[192] = starts;
        __syncthreads();
        units = split_units = starts = longest = 0.f;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const LdsFloats o = (LdsFloats)(uintptr_t)(scratch + (uint32_t)(x * 1024 + lane * 4));
            units += o[0];
            split_units += o[64];
            longest = fmaxf(longest, o[128]);
            starts += o[192];
        }
        __syncthreads();  // (the scratch becomes part of a ring)
        const float t = split_units > (float)p.split_cap ? 3.0e38f : split_time(units, split_units, starts, longest, total, memory);
        const float best = __uint_as_float(~wave_max(~__float_as_uint(t)));  // (positive floats order like their bits)
        const int pick = __builtin_ctzll(__ballot(t == best) | (1ull << 63));
        const int Lb = __builtin_amdgcn_readlane(L, pick);
        // (no candidate fits the workspace only if candidate 0 splits as well: caches of 2^27 keys, whose halves
        // split_count can no longer tell apart)
        if (splittable > 0 && best < 3.0e38f && (least < 64 || !whole_batch(p, least, least_units(p, rows)))) n = split_count(me.cost, Lb, 1.f / (float)Lb);
        const float whole_units = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(units), 0));  // (candidate 0's)
        few_even = total >= 0.8f * (float)h_max * whole_units && !__any(!few_rows(p, nq));
        if (few_even && few_stay_whole((unsigned)whole_units)) n = 1;
    }
    if (me.whole || items == 0 || n < 1) n = 1;
    if (blockIdx.x == 0) p.ws_n[lane] = n;  // every lane its sequence's, for the merge kernel
    const unsigned mine = (unsigned)items * (unsigned)n;
    const unsigned slots = n > 1 ? mine : 0u;
    const unsigned slots_incl = wave_inclusive_scan(slots);
    const unsigned ahead = wave_inclusive_scan(mine) - mine;
    const unsigned from = die_share(mine, ahead, xcd), chunk = die_share(mine, ahead, xcd + 1) - from;
    const bool few = few_rows(p, nq);
    const bool in_rows = few_even && few_in_row_tiles(p, wave_read_lane(ahead + mine, 63)) && !__any(n > 1);
    const unsigned incl_rows = wave_inclusive_scan(few ? 0u : chunk), incl_few = wave_inclusive_scan(few ? chunk : 0u);
    const unsigned n_rows = wave_read_lane(incl_rows, 63), n_few = wave_read_lane(incl_few, 63);
    if (rank >= n_rows + n_few) return false;
    bool take_few;
    unsigned at;
    unit_of_rank(rank, n_rows, n_few, take_few, at);
    const unsigned incl = take_few ? incl_few : incl_rows;
    const int b = __popcll(__ballot(incl <= at));  // sequences that end at or before it
    const unsigned base = b ? wave_read_lane(incl, b - 1) : 0u;
    const unsigned tiles = wave_read_lane((unsigned)me.tiles, b);
    const int nq_b = (int)wave_read_lane((unsigned)nq, b);
    unsigned r = wave_read_lane(from, b) + (at - base);
    si.n = (int)wave_read_lane((unsigned)n, b);
    si.slot = (b ? wave_read_lane(slots_incl, b - 1) : 0u) + r;
    w.b = b;
    const unsigned per_head = tiles * (unsigned)si.n;
    w.kvh = (int)(r / per_head);
    r -= (unsigned)w.kvh * per_head;
    si.s = (int)(r / tiles);
    split_tile(p, nq_b, r - (unsigned)si.s * tiles, w);
    if (!split_geom(p, lengths, b, sg)) return false;
    if (in_rows) si.n = 0;  // (said in another field, it cost other batches 1 us: scalar registers move to vector ones)
    return true;
}

}  // namespace swaa

#endif  // SWAA_FWD_SPLIT_H_
