// Decode-shape attention, head dimension 128, gfx950: the Nq newest tokens of a
// sequence attend to a cache of Nk keys and values (paper Sec. 3.1.1: all of
// them under FA Decode; their window plus the sink tokens of Sec. 3.2.1 when
// decoding stays on sliding-window attention).
//
// With a handful of query rows the cache is read once and nothing is reused:
// the bound is HBM bandwidth, and what matters is the number of bytes in flight.
//
//   * The G query heads x Nq rows of one (batch, KV head) pair are the 32
//     columns of an MFMA tile (more rows: more column tiles), so one pass over
//     K and V serves the whole GQA group.  Padding columns cost matrix-core
//     time only, of which there is plenty.
//   * The visited keys are cut into splits; a workgroup is FOUR waves, each with a quarter of the
//     split and a ring of 32-key half tiles (K 8 KiB + V 8 KiB per stage) in LDS of its own,
//     filled by global_load_lds_dwordx4 with whole 256-byte rows per 16 lanes.  No barriers in
//     the loop: a wave waits on its own copies only.  One stage per wave (64 KiB of LDS per
//     workgroup, two to a CU: 128 KiB of copies in flight per CU, 32 MiB over the chip): the
//     registers are the second stage.  Workgroups that compute two column tiles take a two-stage
//     ring, one to a CU.
//   * Short calls are chains of latencies (decode of 682 tokens: 9.5 us as a graph, 1.9 of them each launch's own):
//     arguments in one trip (fetch_args), copies without a product or a clamp per row, one barrier and the valid
//     columns only where the waves' results meet, and a merge that asks for everything it needs at once.  By timestamps
//     in the kernel, us: arguments and plan 1.0 -> 0.4, first copies and Q 1.0 -> 0.7, meeting of the waves
//     1.8 -> 1.0; the kernel 6.4 -> 4.9, the merge 4.2 -> 3.2 (window 8192 of 128k tokens 13.0 -> 10.0 in all).
//   * At the end the four waves' results are added up through LDS; a sequence with one split
//     then writes its output from here, and the merge kernel is not needed.  (Single-wave
//     workgroups, whose every result went through the workspace: 64 sequences x 2k tokens 101 us,
//     now 94; 16 x window 2k 30.2 -> 26.9; 1 x window 8k 15.2 -> 13.2; 64 sequences x 4k tokens with
//     16 new tokens each 230 -> 192; 96 sequences of 0.3-20k tokens 382 -> 338, 5.9 TB/s.)
//   * Per half: all K and V^T operand fragments go from LDS to registers (V^T through transposing
//     reads), the copy of the next half is issued into the stage just emptied, and only then the
//     arithmetic runs: S^T = K Q^T (8 MFMAs), max-based softmax (mask only on halves that are not
//     fully visible), O^T += V^T P^T (8 MFMAs).  The copies thus never wait for arithmetic.  The
//     query rows are loaded from HBM in operand layout and parked in AccVGPRs.
//   * The cache is a contiguous strided tensor or a paged one (a block table of
//     page numbers per sequence, pages of page_size tokens: the layout of a
//     serving engine's cache manager); sequences of a batch may have different
//     cache lengths (seq_lens): the splits are then planned on the device, in
//     proportion to the lengths (DecodeParams::ragged).
//   * Each workgroup leaves (O unnormalised, reference, row sum) for its valid
//     columns in the workspace; swaa_decode_merge_kernel combines the splits.
//
// The split kernel declares no static LDS: its dynamic LDS starts at address 0
// and all its LDS accesses use plain byte addresses.
#include <atomic>
#include <type_traits>

#include "swaa_decode.h"
#include "swaa_tile_d128.h"

namespace swaa {
namespace {

constexpr int kDStageBytes = 2 * kHalfBytes;          // K half, then V half
// Stages of a wave's ring and workgroups per CU: the 382 registers of two column tiles leave one wave
// per SIMD, so one workgroup, whose waves then take two stages each.
constexpr int decode_stages(int tiles) { return tiles == 2 ? 2 : 1; }
constexpr int decode_wgs_per_cu(int tiles) { return tiles == 2 ? 1 : 2; }
constexpr int kDWaves = 4;
constexpr int kDThreads = 64 * kDWaves;
// LDS of a workgroup: every wave's ring, then the waves' references and row sums at the end
constexpr int decode_wave_bytes(int tiles) { return decode_stages(tiles) * kDStageBytes; }
constexpr int decode_smem_bytes(int tiles) { return kDWaves * (decode_wave_bytes(tiles) + tiles * 512); }
constexpr int kCopiesPerHalf = 16;                    // wave instructions per stage: 8 for K, 8 for V
constexpr int kMergeThreads = 256;
constexpr long long kDResident = 512;                 // workgroups of one column tile that run at once
constexpr long long kDResidentPairs = 256;            // ... of two

// ---- the split plan of a batch with per-sequence lengths, worked out by every workgroup of the
// split kernel (DecodeParams::ragged has the rules) ----
// Lane l keeps the lengths of sequences l, 64 + l, ... and the halves they visit (0 beyond the batch).
constexpr int kRaggedLaneRounds = kRaggedMaxBatch / 64;
struct RaggedHalves {
    int nk[kRaggedLaneRounds];
    unsigned n[kRaggedLaneRounds];
};
__device__ __forceinline__ RaggedHalves ragged_halves(const DecodeParams &p, int lane) {
    RaggedHalves h;
#pragma unroll
    for (int r = 0; r < kRaggedLaneRounds; ++r) h.nk[r] = p.seq_lens[min(64 * r + lane, p.B - 1)];
    static_assert(kRaggedLaneRounds == 4, "");
    asm volatile("" : "+v"(h.nk[0]), "+v"(h.nk[1]), "+v"(h.nk[2]), "+v"(h.nk[3]));  // (all asked for at once, not one behind the other's branch)
#pragma unroll
    for (int r = 0; r < kRaggedLaneRounds; ++r) {
        h.nk[r] = max(min(h.nk[r], p.Nk), p.Nq);
        h.n[r] = 64 * r + lane < p.B ? (unsigned)visited_halves(h.nk[r], p.Nq, p.W, p.S).n : 0u;
    }
    return h;
}
__device__ __forceinline__ unsigned ragged_halves_per_split(const DecodeParams &p, const RaggedHalves &h) {
    auto sum_over_sequences = [&](auto f) {
        unsigned mine = 0;
#pragma unroll
        for (int r = 0; r < kRaggedLaneRounds; ++r) mine += f(h.n[r]);
        return wave_read_lane(wave_inclusive_scan(mine), 63);
    };
    const unsigned target = (unsigned)p.units_target;
    const unsigned total = sum_over_sequences([](unsigned n) { return n; });
    unsigned hps = fastdiv(total + target - 1, p.div_target);
    // (splits of less than min_halves only where they are needed to have a workgroup per compute unit)
    const unsigned wide = min(fastdiv(4 * total + target - 1, p.div_target), (unsigned)p.min_halves);
    hps = (max(max(hps, wide), 4u) + 3u) & ~3u;  // (whole quarters for the four waves)
    // Rounding up per sequence can leave a few units more than the target, i.e. a handful of
    // workgroups in one more round than planned: lengthen the splits until the count fits (a
    // few steps; whatever they end on, the count stays below units_target + B).
    for (int it = 0; it < 4; ++it) {
        const unsigned units = sum_over_sequences([&](unsigned n) { return (n + hps - 1) / hps; });
        if (units <= target) break;
        const unsigned longer = fastdiv(hps * units + target - 1, p.div_target);
        hps = longer > hps ? longer : hps + 1;
    }
    return hps;
}
// The sequence and the split of unit `unit` of the list (sequence 0's splits, then sequence 1's, ...)
// and how many splits and keys that sequence has; false beyond the list's end.
__device__ __forceinline__ bool ragged_find(const RaggedHalves &h, unsigned hps, unsigned unit, int &b, int &split, int &n_splits, int &nk) {
    unsigned before = 0;
#pragma unroll
    for (int r = 0; r < kRaggedLaneRounds; ++r) {
        const unsigned mine = (h.n[r] + hps - 1) / hps;
        const unsigned incl = wave_inclusive_scan(mine);
        const unsigned in_round = wave_read_lane(incl, 63);
        if (unit - before < in_round) {
            const unsigned rel = unit - before;
            const int n = __popcll(__ballot(incl <= rel));  // sequences among these 64 that end at or before the unit
            const unsigned base = n ? wave_read_lane(incl, n - 1) : 0u;
            // (the same in all lanes; read through the first lane so that the compiler knows it
            // and keeps the addresses built from them in scalar registers)
            b = __builtin_amdgcn_readfirstlane(64 * r + n);
            split = __builtin_amdgcn_readfirstlane((int)(rel - base));
            n_splits = (int)wave_read_lane(mine, n);
            nk = (int)wave_read_lane((unsigned)h.nk[r], n);
            return true;
        }
        before += in_round;
    }
    return false;
}

// kPaged: k and v are a paged cache addressed through p.block_table (its own instantiation).
// kTiles: column tiles a workgroup computes from the same K and V fragments (1, or 2 when a pair has more than 32
// query rows: two tiles in two workgroups read every key twice, which only some sizes make up for, see plan_decode).
template <bool kF16, bool kPaged, int kTiles>
__global__ __launch_bounds__(kDThreads, decode_wgs_per_cu(kTiles)) void swaa_decode_split_kernel(const DecodeParams p) {
    fetch_args<DecodeParams>();
    // Workgroups reach the eight dies round-robin; the list has fewer than 2^31 items: 32-bit
    // arithmetic, divisions as multiplications.  Sequences of one length: die x takes the x-th
    // contiguous chunk of the item list (a die streams neighbouring memory: 3 % faster on one
    // long sequence).  Per-sequence lengths: the units (sequence, split) x KV heads go to the
    // dies in turn, so that whatever the lengths every die gets its share of the long sequences.
    // Either way the column-tile groups of one (pair, split), which read the same keys, share a die.
    constexpr int kDStages = decode_stages(kTiles);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned items = (unsigned)p.wg_items;
    unsigned witem;
    if (p.ragged) {
        const unsigned per_round = kXcds * (unsigned)p.n_ctgroups;
        const unsigned round = fastdiv(blockIdx.x, p.div_per_round), rem = blockIdx.x - round * per_round;
        witem = round * per_round + (rem % kXcds) * (unsigned)p.n_ctgroups + rem / kXcds;
    } else {
        const unsigned chunk = (items + kXcds - 1) / kXcds;
        const unsigned slot = blockIdx.x / kXcds;
        witem = (blockIdx.x % kXcds) * chunk + slot;
        if (slot >= chunk) return;
    }
    if (witem >= items) return;
    const unsigned item_ct = fastdiv(witem, p.div_ctgroups);      // witem / n_ctgroups
    const int ctg = (int)(witem - item_ct * (unsigned)p.n_ctgroups);
    int b, kvh, split, halves_per_split, n_splits;
    int Nk;  // this sequence's cache length (at least the query rows themselves)
    size_t slot0;  // workspace slot of the item's column tile 0
    if (p.ragged) {
        const unsigned unit = fastdiv(item_ct, p.div_hkv);        // (sequence, split) units, KV head innermost
        kvh = (int)(item_ct - unit * (unsigned)p.Hkv);
        const RaggedHalves rh = ragged_halves(p, lane);
        halves_per_split = __builtin_amdgcn_readfirstlane((int)ragged_halves_per_split(p, rh));
        if (!ragged_find(rh, (unsigned)halves_per_split, unit, b, split, n_splits, Nk)) return;  // beyond the true list
        slot0 = (size_t)item_ct * p.n_coltiles;
        // the sequence's first workgroup tells the merge kernel where its splits are (all lanes
        // store the same two words: a branch on the lane id here would make the compiler treat
        // what follows as lane-dependent, and the copies' base addresses must stay scalar)
        if (split == 0 && kvh == 0 && ctg == 0) {
            p.ws_units[2 * b] = (int)unit;
            p.ws_units[2 * b + 1] = n_splits;
        }
    } else {
        const unsigned upair = fastdiv(item_ct, p.div_splits);    // witem / (n_ctgroups * n_splits)
        split = (int)(item_ct - upair * (unsigned)p.n_splits);
        b = (int)fastdiv(upair, p.div_hkv);
        kvh = (int)upair - b * p.Hkv;
        halves_per_split = p.halves_per_split;
        n_splits = p.n_splits;
        slot0 = ((size_t)upair * p.n_splits + split) * p.n_coltiles;
        // (read as constant memory -- nothing writes the lengths while the kernel runs -- so that it is a scalar load)
        typedef const int __attribute__((address_space(4))) *ConstInts;
        Nk = p.seq_lens ? max(min(((ConstInts)p.seq_lens)[b], p.Nk), p.Nq) : p.Nk;
    }
    // this workgroup's column tiles and the workspace slots of their partial results
    int ct[kTiles];
    bool tile_valid[kTiles];
    size_t item[kTiles];
#pragma unroll
    for (int j = 0; j < kTiles; ++j) {
        ct[j] = ctg * kTiles + j;
        tile_valid[j] = ct[j] < p.n_coltiles;  // (uniform; an odd number of tiles leaves the last workgroup one)
        item[j] = slot0 + min(ct[j], p.n_coltiles - 1);
    }

    const int l32 = lane & 31;
    const int hf = lane >> 5;
    const int W = p.W, S = p.S;
    const VisitedHalves vh = visited_halves(Nk, p.Nq, W, S);

    // this lane's query column in each tile: row c of the pair's G x Nq block (clamped: padding
    // columns repeat the last row and are never stored)
    bool col_valid[kTiles];
    int cc[kTiles], qpos[kTiles];
#pragma unroll
    for (int j = 0; j < kTiles; ++j) {
        const int c = ct[j] * 32 + l32;
        col_valid[j] = tile_valid[j] && c < p.cols;
        cc[j] = min(c, p.cols - 1);
        qpos[j] = Nk - p.Nq + (cc[j] - (int)fastdiv((unsigned)cc[j], p.div_nq) * p.Nq);  // its position in the sequence
    }
    const int pos_min = Nk - p.Nq, pos_max = Nk - 1;

    const int h_begin = split * halves_per_split;
    const int n_split = min(vh.n - h_begin, halves_per_split);
    if (n_split <= 0) {
        // a shorter sequence has no keys for this split: an empty partial result (weight 0 in the merge)
#pragma unroll
        for (int j = 0; j < kTiles; ++j)
            if (col_valid[j] && hf == 0 && wave == 0) {
                p.ws_ml[item[j] * 64 + l32] = -INFINITY;
                p.ws_ml[item[j] * 64 + 32 + l32] = 0.f;
            }
        return;
    }
    // Every wave takes a quarter of the split, contiguous: with the waves' halves interleaved the
    // streams of all workgroups are a power of two apart (64 halves of 8 KiB on one 128k-token
    // sequence) and meet on the same memory channels: 117 us instead of 99.
    const int quarter = (n_split + kDWaves - 1) / kDWaves;
    const int n_mine = max(0, min(quarter, n_split - wave * quarter));
    auto first_key = [&](int t) {
        const int h = h_begin + quarter * wave + t;
        return 32 * (h < vh.n_sink ? h : h - vh.n_sink + vh.band0);
    };

    constexpr bool paged = kPaged;
    const uint32_t k_rsb = (uint32_t)(p.k_sn * 2), v_rsb = (uint32_t)(p.v_sn * 2);  // row strides in bytes
    const char *kg = reinterpret_cast<const char *>(p.k + (paged ? 0 : b * p.k_sb) + (long long)kvh * p.k_sh);
    const char *vg = reinterpret_cast<const char *>(p.v + (paged ? 0 : b * p.v_sb) + (long long)kvh * p.v_sh);
    // (the table is only read while the kernel runs: addressed as constant memory, so that the
    // lookups are scalar loads -- as vector loads they would share the tile copies' counter, and
    // waiting for a table entry would mean waiting for every copy in flight)
    typedef const int __attribute__((address_space(4))) *TablePtr;
    const TablePtr bt = paged ? (TablePtr)(p.block_table + (size_t)b * p.bt_stride) : nullptr;

    const HalfCopy half_copy(lane, k_rsb, v_rsb);
    const int lrow = lane >> 4;
    // Paged cache: the block-table entries one half needs -- one if a page holds a multiple of 32
    // tokens, two for a multiple of 16, else none here (looked up per copy instruction).  They
    // are scalar loads with a long way to go, asked for one loop iteration before the copy.
    struct Pages {
        int a, b;
    };
    const int pages_per_half = !paged ? 0 : p.page_size % 32 == 0 ? 1 : p.page_size % 16 == 0 ? 2 : 0;
    auto lookup = [&](int t) __attribute__((always_inline)) {
        Pages pg{0, 0};
        if constexpr (paged) {
            if (pages_per_half != 0) {
                const int k0 = first_key(t);
                pg.a = bt[fastdiv((unsigned)k0, p.div_page)];
                pg.b = pages_per_half == 2 ? bt[fastdiv((unsigned)min(k0 + 16, Nk - 1), p.div_page)] : pg.a;
            }
        }
        return pg;
    };
    auto issue_half = [&](int t, int stage, const Pages pg) __attribute__((always_inline)) {
        const int k0 = first_key(t);
        const uint32_t lds = (uint32_t)(wave * decode_wave_bytes(kTiles) + stage * kDStageBytes);
        const char *kb[2], *vb[2];
        if constexpr (paged) {
            if (pages_per_half == 0) {
                // page_size is a multiple of 4 only: the four rows of one instruction share a
                // page, so the page number is a uniform (scalar) table lookup per instruction
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int key4 = min(k0 + 4 * i, Nk - 1) & ~3;  // first row of the instruction, inside the cache
                    const unsigned pi = fastdiv((unsigned)key4, p.div_page);
                    const int page = min(max(bt[pi], 0), p.num_pages - 1);  // inside the cache whatever the table says
                    const int in_page = key4 - (int)pi * p.page_size;
                    const int back = max(key4 + lrow - (Nk - 1), 0);
                    HalfCopy::row4(lds + (uint32_t)(i * 1024), half_copy.k_lane[i & 3] - (uint32_t)back * k_rsb,
                                   kg + ((long long)page * p.k_sb + (long long)in_page * p.k_sn) * 2);
                    HalfCopy::row4(lds + (uint32_t)(kHalfBytes + i * 1024), half_copy.v_lane - (uint32_t)back * v_rsb,
                                   vg + ((long long)page * p.v_sb + (long long)in_page * p.v_sn) * 2);
                }
                return;
            }
            // page_size a multiple of 16: rows 0..15 of the half lie in one page, rows 16..31 in one
            // (the same one if page_size is a multiple of 32); their numbers came with `pg`.  Row
            // offsets count from the half's first row, so the second base steps back 16 rows; if
            // the cache ends inside the first 16 rows, every later row repeats its last row there.
            // (page strides and row strides of a paged cache fit 32 bits -- the entry point checks --
            // so each product is one 32 x 32 -> 64 bit multiplication, not the 64 x 64 bit one that
            // costs six: this arithmetic sits in front of every copy of the wave's only instruction stream)
            auto base_of = [](const char *g, long long sb, long long sn, int page, int row) __attribute__((always_inline)) {
                const long long elems = (long long)((unsigned long long)(unsigned)page * (unsigned)sb) + (long long)row * (int)sn;
                return g + 2 * elems;
            };
            const int in_a = k0 - (int)fastdiv((unsigned)k0, p.div_page) * p.page_size;
            const int page_a = min(max(pg.a, 0), p.num_pages - 1);
            kb[0] = kb[1] = base_of(kg, p.k_sb, p.k_sn, page_a, in_a);
            vb[0] = vb[1] = base_of(vg, p.v_sb, p.v_sn, page_a, in_a);
            if (pages_per_half == 2 && k0 + 16 <= Nk - 1) {
                const int in_b = k0 + 16 - (int)fastdiv((unsigned)(k0 + 16), p.div_page) * p.page_size;
                const int page_b = min(max(pg.b, 0), p.num_pages - 1);
                kb[1] = base_of(kg, p.k_sb, p.k_sn, page_b, in_b - 16);
                vb[1] = base_of(vg, p.v_sb, p.v_sn, page_b, in_b - 16);
            }
        } else {
            kb[0] = kb[1] = kg + (size_t)k0 * k_rsb;  // uniform
            vb[0] = vb[1] = vg + (size_t)k0 * v_rsb;
        }
        half_copy.half(lds, kb, vb, Nk - 1 - k0);
    };
    const LaneAddr la = make_lane_addr(lane, 0);

    // ---- start-up: the first halves into the stages and this lane's Q fragments (B operand of S^T = K Q^T: query
    // row l32, 16 bytes at 32 ks + 16 hf) straight from HBM with ordinary loads.  The compiler waits for all of
    // them, the copies included, before it parks the first fragment.  The copies go first (Q's addresses and requests in
    // front of them are 0.1 us) unless they have a page to look up: Q is asked for while the table entry is on its way
    // (four sequences of 0.4-10k tokens 10.0 us, behind the copies 10.25). ----
    const Pages pg_first = n_mine >= 1 ? lookup(0) : Pages{0, 0};
    auto copy_first = [&]() __attribute__((always_inline)) {
        if (n_mine >= 1) issue_half(0, 0, pg_first);
        if (kDStages >= 2 && n_mine >= 2) issue_half(1, 1, lookup(1));
    };
    if constexpr (!paged) copy_first();
    bf16x8 qf[kTiles][kKS];
#pragma unroll
    for (int j = 0; j < kTiles; ++j) {
        const char *qrow = reinterpret_cast<const char *>(p.q + ((size_t)b * p.Hq + (size_t)kvh * p.G) * p.Nq * kD) +
                           (size_t)cc[j] * kRowBytes + 16 * hf;
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) qf[j][ks] = *reinterpret_cast<const bf16x8 *>(qrow + 32 * ks);
    }
    if constexpr (paged) copy_first();
    // (the idle cycles keep the loads two wait states away from the first MFMA that reads them)
#pragma unroll
    for (int j = 0; j < kTiles; ++j)
        asm volatile("s_nop 1"
                     : "+a"(qf[j][0]), "+a"(qf[j][1]), "+a"(qf[j][2]), "+a"(qf[j][3]), "+a"(qf[j][4]), "+a"(qf[j][5]),
                       "+a"(qf[j][6]), "+a"(qf[j][7]));
    Pages pg_next = n_mine > kDStages ? lookup(kDStages) : Pages{0, 0};  // of the half the loop's first iteration issues

    f32x16 oacc[kTiles][kDB];
    RowState rs[kTiles];
#pragma unroll
    for (int j = 0; j < kTiles; ++j) {
#pragma unroll
        for (int db = 0; db < kDB; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) oacc[j][db][e] = 0.f;
        pin_acc(oacc[j]);
        rs[j].mc = -INFINITY;
        rs[j].l = 0.f;
        rs[j].lb = 0.f;
    }
    const float c2 = p.scale_log2;

    int stage = 0;
    for (int t = 0; t < n_mine; ++t) {
        // half t has landed when at most the copies of the halves issued after it are outstanding
        const int later = min(n_mine - 1 - t, kDStages - 1);
        if (later == 1)
            asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
        else
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        static_assert(kDStages <= 2 && kCopiesPerHalf == 16, "wait counts above");

        const uint32_t so = (uint32_t)(wave * decode_wave_bytes(kTiles) + stage * kDStageBytes);
        const int k0h = first_key(t);
        // no mask when every key of the half is visible to every column: at or below the
        // oldest row's diagonal, and inside the newest row's window or all sinks
        const bool masked = !((k0h + 31 <= pos_min) && ((k0h > pos_max - W) || (k0h + 31 < S)));

        // all operand fragments of the half go to registers first; once they are there the
        // stage is free and the copy of a later half leaves before any arithmetic
        bf16x8 kf[kKS], vf[2][kDB];
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) kf[ks] = load_k_frag(la, so, ks);
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int db = 0; db < kDB; ++db) vf[st][db] = load_v_frag(la, so + kHalfBytes, st, db);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (t + kDStages < n_mine) issue_half(t + kDStages, stage, pg_next);
        if (t + kDStages + 1 < n_mine) pg_next = lookup(t + kDStages + 1);  // lands under this iteration's arithmetic

#pragma unroll
        for (int j = 0; j < kTiles; ++j) {
            if (j > 0 && !tile_valid[j]) continue;  // (uniform)
            f32x16 s;
            bf16x8 pf[2];
            float alpha;
            mfma_s_first<kF16>(s, kf[0], qf[j][0]);
#pragma unroll
            for (int ks = 1; ks < kKS - 1; ++ks) mfma_s<kF16>(s, kf[ks], qf[j][ks]);
            mfma_s_settled<kF16>(s, kf[kKS - 1], qf[j][kKS - 1]);
            if (masked)
                softmax_half<true, kF16>(s, k0h, qpos[j], W, S, hf, c2, rs[j], pf, alpha);
            else
                softmax_half<false, kF16>(s, k0h, qpos[j], W, S, hf, c2, rs[j], pf, alpha);
            rescale(oacc[j], alpha);
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
                for (int db = 0; db < kDB; ++db) {
                    if (st == 1 && db == kDB - 1)
                        mfma_acc_settled<kF16>(oacc[j][db], vf[st][db], pf[st]);  // the accumulators are read below / next time round
                    else
                        mfma_acc<kF16>(oacc[j][db], vf[st][db], pf[st]);
                }
        }
        stage = (stage + 1 == kDStages) ? 0 : stage + 1;
    }

    // ---- the four waves' results are added up through LDS (leave_result) and leave as the split's partial
    // result -- or, with one split, as the output itself ----
    constexpr uint32_t kMl = (uint32_t)(kDWaves * decode_wave_bytes(kTiles));
#pragma unroll
    for (int j = 0; j < kTiles; ++j)
        leave_result((uint32_t)(wave * decode_wave_bytes(kTiles) + j * kDStageBytes), kMl + (uint32_t)((j * kDWaves + wave) * 512), l32, hf,
                     col_valid[j], oacc[j], rs[j]);
    __syncthreads();
    const size_t row0 = ((size_t)b * p.Hq + (size_t)kvh * p.G) * p.Nq;
#pragma unroll
    for (int j = 0; j < kTiles; ++j) {
        const int n_chunks = tile_valid[j] ? 32 * min(32, p.cols - 32 * ct[j]) : 0;
        for (int i = (int)threadIdx.x; i < n_chunks; i += kDThreads) {
            const int c = i >> 5, q = i & 31;  // column of the tile; its head-dimension elements 4 q ..
            float m, l;
            f32x4_t o4 = add_results((uint32_t)(j * kDStageBytes), (uint32_t)decode_wave_bytes(kTiles), kMl + (uint32_t)(j * kDWaves * 512), c, q, m, l);
            if (n_splits == 1) {
                const size_t row = row0 + (size_t)(32 * ct[j] + c);
                o4 *= 1.f / l;
                const bf16x2 lo = pack_pair<kF16>(o4[0], o4[1]), hi = pack_pair<kF16>(o4[2], o4[3]);
                *reinterpret_cast<bf16x4 *>(p.out + row * kD + 4 * q) = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
                if (q == 0) p.lse[row] = (m + __builtin_amdgcn_logf(l)) * 0.69314718055994530942f;
            } else {
                *reinterpret_cast<f32x4_t *>(p.ws_o + (item[j] * p.col_stride + c) * kD + 4 * q) = o4;
                if (q == 0) {
                    // (a sum that is not a number travels with a finite reference: -inf, the largest score of a column that
                    // sees NaN only, would mark the split as empty, and the merge would leave it out)
                    p.ws_ml[item[j] * 64 + c] = non_finite(l) ? 0.f : m;
                    p.ws_ml[item[j] * 64 + 32 + c] = l;
                }
            }
        }
    }
}

// ---- merging the splits: out = sum_s 2^(mc_s - m) O_s / sum_s 2^(mc_s - m) l_s with m = max_s mc_s;
// lse = (m + log2 of the denominator) ln 2 ----
// What the merge needs to know, two lines of arguments instead of the split kernel's six.
struct MergeParams {
    const float *ws_o, *ws_ml;
    const int *ws_units;
    __bf16 *out;
    float *lse;
    FastDiv div_nq, div_hq, div_g;
    int Nq, Hq, Hkv, G, n_splits, n_coltiles, col_stride, B;
    int ragged, fp16;
    unsigned rows, n_small;  // B * Hq * Nq; workgroups of the ragged launch that take kMergeRows rows each
};
// One output row (b, hq, r) and where its partial results are: n_splits items, item_step workspace
// slots apart, the first at item0.
struct MergeRow {
    unsigned row;
    int col;
    int n_splits;
    long long item0, item_step;
};
__device__ __forceinline__ MergeRow merge_row(const MergeParams &p, unsigned row) {
    // (The merge is bound by its chain of dependent steps.  With three 64-bit and two 32-bit divisions here, a hundred
    // instructions each, one sequence of 2000 tokens took 11.1 us in all on 32 heads, with multiplications 10.6; 8 heads on 8, 4096
    // tokens: 11.7, 11.0; window 8192 of 131072: 15.3, 14.9.)
    MergeRow m;
    m.row = row;
    const unsigned head_row = fastdiv(row, p.div_nq);
    const int r = (int)(row - head_row * (unsigned)p.Nq);
    const int b = (int)fastdiv(head_row, p.div_hq);
    const int hq = (int)(head_row - (unsigned)b * (unsigned)p.Hq);
    const int kvh = (int)fastdiv((unsigned)hq, p.div_g);
    const int c = (hq - kvh * p.G) * p.Nq + r;
    long long slot0, step;
    if (p.ragged) {  // (the device-side plan: the sequence's first split workgroup has left it here)
        m.n_splits = p.ws_units[2 * b + 1];
        slot0 = (long long)p.ws_units[2 * b] * p.Hkv + kvh;
        step = p.Hkv;
    } else {
        m.n_splits = p.n_splits;
        slot0 = ((long long)b * p.Hkv + kvh) * p.n_splits;
        step = 1;
    }
    m.col = c & 31;
    m.item0 = slot0 * p.n_coltiles + (c >> 5);
    m.item_step = step * p.n_coltiles;
    return m;
}
// Elements 4 q .. 4 q + 3 of a row.
__device__ __forceinline__ void merge_store(const MergeParams &p, unsigned row, int q, f32x4_t o, float l, float m) {
    o /= l;
    const bf16x2 lo = p.fp16 ? pack_pair<true>(o[0], o[1]) : pack_pair<false>(o[0], o[1]);
    const bf16x2 hi = p.fp16 ? pack_pair<true>(o[2], o[3]) : pack_pair<false>(o[2], o[3]);
    *reinterpret_cast<bf16x4 *>(p.out + (size_t)row * kD + 4 * q) = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
    if (q == 0) p.lse[row] = (m + __builtin_amdgcn_logf(l)) * 0.69314718055994530942f;
}
// Largest value and sum over the 64 lanes of a wave, all of them active (shift steps as in wave_inclusive_scan).
template <typename F>
__device__ __forceinline__ float wave_reduce(float x, float none, F f) {
    const int id = __float_as_int(none);
    auto step = [&](auto ctrl, auto rows) {
        x = f(x, __int_as_float(__builtin_amdgcn_update_dpp(id, __float_as_int(x), decltype(ctrl)::value, decltype(rows)::value, 0xf, false)));
    };
    using std::integral_constant;
    step(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});
    step(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

// A whole workgroup on one row (many splits): 32 threads to a split, four elements each, eight splits side by side.
// Every wave finds the largest reference and the sum of the l by itself, a split per lane, from loads that go out
// together with the first O's: one trip to memory and one barrier.
__device__ __forceinline__ void merge_row_by_workgroup(const MergeParams &p, const MergeRow &mr, f32x4_t *red) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int q = tid % 32, g = tid / 32;
    constexpr int kGroups = kMergeThreads / 32, kBatch = 4;
    const int n = mr.n_splits;
    auto ml_of = [&](int s) { return p.ws_ml + (mr.item0 + s * mr.item_step) * 64 + mr.col; };
    // A split that saw no visible key has reference -inf and may not have written its O: it is loaded all the same
    // (the workspace is there) and left out of the sums by selection, not by a branch; so is what lies beyond the last split.
    float mcs[kBatch];
    f32x4_t os[kBatch];
    auto load = [&](int s0) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int s = s0 + u * kGroups, at = min(s, n - 1);
            mcs[u] = *ml_of(at);
            os[u] = *reinterpret_cast<const f32x4_t *>(p.ws_o + ((mr.item0 + at * mr.item_step) * p.col_stride + mr.col) * kD + 4 * q);
            if (s >= n) mcs[u] = -INFINITY;
        }
    };
    float mc = *ml_of(min(lane, n - 1)), l = *(ml_of(min(lane, n - 1)) + 32);
    load(g);
    if (lane >= n) mc = -INFINITY;
    float m = mc;
    for (int s = lane + 64; s < n; s += 64) m = fmaxf(m, *ml_of(s));
    m = wave_reduce(m, -INFINITY, [](float a, float b) { return fmaxf(a, b); });  // finite: every row sees at least its own key
    l = mc == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mc - m) * l;
    for (int s = lane + 64; s < n; s += 64) {
        const float mcx = *ml_of(s), w = __builtin_amdgcn_exp2f(mcx - m) * *(ml_of(s) + 32);
        l += mcx == -INFINITY ? 0.f : w;
    }
    l = wave_reduce(l, 0.f, [](float a, float b) { return a + b; });
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = g;;) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const bool empty = mcs[u] == -INFINITY;
            const float w = __builtin_amdgcn_exp2f(mcs[u] - m);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += empty ? 0.f : w * os[u][e];
        }
        s0 += kBatch * kGroups;
        if (s0 - g >= n) break;  // (the same in all groups)
        load(s0);
    }
    red[tid] = acc;
    __syncthreads();
    if (g == 0) {
#pragma unroll
        for (int gg = 1; gg < kGroups; ++gg) acc += red[gg * 32 + q];
        merge_store(p, mr.row, q, acc, l, m);
    }
}

// 32 threads (four head dimension elements each) on one row of at most kMergeRowSplits splits: every
// thread adds up the row's splits by itself -- no exchange between threads.
constexpr int kMergeRowSplits = 8;
__device__ __forceinline__ void merge_row_by_group(const MergeParams &p, const MergeRow &mr, int q) {
    float mcs[kMergeRowSplits], ls[kMergeRowSplits];
    f32x4_t os[kMergeRowSplits];
    // (a split that saw no visible key has reference -inf and may not have written its O: loaded all
    // the same and left out by selection; splits beyond the row's repeat the last one and count as empty)
#pragma unroll
    for (int s = 0; s < kMergeRowSplits; ++s) {
        const bool there = s < mr.n_splits;
        const long long it = mr.item0 + (there ? s : 0) * mr.item_step;
        mcs[s] = p.ws_ml[it * 64 + mr.col];
        ls[s] = p.ws_ml[it * 64 + 32 + mr.col];
        os[s] = *reinterpret_cast<const f32x4_t *>(p.ws_o + (it * p.col_stride + mr.col) * kD + 4 * q);
        if (!there) mcs[s] = -INFINITY;
    }
    float m = mcs[0];
#pragma unroll
    for (int s = 1; s < kMergeRowSplits; ++s) m = fmaxf(m, mcs[s]);  // finite: every row sees at least its own key
    float l = 0.f;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < kMergeRowSplits; ++s) {
        const bool empty = mcs[s] == -INFINITY;
        const float w = __builtin_amdgcn_exp2f(mcs[s] - m);
        l += empty ? 0.f : w * ls[s];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += empty ? 0.f : w * os[s][e];
    }
    merge_store(p, mr.row, q, acc, l, m);
}

// Sequences of one length, more than kMergeRowSplits splits per pair: one workgroup per output row.
__global__ __launch_bounds__(kMergeThreads) void swaa_decode_merge_kernel(const MergeParams p) {
    __shared__ f32x4_t red[kMergeThreads];
    merge_row_by_workgroup(p, merge_row(p, blockIdx.x), red);
}

// Sequences of one length, at most kMergeRowSplits splits per pair: kMergeRows output rows
// per workgroup.  A batch of many sequences has thousands of rows of two or three splits each;
// one workgroup of 1024 threads per row spent most of the merge waiting for workgroup slots (64
// sequences x 8 new tokens: the call took 275 us, 70 of them here).
constexpr int kMergeRows = kMergeThreads / 32;
__global__ __launch_bounds__(kMergeThreads) void swaa_decode_merge_rows_kernel(const MergeParams p) {
    const unsigned row = blockIdx.x * kMergeRows + threadIdx.x / 32;
    if (row >= p.rows) return;
    merge_row_by_group(p, merge_row(p, row), threadIdx.x % 32);
}

// Per-sequence lengths: both at once.  The first n_small workgroups take kMergeRows rows
// each and merge those of at most kMergeRowSplits splits, 32 threads per row.  The rows of the
// sequences with more splits -- there are at most (units_target + B) / (kMergeRowSplits + 1) such
// sequences -- are left to the workgroups behind them, one row each: workgroup n_small + k looks
// for the (k / (Hq Nq))-th such sequence in the plan the split kernel has left (a prefix sum of
// flags over the lanes, every wave for itself) and goes home if there is none.
__global__ __launch_bounds__(kMergeThreads) void swaa_decode_merge_ragged_kernel(const MergeParams p) {
    __shared__ f32x4_t red[kMergeThreads];
    if (blockIdx.x < p.n_small) {
        const unsigned row = blockIdx.x * kMergeRows + threadIdx.x / 32;
        if (row >= p.rows) return;
        const MergeRow mr = merge_row(p, row);
        if (mr.n_splits > 1 && mr.n_splits <= kMergeRowSplits) merge_row_by_group(p, mr, threadIdx.x % 32);
        return;
    }
    const unsigned k = blockIdx.x - p.n_small, rows_per_seq = (unsigned)(p.Hq * p.Nq);
    const unsigned want = k / rows_per_seq;  // the want-th sequence with many splits (from 0)
    const int lane = threadIdx.x & 63;
    unsigned before = 0;
    int b = -1;
    for (int c0 = 0; c0 < p.B; c0 += 64) {
        const bool many = c0 + lane < p.B && p.ws_units[2 * (c0 + lane) + 1] > kMergeRowSplits;
        const unsigned incl = wave_inclusive_scan(many ? 1u : 0u);
        const unsigned in_round = wave_read_lane(incl, 63);
        if (want - before < in_round) {
            b = c0 + __popcll(__ballot(incl <= want - before));
            break;
        }
        before += in_round;
    }
    if (b < 0) return;  // (the same in every wave of the workgroup)
    merge_row_by_workgroup(p, merge_row(p, (unsigned)b * rows_per_seq + (k - want * rows_per_seq)), red);
}

}  // namespace

void plan_decode(DecodeParams &p, bool ragged, bool own_scratch) {
    p.cols = p.G * p.Nq;
    p.n_coltiles = (p.cols + 31) / 32;
    p.col_stride = p.cols < 32 ? p.cols : 32;
    // an upper bound on the halves any sequence of at most Nk tokens visits (a shorter sequence's
    // band can straddle one half more than the longest one's): the splits are planned for it
    const int all = (p.Nk + 31) / 32;
    const int bound = (p.S + 31) / 32 + (p.W + p.Nq - 2) / 32 + 2;
    p.n_halves = all < bound ? all : bound;
    p.ragged = ragged && p.B >= 2 && p.B <= kRaggedMaxBatch && (long long)p.B * p.n_halves < 0x7fffffffLL ? 1 : 0;
    // Two column tiles per workgroup read every key once, but only one such workgroup fits a compute unit.  One
    // tile each where that makes one round of workgroups alone on their compute units (at least 128 pairs of
    // tiles, up to 256 tiles), or 1.5 rounds at most instead of two (257 pairs of tiles and more, up to 768 tiles).
    // (128 pairs of at most 192 tiles on long keys: two splits of two tiles each are one round as well, and the
    // keys are read once.)  Measured, two tiles / one tile (us; 8 KV heads, bf16, 40 columns or, *, 80; one split):
    //   16 x 2k 36.7 / 25.4    16 x 16k 216 / 191     8 x 8k* 115 / 71.3    10 x 8k* 114 / 86.2
    //   20 x 4k 69.0 / 84.8    28 x 16k 319 / 370    12 x 8k* 115 / 139     16 x 8k* 126 / 150
    //   33 x 1k 47.5 / 33.8    33 x 8k 286 / 247     40 x 4k 158 / 135      17 x 8k* 222 / 148
    //   48 x 4k 162 / 150      48 x 16k 577 / 570    56 x 4k 174 / 189      24 x 8k* 225 / 223
    const long long tiles = (long long)p.B * p.Hkv * p.n_coltiles, tile_pairs = (long long)p.B * p.Hkv * ((p.n_coltiles + 1) / 2);
    const bool two_splits = tile_pairs == 128 && tiles <= 192 && p.n_halves >= 384;
    const bool one_each = !p.ragged && !two_splits && tile_pairs >= 128 && (tiles <= 256 || (tile_pairs > 256 && tiles <= 768));
    p.tiles_per_item = p.n_coltiles >= 2 && !one_each ? 2 : 1;
    p.n_ctgroups = (p.n_coltiles + p.tiles_per_item - 1) / p.tiles_per_item;
    const long long groups = (long long)p.B * p.Hkv * p.n_ctgroups;
    p.div_ctgroups = make_fastdiv((unsigned)p.n_ctgroups);
    p.div_per_round = make_fastdiv((unsigned)(kXcds * p.n_ctgroups));
    p.div_hkv = make_fastdiv((unsigned)p.Hkv);
    p.div_nq = make_fastdiv((unsigned)p.Nq);
    p.div_hq = make_fastdiv((unsigned)p.Hq);
    p.div_g = make_fastdiv((unsigned)p.G);
    if (p.ragged) {
        // Per-sequence lengths: about this many workgroups, cut on the device in proportion to the
        // sequences' lengths.  Up to one per resident place (512; 256 with two column tiles) they are
        // cut into twice as many; more (pair, column tile) groups than that need some surplus to even
        // out the lengths, the less the more columns a partial result has.  Measured over the number
        // of workgroups (us; 8 KV heads, binary16, pages of 16):
        //   128 sequences of 0.2-8k tokens             1152: 246, 2048: 234, 2304: 233, 4096: 239
        //   75 of 0.2-17k                               512: 307, 1152: 226, 2048: 222, 4096: 228
        //   66 of 0.1-4k                                512: 57.5, 1152: 45.3, 2048: 46.1, 4096: 53.1
        //   92 of 1-9k, window 1k, 20 columns           512: 94.4, 1152: 96.8, 1536: 115, 4096: 129
        //   65 of 0.2-10k, window 8k, 20 columns        512: 166, 1152: 158, 2048: 170, 4096: 186
        //   56 of 0.2-23k, window 1k, 16 columns        512: 43.7, 1024: 52.3  (min_halves: three splits of 12)
        //   80 of 0.3-4k, 36 columns                    288: 145, 576: 148, 1152: 176, 2048: 202
        const long long resident = 256LL * decode_wgs_per_cu(p.tiles_per_item);
        long long wgs = 2 * resident;
        if (groups > resident && p.tiles_per_item == 1) {
            wgs = p.cols <= 8 ? 2 * groups : groups;
            wgs = wgs < 1152 ? 1152 : wgs > 2304 ? 2304 : wgs;
        }
        p.min_halves = p.cols <= 8 ? 16 : 40;
        const long long units = wgs / ((long long)p.Hkv * p.n_ctgroups);
        p.units_target = (int)(units < 1 ? 1 : units);
        p.div_target = make_fastdiv((unsigned)p.units_target);
        // (at most units_target + B units by the rounding of the device's division, and no
        // sequence has more than ceil(n_halves / 4) splits)
        const long long most = (long long)p.B * ((p.n_halves + 3) / 4);
        p.max_units = (int)(p.units_target + p.B < most ? p.units_target + p.B : most);
        p.halves_per_split = p.n_splits = 0;
        p.div_splits = make_fastdiv(1u);
        p.wg_items = (long long)p.max_units * p.Hkv * p.n_ctgroups;
        p.items = (long long)p.max_units * p.Hkv * p.n_coltiles;
        return;
    }
    // Sequences of one length.  A workgroup draws at most 50 GB/s, so 128 of them come near the
    // rate of the memory and 192 reach it; more splits than that only cost the merge kernel and its
    // traffic, and a power of two of them reads streams that are a power of two apart and meet on
    // the same memory channels.  What also counts is how full the last round of workgroups is, and whether
    // few compute units have one workgroup more than the others.  Measured over n splits (us; 8 KV heads, bf16).
    // One column tile:
    //   1 sequence x 128k tokens      n = 16: 106, 20: 96.7, 24: 96.6, 32: 99.5, 48: 103, 64: 99.7
    //   1 x 100k                      n = 16: 84.9, 24: 78.2, 32: 90.0, 48: 82.1, 64: 90.5
    //   2 x 60k                       n = 8: 98, 12: 90.5, 16: 121, 24: 95.0, 32: 105
    //   4 x 123k, 4 new tokens        n = 4: 370, 6: 330, 8: 437, 12: 350, 16: 354, 32: 367
    //   5 x 40k                       n = 4: 143, 5: 144, 6: 151, 7: 187, 12: 148
    //   8 x 32k                       n = 2: 197, 3: 182, 4: 181, 6: 189, 8: 183
    //   1 x window 8k                 n = 12: 15.7, 16: 15.0, 24: 14.2, 32: 14.3
    //   4 x 8k                        n = 4: 29.4, 6: 28.3, 8: 28.8, 16: 28.8, 32: 35.4
    //   1 x 500                       n = 1: 10.1, 4: 10.6
    //   16 x window 2k                n = 1: 27.3, 2: 30.4, 4: 30.5    (one split: no merge kernel)
    //   16 x 4k                       n = 1: 43.4, 2: 47.9, 4: 47.9
    //   16 x 20k                      n = 1: 236, 2: 224, 4: 226
    //   22 x 20k                      n = 1: 295, 2: 333, 3: 351, 4: 307
    //   32 x 20k                      n = 1: 432, 2: 437, 4: 440
    //   28 x 16k, 8 new tokens        n = 1: 306, 2: 330, 3: 333
    //   33 x 2k                       n = 1: 60.2, 4: 52.4    33 x 16k   n = 1: 495, 2: 427, 4: 396
    //   40 x 4k                       n = 1: 135, 4: 122      48 x 4k    n = 1: 144, 2: 145, 4: 147
    //   33 x 2k, 8 new tokens         n = 1: 61.3, 3: 63.9    33 x 16k, 8 new tokens   n = 1: 496, 3: 442
    //   64 x 2k                       n = 1: 96.7, 2: 101, 4: 106
    //   100 x 4k                      n = 1: 312, 2: 306, 4: 294, 8: 294
    //   256 x 1k                      n = 1: 183, 2: 196
    // Two column tiles (or, *, three: 80 columns) per workgroup, 64 KiB of partial results per split:
    //   4 x 8k*                       n = 2: 68.0, 3: 53.1, 4: 46.0, 5: 63.2
    //   5 x 16k*                      n = 2: 120, 3: 89.4, 4: 127      7 x 16k*   n = 1: 212, 2: 124, 4: 131
    //   5 x 16k                       n = 4: 72.4, 5: 68.8, 6: 70.9    8 x 16k    n = 2: 124, 3: 107, 4: 108
    //   4 x 10k                       n = 6: 39.2, 8: 58.4             1 x 13k*   n = 12: 30.1, 16: 43.4
    //   64 x 4k, 16 new tokens        n = 1: 204, 2: 247, 4: 266
    //   65 x 16k                      n = 1: 900, 4: 823              72 x 24k   n = 1: 1353, 4: 1261
    //   65 x 8k                       n = 1: 461, 4: 454              80 x 16k   n = 1: 933, 4: 972
    // Several column tiles, one per workgroup (40 columns):
    //   33 x 8k                       n = 1: 247, 2: 237, 3: 232, 4: 228    40 x 8k   n = 1: 261, 2: 256, 3: 266
    //   36 x 8k                       n = 1: 258, 2: 247, 3: 243, 4: 252    44 x 8k   n = 1: 267, 2: 296
    const long long few = p.n_halves <= 16 ? 1 : (192 + groups / 2) / groups < 48 ? (192 + groups / 2) / groups : 48;
    long long n = 1;
    bool may_exceed = false;  // the static array, where a workspace is given
    if (p.tiles_per_item == 2) {
        const long long last = (groups - 1) % kDResidentPairs + 1;  // workgroups in the last round
        if (groups <= 128) {
            n = few;
            if (groups >= 64 && kDResidentPairs / groups > n && p.n_halves > 16) n = kDResidentPairs / groups;
        }
        if (groups > kDResidentPairs && last <= kDResidentPairs / 4 && p.n_halves >= 384)
            n = 4;
        may_exceed = groups > 128;
    } else if (p.n_coltiles >= 2) {
        if (groups > kDResident && p.n_halves >= 128) n = groups <= 544 ? 4 : p.n_halves < 192 ? 1 : groups <= 608 ? 3 : groups <= 656 ? 2 : 1;
        may_exceed = true;
    } else if (groups < 128) {
        n = few;
    } else if (groups <= kDResident) {
        if (groups == 128 && p.cols <= 8 && p.n_halves >= 256) n = 4;  // (one workgroup per compute unit at half of them draws too little)
        if (groups > 256 && groups <= 320 && p.n_halves >= (p.cols <= 8 ? 64 : 192)) n = 4;
    } else if (groups < 4 * kDResident && p.n_halves > 96) {
        n = 4;
    }
    // A call whose partial results fit the library's own scratch array with fewer splits gets no more than fit
    // (whatever the window, so that the next rule holds).
    const long long split_bytes = (long long)p.B * p.Hkv * p.n_coltiles * ((long long)p.col_stride * kD + 64) * (long long)sizeof(float);
    if (split_bytes <= kDecodeStaticScratchBytes && (own_scratch || !may_exceed))
        while (n > 1 && (n + n / 8) * split_bytes > kDecodeStaticScratchBytes) --n;
    // The workspace is sized for the most splits any smaller number of halves would get: a caller's
    // workspace for a full-attention layer serves the windowed layers of the same model.
    const long long most = n == 1 ? 1 : (p.n_halves + 3) / 4 < n + n / 8 ? (p.n_halves + 3) / 4 : n + n / 8;
    // (whole quarters for the four waves: rounded down if that makes at most an eighth more splits, else up)
    long long hps = n == 1 ? p.n_halves : p.n_halves / n / 4 * 4;
    if (n > 1 && (hps < 4 || (p.n_halves + hps - 1) / hps > n + n / 8)) hps = (p.n_halves + 4 * n - 1) / (4 * n) * 4;
    p.halves_per_split = (int)hps;
    p.n_splits = (int)((p.n_halves + hps - 1) / hps);
    p.wg_items = groups * p.n_splits;
    p.items = (long long)p.B * p.Hkv * p.n_coltiles * most;
    p.div_splits = make_fastdiv((unsigned)p.n_splits);
}

long long decode_workspace_floats(const DecodeParams &p) {
    // (per item O and 64 floats of references and row sums; ragged: two ints per sequence on top, rounded to 16 bytes)
    return p.items * ((long long)p.col_stride * kD + 64) + (p.ragged ? (2LL * p.B + 3) / 4 * 4 : 0);
}

// ---- scratch memory for callers that cannot allocate -----------------------------------
// swaa_attn_decode_static keeps the partial results of the key splits here instead of in
// a caller's workspace.  In host code the array's name is only a stand-in for the device
// object: its device address comes from hipGetSymbolAddress, asked once per device with
// that device current (every GPU the library runs on holds its own copy of the array at
// its own address until the process ends), and host code passes that address, never the
// name, to kernels.
static __device__ __align__(256) unsigned char scratch[kDecodeStaticScratchBytes];

hipError_t decode_static_scratch(void **ptr) {
    constexpr int kMaxDevices = 64;
    static std::atomic<void *> address[kMaxDevices];  // zero-initialised
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    void *a = address[dev].load(std::memory_order_acquire);
    if (!a) {
        err = hipGetSymbolAddress(&a, HIP_SYMBOL(scratch));
        if (err != hipSuccess) return err;
        if (!a) return hipErrorInvalidSymbol;
        address[dev].store(a, std::memory_order_release);  // (two threads racing here store the same value)
    }
    *ptr = a;
    return hipSuccess;
}

hipError_t launch_decode(const DecodeParams &p, hipStream_t stream) {
    // (a whole number of rounds of 8 x column-tile groups covers both item orders)
    const long long per_round = (long long)kXcds * p.n_ctgroups;
    const long long chunk = (p.wg_items + kXcds - 1) / kXcds;
    const long long wgs = p.ragged ? (p.wg_items + per_round - 1) / per_round * per_round : chunk * kXcds;
    const dim3 grid((unsigned)wgs);
    const bool paged = p.block_table != nullptr;
    hipError_t err = hipSuccess;
    auto launch = [&](auto f16, auto pg, auto tiles) {
        constexpr int kT = decltype(tiles)::value;
        constexpr auto kernel = swaa_decode_split_kernel<decltype(f16)::value, decltype(pg)::value, kT>;
        err = allow_lds<kernel, decode_smem_bytes(kT)>();
        if (err != hipSuccess) return;
        hipLaunchKernelGGL(kernel, grid, dim3(kDThreads), decode_smem_bytes(kT), stream, p);
    };
    auto pick_tiles = [&](auto f16, auto pg) {
        if (p.tiles_per_item == 2)
            launch(f16, pg, std::integral_constant<int, 2>{});
        else
            launch(f16, pg, std::integral_constant<int, 1>{});
    };
    if (p.fp16 && paged)
        pick_tiles(std::true_type{}, std::true_type{});
    else if (p.fp16)
        pick_tiles(std::true_type{}, std::false_type{});
    else if (paged)
        pick_tiles(std::false_type{}, std::true_type{});
    else
        pick_tiles(std::false_type{}, std::false_type{});
    if (err == hipSuccess) err = hipGetLastError();
    if (err != hipSuccess || (!p.ragged && p.n_splits == 1)) return err;
    const long long rows = (long long)p.B * p.Hq * p.Nq;
    const unsigned n_small = (unsigned)((rows + kMergeRows - 1) / kMergeRows);
    const MergeParams mp{p.ws_o, p.ws_ml, p.ws_units, p.out, p.lse, p.div_nq, p.div_hq, p.div_g,
                         p.Nq, p.Hq, p.Hkv, p.G, p.n_splits, p.n_coltiles, p.col_stride, p.B,
                         p.ragged, p.fp16, (unsigned)rows, n_small};
    if (p.ragged) {
        long long many = ((long long)p.units_target + p.B) / (kMergeRowSplits + 1);  // sequences that can have more splits
        many = many < p.B ? many : p.B;
        if (n_small + many * p.Hq * p.Nq > 0x7fffffffLL) return hipErrorInvalidValue;
        hipLaunchKernelGGL(swaa_decode_merge_ragged_kernel, dim3(n_small + (unsigned)(many * p.Hq * p.Nq)), dim3(kMergeThreads), 0,
                           stream, mp);
    } else if (p.n_splits <= kMergeRowSplits) {
        hipLaunchKernelGGL(swaa_decode_merge_rows_kernel, dim3(n_small), dim3(kMergeThreads), 0, stream, mp);
    } else {
        hipLaunchKernelGGL(swaa_decode_merge_kernel, dim3((unsigned)rows), dim3(kMergeThreads), 0, stream, mp);
    }
    return hipGetLastError();
}

}  // namespace swaa
