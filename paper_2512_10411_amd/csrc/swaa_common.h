// Types, the kernel parameter block and the work decomposition shared by the
// attention-forward kernels of libswaa (gfx950 only).
#ifndef SWAA_COMMON_H_
#define SWAA_COMMON_H_

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

namespace swaa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kBk = 64;        // keys per KV tile
constexpr int kThreads = 256;  // per workgroup of the forward kernels that leave scheduling to the compiler
constexpr int kWgRows = 256;   // query rows (head x position) per workgroup of the dQ kernels
constexpr int kFwdWgRows = 128;  // query rows (head x position) per workgroup of the forward kernels
constexpr int kXcds = 8;       // accelerator dies; workgroups are dealt to them round-robin

// Division of a number below 2^31 by a divisor fixed at launch, as a multiplication: with
// l = ceil(log2 d) and m = ceil(2^(31 + l) / d) (which fits 32 bits), n / d = (n * m) >> (31 + l)
// exactly: m d - 2^(31 + l) < d <= 2^l, so the product overshoots n / d by less than 1 / d.
// Every wave of every workgroup decodes its work item with three such divisions; done the long
// way they are about a hundred instructions in front of the first memory request.
struct FastDiv {
    unsigned m;
    int sh;  // negative: the divisor is 1
};
inline FastDiv make_fastdiv(unsigned d) {
    FastDiv f{0u, -1};
    if (d <= 1) return f;
    int l = 0;
    while ((1ull << l) < d) ++l;
    f.m = (unsigned)(((1ull << (31 + l)) + d - 1) / d);
    f.sh = l - 1;
    return f;
}
__host__ __device__ __forceinline__ unsigned fastdiv(unsigned n, const FastDiv f) {
    return f.sh < 0 ? n : (unsigned)(((unsigned long long)n * f.m) >> 32) >> f.sh;  // (the upper half of one 32 x 32 bit product)
}

// First statement of a kernel of short calls: brings its argument block (a struct Args, the kernel's first argument) into the
// scalar cache in one round trip.  The compiler loads arguments where they are first used, a line of 64 bytes at a time, and a
// line that no cache holds (a launch has a block of its own; a captured one is replayed from the same) is 350 ns away:
// three to five such waits stood in front of the first request to memory.  us a call: one new token on a window of 8192
// 12.9 -> 12.3; short prompts of 300 tokens 8.55 -> 8.35; 84 tokens, D = 64, 6.0 -> 5.4.  Kernels of longer calls gain nothing
// (the pipelined forward loses 0.4 % on packed prompts).  Workgroups behind the first round find the lines there.
template <typename Args>
__device__ __forceinline__ void fetch_args() {
    static_assert(sizeof(Args) % 4 == 0, "");
    if (blockIdx.x >= 512) return;
    const auto args = (const int __attribute__((address_space(4))) *)__builtin_amdgcn_kernarg_segment_ptr();
    int word;  // (waited for in the same block, so that nothing is in flight behind it, and taken by a statement of its own.  The compiler's own
               // loads in front of one statement that takes them all: a wait more in the decode kernel, 8 x 2000 keys 16.07 -> 16.25 us)
    asm volatile(".set swaa_line, 0\n\t"
                 ".rept %c2\n\t"
                 "s_load_dword %0, %1, swaa_line\n\t"
                 ".set swaa_line, swaa_line + 64\n\t"
                 ".endr\n\t"
                 "s_load_dword %0, %1, %c3\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&s"(word)
                 : "s"(args), "n"((sizeof(Args) + 63) / 64), "n"(sizeof(Args) - 4));
    asm volatile("" ::"s"(word));
}

struct FwdParams {
    const __bf16 *q;
    const __bf16 *k;
    const __bf16 *v;
    __bf16 *out;
    float *lse;
    // element strides of batch entry, head and row; the head dimension is contiguous
    long long q_sb, q_sh, q_sn;
    long long k_sb, k_sh, k_sn;
    long long v_sb, v_sh, v_sn;
    long long o_sb, o_sh, o_sn;
    long long lse_sb, lse_sh;  // rows contiguous
    // packed variable-length batches: device arrays of B + 1 row offsets along the row
    // axis (sequence b owns rows [cu[b], cu[b+1])), batch strides unused; or null
    const int *cu_q;
    const int *cu_k;
    // per-sequence prompt lengths (device, B ints) in place of P below, or null
    const int *n_prompts;
    // paged key/value cache (pipelined kernel only), or block_table null: token j of sequence b
    // lives in page block_table[b * bt_stride + j / page_size], row j % page_size; k, v then point
    // at page 0 and k_sb, v_sb are the page strides.  page_size is a multiple of 16.
    const int *block_table;
    int bt_stride, page_size, num_pages;
    int fp16;  // the 16-bit elements of q, k, v, out are IEEE binary16 instead of bfloat16
    int B, Hq, Hkv;
    int Nq, Nk;  // query rows and keys per sequence (the largest ones when cu_q / cu_k are given)
    int W, S;    // clamped to [1, Nk] and [0, Nk]
    int P;       // rows at positions >= P are generated tokens and see every earlier key; clamped to [0, Nk]
    int G;       // Hq / Hkv
    float scale, scale_log2;
    // Work decomposition.  Per (batch, KV head) "pair" the G query heads are
    // cut into n4 groups of 4 heads, at most one group of 2 heads and at most
    // one single head; a workgroup is wg_rows query rows (head x position) on one
    // KV head: 4 heads x wg_rows/4 positions, 2 x wg_rows/2 or 1 x wg_rows.
    int wg_rows;  // kFwdWgRows (forward kernels) or 256 (backward kernels)
    int n4, has2, has1;
    int nt_h4, nt_h2, nt_h1;  // row tiles of a sequence of Nq rows for workgroups of 4, 2 and 1 heads
    FastDiv div_tiles_per_pair, div_hkv, div_nt_h4;  // for the work-list decode of every workgroup
    FastDiv div_page;  // page_size (paged caches)
    int tiles_per_pair;
    int die_shift, die_pairs, die_items, fold;  // which items a die takes, and in which order (plan_work)
    FastDiv div_die_pairs;
    long long total_items;
    long long chunk;  // work items per XCD
    // Packed batches whose total number of query rows the caller has stated: the work list holds
    // every sequence's own row tiles, one sequence after the other (no items for rows a shorter
    // sequence does not have); total_items and chunk are then upper bounds, the workgroups work
    // out the true ones from cu_q / cu_k (decode_work_packed).
    int packed_compact;
    long long total_rows;  // query rows of the whole packed batch (packed_compact)
    // Split keys (plan_fwd_split, and swaa_fwd_split.h on the device): the tiles of a sequence are cut into
    // several workgroups along the keys, whose partial results a second kernel merges.
    // 0: not split; 1: the split counts are worked out on the device from the sequences'
    // lengths; >= 2: this many for every sequence (fixed-length batches); -1: whole keys, and no merge
    // (fixed-length batches of few rows, swaa_fwd_few_rows.h).
    int split_keys;
    int few_only;  // the host expects no splits: the plan is for the sake of few rows, and may be dropped
    // One sequence whose lengths the host knows as upper bounds (split_keys 1): how many splits it gets if it is as long as they say
    // (0: the host makes no plan), and what it then costs (SplitSeq); the device plans for any other.
    int bound_splits, bound_cost;
    long long split_items;  // upper bound on the row tiles (times KV heads) of the batch
    int split_cap;  // partial results the workspace holds
    float *ws_o;    // [split_cap][4 waves][16][64 lanes][4]: unnormalised O in accumulator order
    float *ws_ml;   // [split_cap][4 waves][2][32]: reference (log2 units) and row sum
    int *ws_n;      // [64]: split count of each sequence, for the merge kernel
};

// One sequence as a workgroup sees it: the query rows are the newest nq of its nk
// tokens (row r sits at position nk - nq + r; nq = nk for a plain prefill).
struct SeqGeom {
    int nq, nk;
    int n_prompt;  // rows at positions >= n_prompt are generated tokens
    long long q_row0, k_row0;  // first row along the row axis of q / out / lse and of k / v
    long long q_batch, k_batch;  // batch index to multiply the batch strides with
};
__device__ __forceinline__ bool seq_geom(const FwdParams &p, int b, SeqGeom &g) {
    if (p.cu_q) {
        g.q_row0 = p.cu_q[b];
        g.nq = p.cu_q[b + 1] - (int)g.q_row0;
        g.q_batch = 0;
    } else {
        g.q_row0 = 0;
        g.nq = p.Nq;
        g.q_batch = b;
    }
    if (p.cu_k) {
        g.k_row0 = p.cu_k[b];
        g.nk = p.cu_k[b + 1] - (int)g.k_row0;
        g.k_batch = 0;
        if (p.block_table) g.k_row0 = 0;  // a paged cache: the offsets only give the lengths
    } else if (p.block_table) {
        g.k_row0 = 0;
        g.nk = p.Nk;
        g.k_batch = 0;
    } else {
        g.k_row0 = 0;
        g.nk = p.Nk;
        g.k_batch = b;
    }
    g.n_prompt = p.n_prompts ? max(p.n_prompts[b], 0) : p.P;
    g.nq = min(min(g.nq, p.Nq), g.nk);  // never more rows than the plan covers, nor than tokens
    g.nk = min(g.nk, p.Nk);
    return g.nq > 0;
}

// What one workgroup computes.
struct WorkItem {
    int b, kvh;  // batch entry, KV head
    int hpb;     // query heads in this workgroup: 4, 2 or 1
    int h0;      // first of them, relative to the GQA group
    int pt;      // row tile of 256/hpb rows
};

// Inclusive prefix sum of x over the 64 lanes of a wave, all of them active: four shift-and-add
// steps inside each row of 16 lanes (a lane without a source adds 0), then lane 15 of rows 0 and 2
// into rows 1 and 3, then lane 31 into rows 2 and 3 -- data-parallel-primitive operands of the
// vector adds, no trip through the LDS crossbar as with the shuffle functions.
__device__ __forceinline__ unsigned wave_inclusive_scan(unsigned x) {
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);  // row_shr:8
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15, rows 1 and 3
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31, rows 2 and 3
    return x;
}
// Lane `src` (the same in all lanes) of x, as a uniform value.
__device__ __forceinline__ unsigned wave_read_lane(unsigned x, int src) {
    return (unsigned)__builtin_amdgcn_readlane((int)x, src);
}

// The work list of a packed batch, sequence by sequence: sequence b of nq_b query rows (the
// smaller of its rows, the plan's Nq and its keys -- what seq_geom makes of it) has Hkv pairs of
// n4 ceil(nq_b / r4) + has2 ceil(nq_b / r2) + has1 ceil(nq_b / r1) row tiles, r4 = wg_rows / 4
// and so on.  EVERY sequence's items are cut into eight contiguous chunks, one per XCD (XCD x
// works through chunk x of sequence 0, then chunk x of sequence 1, ...): the sequences' caches
// differ in length, so a chunk of the whole list would leave the long ones to one or two dies.
// Every wave reads the sequence lengths (64 per round, one per lane) and finds the sequence
// that holds its slot by a prefix sum of the chunk lengths over the lanes.
__device__ __forceinline__ bool decode_work_packed(const FwdParams &p, WorkItem &w) {
    const int lane = threadIdx.x & 63;
    const unsigned bid = blockIdx.x;
    const unsigned xcd = bid % kXcds, slot = bid / kXcds;
    const int s1 = p.wg_rows == 128 ? 7 : 8;  // log2 of the rows of a one-head tile (two heads: half, four: a quarter)
    auto rows_of = [&](int b) {  // nq_b of sequence b (0 for b >= B)
        if (b >= p.B) return 0;
        const int nq = p.cu_q[b + 1] - p.cu_q[b];
        const int nk = p.cu_k[b + 1] - p.cu_k[b];
        return max(0, min(min(nq, p.Nq), min(nk, p.Nk)));
    };
    auto tiles_of = [&](int nq) {  // row tiles of one pair
        return (unsigned)(p.n4 * ((nq + (1 << (s1 - 2)) - 1) >> (s1 - 2)) + p.has2 * ((nq + (1 << (s1 - 1)) - 1) >> (s1 - 1)) +
                          p.has1 * ((nq + (1 << s1) - 1) >> s1));
    };
    unsigned before = 0;
    for (int c0 = 0; c0 < p.B; c0 += 64) {
        const int nq = rows_of(c0 + lane);
        const unsigned incl = wave_inclusive_scan((tiles_of(nq) * (unsigned)p.Hkv + kXcds - 1) / kXcds);  // slots of this XCD up to and with the lane's sequence
        const unsigned in_round = wave_read_lane(incl, 63);
        if (slot - before < in_round) {
            const unsigned rel = slot - before;
            const int n = __popcll(__ballot(incl <= rel));  // sequences among these 64 that end at or before the slot
            const unsigned base = n ? wave_read_lane(incl, n - 1) : 0u;
            // (everything below is the same in all lanes, and read from one lane so that the
            // compiler knows it and keeps addresses built from it in scalar registers)
            const int nq_u = (int)wave_read_lane((unsigned)nq, n);
            const unsigned tpp_u = tiles_of(nq_u);
            const unsigned items_u = tpp_u * (unsigned)p.Hkv;
            unsigned r = xcd * ((items_u + kXcds - 1) / kXcds) + (rel - base);  // inside sequence c0 + n
            if (r >= items_u) return false;  // (the sequence's last chunks are shorter)
            w.b = c0 + n;
            w.kvh = (int)(r / tpp_u);
            r -= (unsigned)w.kvh * tpp_u;
            const unsigned nt4 = (unsigned)((nq_u + (1 << (s1 - 2)) - 1) >> (s1 - 2));
            const unsigned nt2 = (unsigned)((nq_u + (1 << (s1 - 1)) - 1) >> (s1 - 1));
            const unsigned nt1 = (unsigned)((nq_u + (1 << s1) - 1) >> s1);
            if (r < (unsigned)p.n4 * nt4) {
                const unsigned g = r / nt4;
                w.hpb = 4;
                w.h0 = 4 * (int)g;
                w.pt = (int)(nt4 - 1 - (r - g * nt4));
                return true;
            }
            r -= (unsigned)p.n4 * nt4;
            if (p.has2 && r < nt2) {
                w.hpb = 2;
                w.h0 = 4 * p.n4;
                w.pt = (int)(nt2 - 1 - r);
                return true;
            }
            if (p.has2) r -= nt2;
            w.hpb = 1;
            w.h0 = p.G - 1;
            w.pt = (int)(nt1 - 1 - r);
            return true;
        }
        before += in_round;
    }
    return false;
}

// Workgroups reach the 8 XCDs round-robin; XCD x takes the x-th contiguous
// chunk of the work list, so the position tiles of one KV head, whose K/V
// bands overlap, run behind the same L2.  Inside a pair, long rows go first; what changes where rows differ
// in length is decided in plan_work.  Workgroup bid's pair and place in that pair's list of tiles:
__host__ __device__ __forceinline__ bool work_place(const FwdParams &p, unsigned bid, unsigned &pair, unsigned &r) {
    // (the entry points refuse work lists of 2^31 items or more: 32-bit arithmetic, whose
    // divisions cost a fraction of the 64-bit ones -- every wave of every workgroup pays them)
    const unsigned xcd = bid % kXcds, sub = xcd & ((1u << p.die_shift) - 1u);
    const unsigned slot = bid / kXcds, place = slot >= (unsigned)p.fold ? (unsigned)p.chunk - 1u - (slot - (unsigned)p.fold) : slot;
    const unsigned off = (place << p.die_shift) + sub, of_pair = fastdiv(off, p.div_die_pairs);
    const unsigned item = ((xcd >> p.die_shift) * (unsigned)p.die_pairs + (off - of_pair * (unsigned)p.die_pairs)) * (unsigned)p.die_items + of_pair;
    if (of_pair >= (unsigned)p.die_items || item >= (unsigned)p.total_items) return false;
    pair = fastdiv(item, p.div_tiles_per_pair);
    r = item - pair * (unsigned)p.tiles_per_pair;
    return true;
}
__device__ __forceinline__ bool decode_work(const FwdParams &p, WorkItem &w) {
    if (p.packed_compact) return decode_work_packed(p, w);
    unsigned pair, r;
    if (!work_place(p, blockIdx.x, pair, r)) return false;
    const unsigned hkv = (unsigned)p.Hkv;
    w.b = (int)fastdiv(pair, p.div_hkv);
    w.kvh = (int)(pair - (unsigned)w.b * hkv);
    const unsigned nt4 = (unsigned)p.nt_h4, nt2 = (unsigned)p.nt_h2;
    if (r < (unsigned)p.n4 * nt4) {
        const unsigned g = fastdiv(r, p.div_nt_h4);
        w.hpb = 4;
        w.h0 = 4 * (int)g;
        w.pt = (int)(nt4 - 1 - (r - g * nt4));
        return true;
    }
    r -= (unsigned)p.n4 * nt4;
    if (p.has2 && r < nt2) {
        w.hpb = 2;
        w.h0 = 4 * p.n4;
        w.pt = (int)(nt2 - 1 - r);
        return true;
    }
    if (p.has2) r -= nt2;
    w.hpb = 1;
    w.h0 = p.G - 1;
    w.pt = p.nt_h1 - 1 - (int)r;
    return true;
}

// log2 of the dies that share a (batch, KV head) pair, where they share one evenly: eight to one pair, four to two, two to four.
inline int die_shift(long long pairs) { return pairs == 1 ? 3 : pairs == 2 ? 2 : pairs == 4 ? 1 : 0; }

// Fills the work-decomposition fields (everything from wg_rows on) for sequences of
// `rows` query rows; needs B, Hkv, G, Nk, W and P.  False if the work list does not fit 31 bits.
// Where the rows differ much in length (a window of half the keys and more, or generated rows behind a prompt):
//   * dies that share a pair take its tiles in turn: with a contiguous part each, one has the long rows and the others are done
//     early (16 heads on 4, full attention, 8192 tokens 281 us, in turn 254; window 8192 of 16384 776, 716).  With generated rows,
//     or prompt lengths of their own, behind narrower windows the few long rows are the time in either order, and if there are
//     none the neighbours' common bands count (prompt lengths that leave no generated row, contiguous / in turn, us:
//        window, of the tokens           1/32          1/16          1/8            1/6            1/4            1/3
//        4 heads on 1   16384 tokens  28.9 / 31.2   41.4 / 47.2   72.2 / 75.4    93.3 / 92.6     131 / 127      173 / 166
//                       65536          269 / 305                   970 / 1024   1277 / 1298     1878 / 1836    2503 / 2283
//        8 on 2         16384         46.5 / 50.3   79.9 / 83.3    134 / 133     175 / 170       251 / 237      326 / 289
//                       65536          513 / 521                  1929 / 1837   2569 / 2370     3825 / 3344    4962 / 4263
//        16 on 4        65536         1007 / 1012                 3743 / 3585   4966 / 4676     7265 / 6610    9463 / 8385
//     32 generated rows, 65536 tokens, window 1/32: 912 / 935, 1020 / 1013 and 1245 / 1251);
//   * a die with several pairs takes the long rows of all of them first, not pair after pair (four sequences of 2048 tokens,
//     32 heads on 8: 139 -> 134, head dimension 64 101 -> 86; four of 4096, 40 heads on 8: 639 -> 617; its backward
//     2277 -> 2215).  Not with more than 192 tiles to a pair, whose keys no longer share the L2 (two of 8192: 934, 951).
//     Where the heads of a pair make tiles of several kinds, the long rows of one kind stand behind the short ones of another,
//     and a list of 45 to 63 tiles, which is not folded, puts them beside the longest (pair after pair / long rows of all first,
//     24 heads on 8: two of 1150 tokens, 54 tiles, 30.3 / 33.8, four of 584, 60 tiles, 21.9 / 24.6; 48 on 8, two of 503, 48 tiles, 19.1 / 20.0):
//     pair after pair there.  Shorter lists have few seconds (40 on 8, two of 430, 36 tiles, 20.6 / 17.0 on half the keys), longer ones more rounds;
//   * where a die's list is one round of two workgroups to a compute unit, its second half is turned round, so that the longest
//     is not beside the longest of the rest but beside the shortest (2048 tokens 44.8 -> 41.7; four sequences of 500 21.2 ->
//     18.1, two of 4000, 8 heads on 8, 90.8 -> 74.2; with the line above).
// Rows of one length stay in contiguous parts, whose bands one L2 holds (4 heads on 1, window 2048, 65536 tokens
// 250 us, in turn 305).
inline bool plan_work(FwdParams &p, int rows, int wg_rows) {
    p.wg_rows = wg_rows;
    p.n4 = p.G / 4;
    p.has2 = (p.G % 4) >= 2 ? 1 : 0;
    p.has1 = p.G % 2;
    p.nt_h4 = (rows + wg_rows / 4 - 1) / (wg_rows / 4);
    p.nt_h2 = (rows + wg_rows / 2 - 1) / (wg_rows / 2);
    p.nt_h1 = (rows + wg_rows - 1) / wg_rows;
    p.tiles_per_pair = p.n4 * p.nt_h4 + p.has2 * p.nt_h2 + p.has1 * p.nt_h1;
    p.packed_compact = 0;
    p.total_items = (long long)p.B * p.Hkv * p.tiles_per_pair;
    const bool rows_differ = 2LL * p.W >= p.Nk || p.P < p.Nk || p.n_prompts;
    const long long pairs = (long long)p.B * p.Hkv;
    const bool in_turn = 2LL * p.W >= p.Nk || (rows_differ && (pairs == 1 ? 4LL : 8LL) * p.W >= p.Nk);
    p.div_tiles_per_pair = make_fastdiv((unsigned)p.tiles_per_pair);
    p.div_hkv = make_fastdiv((unsigned)p.Hkv);
    p.div_nt_h4 = make_fastdiv((unsigned)p.nt_h4);
    p.chunk = (p.total_items + kXcds - 1) / kXcds;
    p.die_shift = in_turn ? die_shift(pairs) : 0;
    const int kinds = (p.n4 > 0) + p.has2 + p.has1;  // of tiles: of four, two and one head
    const bool beside_long = kinds > 1 && p.chunk > 44 && p.chunk < 64;
    p.die_pairs = rows_differ && pairs % kXcds == 0 && p.tiles_per_pair <= 192 && !beside_long ? (int)(pairs / kXcds) : 1;
    p.div_die_pairs = make_fastdiv((unsigned)p.die_pairs);
    p.die_items = p.die_shift || p.die_pairs > 1 ? p.tiles_per_pair : (int)p.chunk;  // (times die_pairs, shared by the dies: chunk)
    p.fold = p.chunk <= 64 && rows_differ && p.n4 + p.has2 + p.has1 == 1 ? 32 : 0x7fffffff;
    return p.chunk * kXcds <= 0x7fffffffLL;
}

// Keys that the longest row of a whole prompt sees, and the pairs of all rows of a head (as swaa_visible_pairs_fa_decode counts them).
inline long long longest_row(const FwdParams &p) { return p.P < p.Nk || (long long)p.W + p.S > p.Nk ? p.Nk : (long long)p.W + p.S; }
inline double pairs_of_rows(const FwdParams &p) {
    const double n = (double)(p.P < p.Nk ? p.P : p.Nk), w = (double)p.W < n ? (double)p.W : n, all = (double)p.Nk;
    const double more = n - w, ramp = (double)p.S < more ? (double)p.S : more;  // rows behind the first window, and those that see less than all sinks beside it
    return w * (w + 1) / 2 + more * w + ramp * (ramp + 1) / 2 + (more - ramp) * (double)p.S + (all * (all + 1) - n * (n + 1)) / 2;
}

// Is the chain of the longest row what the call takes?  Its halves against those of `group` rows that one of `resident` workgroups
// gets on average (the quotient that the rules' tables name): at least `line`, and at least `narrow` with ten halves more for every
// 32 rows, what a workgroup of 32 rows costs outside its loop.  Without these, narrow windows, whose workgroups are little else,
// came out wrong (us, rows together / a head's 32 rows: 8 x 16 heads on 4, 2285 tokens, window 67, one generated row, quotient 7.2:
// 57.9 / 120; D = 64, 8 x 32 on 8, 1600, window 123, 14 generated rows, 3.8: 43.5 / 79.4; backward, D = 64, 8 x 16 on 4, 2195,
// window 342, one, 3.2: 154 / 198).  Of 782 to 870 calls per rule, drawn around the lines (400 to 60000 tokens, windows from 64 on, up to
// 1000 sinks, 8 to 40 heads, 4 on 1), the kernel that it picks is slower than rows together by more than 5 % in 2 (forward, D = 128), 11
// (D = 64), 6 and 9 (backward), by the quotient alone 21, 14, 10 and 23; on average it is 1.0 to 1.7 % behind the better one.
inline bool chain_is_the_time(const FwdParams &p, double resident, int group, double line, double narrow) {
    const double pairs = pairs_of_rows(p), begins = 10.0 * 32 * (double)p.Nk;
    const double need = line * pairs > narrow * (pairs + begins) ? line * pairs : narrow * (pairs + begins);
    return (double)(longest_row(p) / 32) * (resident * group * 32) >= need * (double)p.B * p.Hq;
}

// The plan of a packed batch of B sequences with total_rows query rows in all (each at most
// `rows` long): the compact work list of decode_work_packed, bounded from above -- a sequence
// adds at most one partly filled tile per head group to total_rows / tile rows, and at most one
// slot per XCD for the rounding of its eight chunks.
inline bool plan_work_packed(FwdParams &p, int rows, int wg_rows, long long total_rows) {
    if (!plan_work(p, rows, wg_rows)) return false;
    if (wg_rows != 128 && wg_rows != 256) return true;  // (decode_work_packed knows these two; else the plain list)
    auto bound = [&](int tile_rows) { return (total_rows + tile_rows - 1) / tile_rows + p.B; };
    const long long tiles = p.n4 * bound(wg_rows / 4) + p.has2 * bound(wg_rows / 2) + p.has1 * bound(wg_rows);
    const long long items = (long long)p.Hkv * tiles;
    p.packed_compact = 1;
    p.total_rows = total_rows;
    p.chunk = (items + kXcds - 1) / kXcds + p.B;
    p.total_items = p.chunk * kXcds;
    return p.total_items <= 0x7fffffffLL;
}

// Row block [p0, p0 + rows): a key is inside the window of every prompt row of
// the block iff it lies above the returned bound (last prompt row minus W); a
// block of generated tokens only has no such bound.
__device__ __forceinline__ int window_bound(int p0, int rows, int W, int P) {
    return p0 >= P ? -(1 << 30) : min(p0 + rows - 1, P - 1) - W;
}

// The mask of 32 keys k0 .. k0 + 31 for a row at position qpos, as bits: bit j says whether it sees key k0 + j.
// Three comparisons, two logical operations and a selection per score were 120 to 170 instructions for a half, and their
// results, a pair of scalar registers each, spilled (forward of whole keys 88 to 110 scalar registers, now 0 to 3; split keys 164 to
// 172, now 42 to 65); from the word it is two per score (54 in all; us: four prompts of 643
// tokens 16.2 -> 14.6, seven packed ones of 0.1-7k on a window of 1024 73.1 -> 67.7, four of 8192 on 1024 681 -> 672).
__host__ __device__ __forceinline__ uint32_t keys_below(int n) {  // the first n keys (none below 0, all from 32 on)
    return n >= 32 ? ~0u : (1u << ((n > 0 ? n : 0) & 31)) - 1u;
}
__host__ __device__ __forceinline__ uint32_t visible_keys(int k0, int qpos, int W, int S) {
    return keys_below(qpos + 1 - k0) & (~keys_below(qpos + 1 - W - k0) | keys_below(S - k0));
}
// A lane's 16 scores of a 32 x 32 product belong to keys 8 (e / 4) + 4 hf + e % 4: x where element e's bit is set in
// bits = visible_keys(...) >> 4 hf, -infinity where it is not.
__device__ __forceinline__ float where_visible(uint32_t bits, int e, float x) {
    const uint32_t all = (uint32_t)((int)(bits << (31 - (8 * (e / 4) + e % 4))) >> 31);
    return __uint_as_float((all & __float_as_uint(x)) | (~all & 0xff800000u));
}

// Is x infinite or not a number?  On the bits, and behind the optimiser's back: the build does not honour NaNs
// (-fno-honor-nans), and a comparison, or a test of the bits that the compiler recognises, would be folded.
__device__ __forceinline__ uint32_t opaque_bits(float x) {
    uint32_t bits = __float_as_uint(x);
    asm("" : "+v"(bits));
    return bits;
}
__device__ __forceinline__ bool non_finite(float x) { return (opaque_bits(x) & 0x7fffffffu) >= 0x7f800000u; }

// Lanes l and l^32 hold partial results for the same query column.
__device__ __forceinline__ float half_swap_max(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_swap_sum(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// More than 64 KiB of LDS per workgroup has to be requested once per device.
template <auto kernel, int kBytes>
hipError_t allow_lds() {
    static std::atomic<unsigned long long> configured{0};
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    const unsigned long long bit = 1ull << (dev & 63);
    if (configured.load(std::memory_order_acquire) & bit) return hipSuccess;
    err = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kBytes);
    if (err == hipSuccess) configured.fetch_or(bit, std::memory_order_release);
    return err;
}

// Launchers (one per kernel family); return the HIP error of the launch.
// (the plain kernel: head dimensions 32 .. 256 in steps of 32 except 64 and 128)
hipError_t launch_fwd_simple(const FwdParams &p, int D, hipStream_t stream);
hipError_t launch_fwd_d64(const FwdParams &p, hipStream_t stream);
hipError_t launch_fwd_pipelined_d128(const FwdParams &p, hipStream_t stream);
// Decides whether the call's keys are split over several workgroups per row tile and fills the
// split_* fields (after plan_work / plan_work_packed, whose launch size it enlarges); the bytes of
// workspace the plan needs, 0 if the keys stay whole.
long long plan_fwd_split(FwdParams &p);
void place_fwd_split(FwdParams &p, void *workspace);

}  // namespace swaa

#endif  // SWAA_COMMON_H_
