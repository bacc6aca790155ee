// Sequences of few query rows in the split-key forward: generated tokens in a serving batch.
//
// A row tile of the forward kernel is 32 positions of one to four heads.  A generated token fills one
// position of it, and every wave walks the whole cache for its one valid row: 23 tokens on caches of
// 1-12k tokens took more matrix and vector time than the chunk of 999 rows beside them.  Where the
// G x nq rows of a (sequence, KV head) pair fit one column tile (few_rows), the pair is ONE tile, as in
// the decode kernel: all rows are columns of the same 32 x 32 products, the four waves take a quarter of
// the split's keys each, with a ring of one half (K 8 KiB + V 8 KiB) of their own and no barriers in the
// loop, and their results are added up through LDS.  What bounds it is reading: every key once (466 MB fetched, 470
// by count), at 4.1 TB/s beside a chunk and 5.0 alone of 6.4 for large reads; asking for a half's K before its V is read
// changed nothing.  The softmax is max-based, so there is
// no second pass.  The registers (two workgroups per CU) are those of the forward.
// Measured, row tiles -> this (binary16, pages of 16 tokens): 23 tokens on 1-12k keys beside a chunk of 999 rows on a
// window of 2k, 32 heads on 8, 141 -> 123 us (470 MB: 74 us at the rate of large reads); 31 tokens on 3-28k keys
// beside 500 rows, 40 heads on 8 (five heads were two tiles, each reading the keys) 362 -> 268, 32 heads on 8 266 -> 247;
// 23 tokens alone, 16 heads on 4, 52 -> 48.  Calls that read at HBM's rate in row tiles gain nothing (31 tokens alone, 8 heads on
// 8: 233 -> 233), and whole keys may lose by the way their units fall on the compute units (few_in_row_tiles has the worst of
// it, up to 21 %): 64 sequences on 8000 keys 346 -> 350, 49 on 16 KV heads and 3840 keys 278 -> 293 (64 on 1100 57 -> 53, 16 heads on
// 4 35 -> 26).
#ifndef SWAA_FWD_FEW_ROWS_H_
#define SWAA_FWD_FEW_ROWS_H_

#include "swaa_fwd_split.h"
#include "swaa_tile_d128.h"

namespace swaa {

// LDS of such a workgroup: the four rings, then what the waves' results are weighted with.
constexpr int kFewSmemBytes = 4 * (2 * kHalfBytes + 512);

// One workgroup of four waves on split si of the few-row sequence of wi.  LDS: kFewSmemBytes from address 0.
template <bool kF16, bool kPaged>
__device__ __forceinline__ void few_rows_item(const FwdParams &p, const WorkItem &wi, const SplitItem &si, const SeqGeom &sg) {
    constexpr uint32_t kRing = 2 * kHalfBytes;  // a wave's: K half, then V half
    constexpr int kBelow = kF16 ? 4 : 0;  // as the row tiles' reference: terms keep full precision down to 2^-18 of it
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int l32 = lane & 31, hf = lane >> 5;
    const int Nk = sg.nk, S = p.S, nq = sg.nq, cols = p.G * nq;
    const int pos_off = Nk - nq;
    // this lane's column: row c % nq of the pair's head c / nq (padding columns repeat the last one and are never stored)
    const bool col_valid = l32 < cols;
    const unsigned col = (unsigned)min(l32, cols - 1);
    const unsigned inv_nq = (65536u + (unsigned)nq - 1) / (unsigned)nq;  // col / nq = col * inv_nq >> 16: col, nq <= 32
    const unsigned hc = (col * inv_nq) >> 16;
    const int row = (int)(col - hc * (unsigned)nq);
    const int head = wi.kvh * p.G + (int)hc;
    const int qpos = pos_off + row;
    const int W = qpos >= sg.n_prompt ? Nk : p.W;

    // ---- the schedule, as the row tiles' (halves of 32 keys: sinks, then the band) ----
    const int band_lo = Nk - 1 >= sg.n_prompt ? 0 : max(0, pos_off - p.W + 1);
    const int hb_lo = band_lo >> 5, hb_hi = (Nk - 1) >> 5;
    const int n_sink = min((min(S, band_lo) + 31) >> 5, hb_lo);
    const int n_all = n_sink + (hb_hi - hb_lo + 1);
    const int per = si.n > 1 ? (((n_all + si.n - 1) / si.n) + 3) & ~3 : n_all;  // (whole quarters for the four waves)
    const int h_begin = si.s * per;
    const int n_split = min(per, n_all - h_begin);
    if (n_split <= 0) {  // (rounding up has left nothing: an empty partial result)
        if (wave == 0) p.ws_ml[(size_t)(si.slot * 4u) * 64 + lane] = hf ? 0.f : -INFINITY;
        return;
    }
    const int quarter = (n_split + 3) >> 2;
    const int h_mine = h_begin + wave * quarter;
    const int n_mine = max(0, min(quarter, n_split - wave * quarter));
    auto first_key = [&](int t) __attribute__((always_inline)) {
        const int h = h_mine + t;
        return 32 * (h < n_sink ? h : h - n_sink + hb_lo);
    };

    const uint32_t k_rsb = (uint32_t)(p.k_sn * 2), v_rsb = (uint32_t)(p.v_sn * 2);
    const char *kg = reinterpret_cast<const char *>(p.k + sg.k_batch * p.k_sb + (long long)wi.kvh * p.k_sh + sg.k_row0 * p.k_sn);
    const char *vg = reinterpret_cast<const char *>(p.v + sg.k_batch * p.v_sb + (long long)wi.kvh * p.v_sh + sg.k_row0 * p.v_sn);
    const HalfCopy half_copy(lane, k_rsb, v_rsb);
    const uint32_t ring = (uint32_t)wave * kRing;
    typedef const int __attribute__((address_space(4))) *TablePtr;  // (constant memory: scalar loads)
    const TablePtr bt = kPaged ? (TablePtr)(p.block_table + (size_t)wi.b * p.bt_stride) : nullptr;
    // Paged cache: pages are multiples of 16 tokens, so rows 0..15 of a half share a page and rows 16..31 do.  Both
    // entries are asked for one iteration before the copy that needs them.
    struct Pages {
        int a, b;
    };
    auto lookup = [&](int t) __attribute__((always_inline)) {
        Pages pg{0, 0};
        if constexpr (kPaged) {
            const int k0 = first_key(t);
            pg.a = bt[fastdiv((unsigned)k0, p.div_page)];
            pg.b = bt[fastdiv((unsigned)min(k0 + 16, Nk - 1), p.div_page)];
        }
        return pg;
    };
    auto issue_half = [&](int t, const Pages pg) __attribute__((always_inline)) {
        const int k0 = first_key(t);
        const char *kb[2], *vb[2];
        if constexpr (kPaged) {
            // (row offsets count from the half's first row: the second base steps back 16 rows; if the sequence ends
            // inside the first 16, every later row repeats its last one there.  Clamped to the cache whatever the
            // table says.)
            auto base = [&](int page, int in_page, int i) __attribute__((always_inline)) {
                page = min(max(page, 0), p.num_pages - 1);
                kb[i] = kg + ((long long)page * p.k_sb + (long long)in_page * (long long)(int)p.k_sn) * 2;
                vb[i] = vg + ((long long)page * p.v_sb + (long long)in_page * (long long)(int)p.v_sn) * 2;
            };
            base(pg.a, k0 - (int)fastdiv((unsigned)k0, p.div_page) * p.page_size, 0);
            kb[1] = kb[0];
            vb[1] = vb[0];
            if (k0 + 16 <= Nk - 1) base(pg.b, k0 + 16 - (int)fastdiv((unsigned)(k0 + 16), p.div_page) * p.page_size - 16, 1);
        } else {
            kb[0] = kb[1] = kg + (size_t)k0 * k_rsb;
            vb[0] = vb[1] = vg + (size_t)k0 * v_rsb;
        }
        half_copy.half(ring, kb, vb, Nk - 1 - k0);
    };
    const LaneAddr la = make_lane_addr(lane, 0);

    // ---- the first half and this lane's Q fragments (ordinary loads, asked for while a page of the half is looked up;
    // the compiler's wait covers the copies as well) ----
    const Pages pg_first = n_mine >= 1 ? lookup(0) : Pages{0, 0};
    if (!kPaged && n_mine >= 1) issue_half(0, pg_first);
    bf16x8 qf[kKS];
    {
        const char *qrow = reinterpret_cast<const char *>(p.q + sg.q_batch * p.q_sb + (long long)head * p.q_sh +
                                                          (sg.q_row0 + row) * p.q_sn) + 16 * hf;
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(qrow + 32 * ks);
    }
    if (kPaged && n_mine >= 1) issue_half(0, pg_first);
    asm volatile("s_nop 1"
                 : "+a"(qf[0]), "+a"(qf[1]), "+a"(qf[2]), "+a"(qf[3]), "+a"(qf[4]), "+a"(qf[5]), "+a"(qf[6]), "+a"(qf[7]));
    Pages pg_next = n_mine > 1 ? lookup(1) : Pages{0, 0};

    f32x16 oacc[kDB];
#pragma unroll
    for (int db = 0; db < kDB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[db][e] = 0.f;
    pin_acc(oacc);
    RowState rs;
    rs.mc = -INFINITY;
    rs.l = 0.f;
    rs.lb = 0.f;
    const float c2 = p.scale_log2;
    const int wbound = window_bound(pos_off, nq, p.W, sg.n_prompt);

    for (int t = 0; t < n_mine; ++t) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // half t has landed
        const int k0h = first_key(t);
        const bool masked = !((k0h + 31 <= pos_off) && ((k0h > wbound) || (k0h + 31 < S)));
        // all fragments to registers, then the next half's copy into the same ring, then the arithmetic
        bf16x8 kf[kKS], vf[2][kDB];
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) kf[ks] = load_k_frag(la, ring, ks);
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int db = 0; db < kDB; ++db) vf[st][db] = load_v_frag(la, ring + kHalfBytes, st, db);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (t + 1 < n_mine) issue_half(t + 1, pg_next);
        if (t + 2 < n_mine) pg_next = lookup(t + 2);
        f32x16 s;
        bf16x8 pf[2];
        float alpha;
        mfma_s_first<kF16>(s, kf[0], qf[0]);
#pragma unroll
        for (int ks = 1; ks < kKS - 1; ++ks) mfma_s<kF16>(s, kf[ks], qf[ks]);
        mfma_s_settled<kF16>(s, kf[kKS - 1], qf[kKS - 1]);
        if (masked)
            softmax_half<true, kF16, kBelow>(s, k0h, qpos, W, S, hf, c2, rs, pf, alpha);
        else
            softmax_half<false, kF16, kBelow>(s, k0h, qpos, W, S, hf, c2, rs, pf, alpha);
        rescale(oacc, alpha);
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int db = 0; db < kDB; ++db) {
                if (st == 1 && db == kDB - 1)
                    mfma_acc_settled<kF16>(oacc[db], vf[st][db], pf[st]);  // the accumulators are read below / next time round
                else
                    mfma_acc<kF16>(oacc[db], vf[st][db], pf[st]);
            }
    }

    // ---- the four waves' results through LDS (leave_result) ----
    constexpr uint32_t kMl = 4 * kRing;
    leave_result(ring, kMl + (uint32_t)(wave * 512), l32, hf, col_valid, oacc, rs);
    __syncthreads();
    for (int i = (int)threadIdx.x; i < 32 * cols; i += 256) {
        const int c = i >> 5, q = i & 31;  // column; its head-dimension elements 4 q ..
        float m, l;
        f32x4_t o4 = add_results(0u, kRing, kMl, c, q, m, l);
        if (si.n == 1) {
            const int h = (int)(((unsigned)c * inv_nq) >> 16);
            const long long r = sg.q_row0 + c - h * nq, hq = wi.kvh * p.G + h;
            o4 *= 1.f / l;
            const bf16x2 lo = pack_pair<kF16>(o4[0], o4[1]), hi = pack_pair<kF16>(o4[2], o4[3]);
            *reinterpret_cast<bf16x4 *>(p.out + sg.q_batch * p.o_sb + hq * p.o_sh + r * p.o_sn + 4 * q) = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
            if (q == 0) p.lse[sg.q_batch * p.lse_sb + hq * p.lse_sh + r] = (m + __builtin_amdgcn_logf(l)) * 0.69314718055994530942f;
        } else {
            // (the layout of a row tile's first wave: accumulator order)
            *reinterpret_cast<f32x4_t *>(p.ws_o + (size_t)(si.slot * 4u) * (16 * 64 * 4) + (q >> 1) * 256 + (q & 1) * 128 + c * 4) = o4;
            if (q == 0) {
                // (a sum that is not a number travels with a finite reference: -inf would mark the split as empty)
                p.ws_ml[(size_t)(si.slot * 4u) * 64 + c] = non_finite(l) ? 0.f : m;
                p.ws_ml[(size_t)(si.slot * 4u) * 64 + 32 + c] = l;
            }
        }
    }
}

}  // namespace swaa

#endif  // SWAA_FWD_FEW_ROWS_H_
