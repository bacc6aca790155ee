// Forward of short prompts, head dimension 128, gfx950: sequences of one length whose row tiles do not fill
// the chip.  Mask and results as in swaa_fwd_pipelined.hip.
//
// A workgroup of the pipelined kernel is 128 rows of up to four heads whose four waves walk the same keys one after
// the other: a prompt of 317 tokens on 32 heads is 80 of them, a third of the compute units, and the longest
// walks ten halves of 32 keys.  What bounds such a call is that chain, not the chip.  Here a workgroup is 32 rows of ONE
// head and its four waves take a quarter of the keys each (as in swaa_fwd_few_rows.h: a ring of one half of their own,
// no barriers in the loop, the registers as the second stage, max-based softmax), so that four times as many
// workgroups walk a quarter of the keys; the four results are added up through LDS behind one barrier, and whole rows are
// stored (three barriers and eight bytes per row and store before: 512 tokens 10.4 -> 9.9 us, 317 8.6 -> 8.4).  Each workgroup reads its keys
// for itself, four times the traffic of the pipelined kernel out of L2, which is what ends its use
// (plan_fwd_short has both sides of the line).
//
// No static LDS: the dynamic LDS starts at address 0.
#include <type_traits>

#include "swaa_fwd_short.h"
#include "swaa_tile_d128.h"

namespace swaa {
namespace {

constexpr int kSWaves = 4, kSThreads = 64 * kSWaves;
constexpr int kSRows = 32;                         // query rows of a workgroup
constexpr uint32_t kSRing = 2 * kHalfBytes;        // a wave's: K half, then V half
constexpr uint32_t kSMl = kSWaves * kSRing;        // what the waves' results are weighted with (leave_result)
constexpr int kSBytes = kSWaves * ((int)kSRing + 512);

template <bool kF16>
__global__ __launch_bounds__(kSThreads, 2) void swaa_fwd_short_kernel(const FwdShortParams sp) {
    fetch_args<FwdShortParams>();
    const FwdParams &p = sp.f;
    constexpr int kBelow = kF16 ? 4 : 0;  // as the row tiles' reference: terms keep full precision down to 2^-18 of it
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int l32 = lane & 31, hf = lane >> 5;
    // Long rows first; the (batch, KV head) pair innermost: where the pairs are a multiple of eight, each die
    // keeps to its own, and where they are not, every die gets long and short rows of all.
    const unsigned by_pair = fastdiv(blockIdx.x, sp.div_pairs), pair = blockIdx.x - by_pair * (unsigned)sp.pairs;
    const unsigned by_group = fastdiv(by_pair, sp.div_group), g = by_pair - by_group * (unsigned)p.G;
    const int b = (int)fastdiv(pair, p.div_hkv), kvh = (int)pair - b * p.Hkv;
    const int head = kvh * p.G + (int)g;
    const int r0 = kSRows * (sp.tiles - 1 - (int)by_group);  // first query row
    const int N = p.Nq, S = p.S;  // (whole prompts: as many keys)
    const int n_prompt = p.n_prompts ? max(p.n_prompts[b], 0) : p.P;
    const int p1 = min(r0 + kSRows, N) - 1;  // last row
    const int row = min(r0 + l32, N - 1);             // this lane's column
    const int W = row >= n_prompt ? N : p.W;

    // ---- the schedule, in halves of 32 keys: sinks, then the band; a quarter of them is this wave's ----
    const int band_lo = p1 >= n_prompt ? 0 : max(0, r0 - p.W + 1);
    const int hb_lo = band_lo >> 5, hb_hi = p1 >> 5;
    const int n_sink = min((min(S, band_lo) + 31) >> 5, hb_lo);
    const int n_all = n_sink + (hb_hi - hb_lo + 1);
    const int quarter = (n_all + kSWaves - 1) / kSWaves;
    const int h_mine = wave * quarter;
    const int n_mine = max(0, min(quarter, n_all - h_mine));
    auto first_key = [&](int t) __attribute__((always_inline)) {
        const int h = h_mine + t;
        return 32 * (h < n_sink ? h : h - n_sink + hb_lo);
    };

    // ---- HBM -> LDS copies of one half: instruction i moves rows 4 i .. 4 i + 3, swizzled on the global side.  Rows
    // past the sequence's last key repeat it (they are masked later). ----
    const uint32_t k_rsb = (uint32_t)(p.k_sn * 2), v_rsb = (uint32_t)(p.v_sn * 2);
    const char *kg = reinterpret_cast<const char *>(p.k + b * p.k_sb + kvh * p.k_sh);
    const char *vg = reinterpret_cast<const char *>(p.v + b * p.v_sb + kvh * p.v_sh);
    const int lrow = lane >> 4, lchk = lane & 15;
    const uint32_t ring = (uint32_t)wave * kSRing;
    // (the eight copies of an operand share one M0 value per four and use the instruction's offset field, 1024 i, which
    // moves the LDS address and the global address alike: the lane's offset gives it back)
    uint32_t koff[8], voff[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t r = (uint32_t)(4 * i + lrow);
        const int fk = ((4 * (i & 1) + lrow) << 1) | ((i >> 1) & 1);
        koff[i] = r * k_rsb + (uint32_t)((lchk ^ fk) << 4) - (uint32_t)(1024 * (i & 3));
        voff[i] = r * v_rsb + (uint32_t)((lchk ^ (lrow << 2)) << 4) - (uint32_t)(1024 * (i & 3));
    }
    auto copy4 = [](const uint32_t *vo, const char *base, uint32_t lds) __attribute__((always_inline)) {
        asm volatile(
            "s_mov_b32 m0, %5\n\ts_nop 0\n\t"
            "global_load_lds_dwordx4 %0, %4\n\t"
            "global_load_lds_dwordx4 %1, %4 offset:1024\n\t"
            "global_load_lds_dwordx4 %2, %4 offset:2048\n\t"
            "global_load_lds_dwordx4 %3, %4 offset:3072" ::"v"(vo[0]),
            "v"(vo[1]), "v"(vo[2]), "v"(vo[3]), "s"(base), "s"(lds)
            : "memory");
    };
    auto issue = [&](bool is_k, int k0) __attribute__((always_inline)) {
        const uint32_t rsb = is_k ? k_rsb : v_rsb, lds = ring + (is_k ? 0u : (uint32_t)kHalfBytes);
        const char *base = (is_k ? kg : vg) + (size_t)k0 * rsb;
        const uint32_t *vo = is_k ? koff : voff;
        if (__builtin_expect(k0 + 32 > N, 0)) {
            // (no offset field: a clamped row may lie less than 1024 i bytes behind the half's first)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t off = vo[i] + (uint32_t)(1024 * (i & 3)) - (uint32_t)max(k0 + 4 * i + lrow - (N - 1), 0) * rsb;
                asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base),
                             "s"(lds + (uint32_t)(i * 1024))
                             : "memory");
            }
        } else {
            copy4(vo, base, lds);
            copy4(vo + 4, base, lds + 4096u);
        }
    };
    const LaneAddr la = make_lane_addr(lane, 0);

    // ---- the first half, then this lane's Q fragments (ordinary loads: the compiler's wait covers the copies as well) ----
    if (n_mine > 0) {
        issue(true, first_key(0));
        issue(false, first_key(0));
    }
    bf16x8 qf[kKS];
    {
        const char *qrow = reinterpret_cast<const char *>(p.q + b * p.q_sb + head * p.q_sh + row * p.q_sn) + 16 * hf;
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(qrow + 32 * ks);
    }
    asm volatile("s_nop 1"
                 : "+a"(qf[0]), "+a"(qf[1]), "+a"(qf[2]), "+a"(qf[3]), "+a"(qf[4]), "+a"(qf[5]), "+a"(qf[6]), "+a"(qf[7]));

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
    const int wbound = window_bound(r0, kSRows, p.W, n_prompt);

    for (int t = 0; t < n_mine; ++t) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // half t has landed
        const int k0h = first_key(t);
        const bool masked = !((k0h + 31 <= r0) && ((k0h > wbound) || (k0h + 31 < S)));
        // all fragments to registers, then the next half's copy into the same ring, then the arithmetic
        bf16x8 kf[kKS], vf[2][kDB];
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) kf[ks] = load_k_frag(la, ring, ks);
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int db = 0; db < kDB; ++db) vf[st][db] = load_v_frag(la, ring + kHalfBytes, st, db);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (t + 1 < n_mine) {
            issue(true, first_key(t + 1));
            issue(false, first_key(t + 1));
        }
        f32x16 s;
        bf16x8 pf[2];
        float alpha;
        mfma_s_first<kF16>(s, kf[0], qf[0]);
#pragma unroll
        for (int ks = 1; ks < kKS - 1; ++ks) mfma_s<kF16>(s, kf[ks], qf[ks]);
        mfma_s_settled<kF16>(s, kf[kKS - 1], qf[kKS - 1]);
        if (masked)
            softmax_half<true, kF16, kBelow>(s, k0h, row, W, S, hf, c2, rs, pf, alpha);
        else
            softmax_half<false, kF16, kBelow>(s, k0h, row, W, S, hf, c2, rs, pf, alpha);
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

    // ---- the four waves' results through LDS; 32 threads take a row and store it whole ----
    leave_result((uint32_t)wave * kSRing, kSMl + (uint32_t)(wave * 512), l32, hf, true, oacc, rs);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSRows / 8; ++i) {
        const int c = 8 * i + (int)(threadIdx.x >> 5), q = (int)(threadIdx.x & 31);
        if (r0 + c >= N) break;
        float m, l;
        f32x4_t o4 = add_results(0u, kSRing, kSMl, c, q, m, l);
        o4 *= 1.f / l;
        const bf16x2 lo = pack_pair<kF16>(o4[0], o4[1]), hi = pack_pair<kF16>(o4[2], o4[3]);
        *reinterpret_cast<bf16x4 *>(p.out + b * p.o_sb + head * p.o_sh + (long long)(r0 + c) * p.o_sn + 4 * q) = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
        if (q == 0) p.lse[b * p.lse_sb + head * p.lse_sh + r0 + c] = (m + __builtin_amdgcn_logf(l)) * 0.69314718055994530942f;
    }
}

}  // namespace

// One round of workgroups, two to a compute unit: with more of them the chip is full either way, and rows that share their
// keys read less.  Pipelined / short (us a call from a captured graph; bfloat16, full attention unless stated):
//    units            160           256           320           512                640           1024
//    32 heads on 8                                11.5 / 9.5    14.0 / 11.6                      21.4 / 24.4
//    16 heads on 4    11.2 / 8.6    13.7 / 9.8                  20.5 / 15.3        24.4 / 20.0   35.0 / 35.6
//      window 1024                                                                 21.5 / 19.8   23.1 / 29.5
//    8 heads on 8                   21.3 / 13.3   24.3 / 16.6   34.3 / 23.3        (752: 46.2 / 35.4, window 1024 27.0 / 28.0)
//    4 heads on 1     23.0 / 14.9   32.6 / 20.6                 57.6 / 38.5 (500; window 1024 21.8 / 20.0)
//    40 heads on 8    9.0 / 6.9                                 11.7 / 9.8 (400)   15.2 / 16.6
//    4 x 32 on 8                                                8.9 / 8.8 (128 tokens: the chains are short either way)
// Up to 64 keys there is nothing to share out (32 heads on 8 6.8 / 6.7, 8 on 8 6.3 / 6.4).  Chunks on longer caches are left to
// the plan of split keys (plan_fwd_split), and to the pipelined kernel without a workspace: one result however they are called.  A
// whole prompt's bits depend on this rule: every wave here has a softmax reference of its own, so P is rounded elsewhere than in row
// tiles (relative error against 64 bits, mean over 24 calls: bfloat16 0.00196, row tiles 0.00202; binary16 0.000245, 0.000253).
//
// More units, or longer ones, where the chain of the longest row is what the call takes: its halves against the halves of 128
// rows that one of the 512 resident workgroups gets on average (a quotient), from 3.6 on where windows are not narrow
// (chain_is_the_time).  Generated rows behind a prompt above all.  Pipelined / short (us; 512 generated rows unless stated):
//    8 on 8, 4000 tokens, window 1024, 6.6:  66.0 / 39.1   20000, 5.6: 386 / 200    10374, window 2048, 3.7: 208 / 164
//    4 on 1, 8000, full attention, none, 4.1: 108 / 95.3   8 on 8, 4096, full, none, 4.0: 59.4 / 54.7
//    16 on 4, 3000, window 1024, 3.6:        52.2 / 52.8   2 x 8 on 8, 9000, 2.9: 189 / 180   16 on 4, 16384, 2.8: 273 / 322
//    8 on 8, 3000, window 1024, none, 3.3:   23.8 / 27.9   16 on 4, 2500, full, none, 3.3: 41.1 / 48.6
// Calls of the general form stay on row tiles there: above 4096 tokens, or with more than one round of units, they give a
// contiguous cache the bits of the same call on a paged one.
bool plan_fwd_short(const FwdParams &p, bool general, FwdShortParams &sp) {
    const long long tiles = (p.Nq + kSRows - 1) / kSRows;
    if (p.cu_q || p.block_table || p.Nq != p.Nk || p.Nk <= 64) return false;
    if (p.Nk > 4096 || (long long)p.B * p.Hq * tiles > 512) {
        if (general || (long long)p.B * p.Hq * tiles > 0x7fffffffLL) return false;
        if (longest_row(p) < 72 * 32 || !chain_is_the_time(p, 512, 128, 3.6, 2.35)) return false;
    }
    static_assert(kSRows == 32, "fill_fwd_short's units");
    fill_fwd_short(p, sp);
    return true;
}

hipError_t launch_fwd_short_d128(const FwdShortParams &sp, hipStream_t stream) {
    const dim3 grid((unsigned)(sp.pairs * sp.f.G * sp.tiles));
    auto launch = [&](auto f16) {
        constexpr auto kernel = swaa_fwd_short_kernel<decltype(f16)::value>;
        const hipError_t err = allow_lds<kernel, kSBytes>();
        if (err != hipSuccess) return err;
        hipLaunchKernelGGL(kernel, grid, dim3(kSThreads), kSBytes, stream, sp);
        return hipGetLastError();
    };
    return sp.f.fp16 ? launch(std::true_type{}) : launch(std::false_type{});
}

}  // namespace swaa
