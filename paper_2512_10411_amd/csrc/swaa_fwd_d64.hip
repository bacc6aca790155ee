// SWA + sink attention forward, head dimension 64, gfx950: the mask and the entry points of the plain
// kernel, laid out for what bounds this head dimension.
//
// Per 32 x 32 scores a wave owes the matrix pipe 8 + 2 small products (288 cycles) and the vector ALU 16
// multiply-adds, exponentials (quarter rate) and sums and 8 conversions (416 cycles): the softmax is
// the bound, not the matrix pipe as at 128.  So
//   * four workgroups of four waves (32 query rows each, one KV head) share a compute unit, 128
//     registers per wave: a SIMD always has a wave with vector work;
//   * the softmax reference moves only when some score exceeds it by 2^8 (log2 units), and O is only
//     then rescaled; the search for the maximum is eight three-way maxima per half;
//   * O is divided by the sum of the ROUNDED probabilities, as they weight V: the sums come from the
//     matrix pipe, which has room;
//   * K and V travel HBM -> LDS with global_load_lds_dwordx4 into two buffers of 64 keys, one barrier
//     per tile and no staging through registers;
//   * the schedule is in halves of 32 keys (sink halves, then band halves; two consecutive ones make
//     a tile), a wave skips halves that its rows do not see and masks those on an edge.
// Measured against the plain kernel, which served this head dimension (bf16, Hq 32, Hkv 8): one prompt of
// 16k tokens, window 1024, 199 -> 175 us; four of 16k, window 1024, 816 -> 705 (740 TFLOP/s), full attention
// 4928 -> 4643 (903 TFLOP/s); one of 1000 tokens 24.2 -> 21.4.  At full attention a half costs a SIMD 640
// cycles against the 472 of its vector instructions.
//
// Rows are 128 bytes without padding; 16-byte chunk c of row r lies at chunk c ^ f(r), f(r) = (((r >> 1) & 1) << 2)
// | ((r >> 2) & 3), applied on the global side of the copy: 16 consecutive rows reading one logical chunk
// (K fragments) and 4 consecutive rows reading the same 64 bytes (transposed V fragments) are free of
// bank conflicts.  This kernel declares no static LDS: its dynamic LDS starts at address 0.
#include <type_traits>

#include "swaa_fwd_short.h"
#include "swaa_tile_d128.h"  // (softmax_half and its row state)

namespace swaa {
namespace {

constexpr int kD64 = 64;
constexpr int kKs = kD64 / 16, kDb = kD64 / 32;
constexpr int kRowB = kD64 * 2;
constexpr int kHalfB = 32 * kRowB;          // 4 KiB: one half of K, or of V
constexpr int kTileB = 4 * kHalfB;          // K half 0, K half 1, V half 0, V half 1
constexpr int kSmem64 = 2 * kTileB;         // 32 KiB
constexpr float kSlack = 8.f;  // log2 units a score may exceed its row's reference before that moves

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

template <bool kF16>
__device__ __forceinline__ f32x16 mfma32(const bf16x8 a, const bf16x8 b, const f32x16 c) {
    if constexpr (kF16)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
template <bool kF16>
__device__ __forceinline__ f32x4 mfma16(const bf16x8 a, const bf16x8 b, const f32x4 c) {
    if constexpr (kF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
template <bool kF16>
__device__ __forceinline__ __bf16 round16(float x) {  // the bits of x in the element format
    if constexpr (kF16)
        return __builtin_bit_cast(__bf16, (_Float16)x);
    else
        return (__bf16)x;
}
__device__ __forceinline__ bf16x8 lds16(uint32_t addr) {
    return *(const bf16x8 __attribute__((address_space(3))) *)(uintptr_t)addr;
}
__device__ __forceinline__ s16x4 lds8_tr(uint32_t addr) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)(uintptr_t)addr);
}

template <bool kF16>
__global__ __launch_bounds__(kThreads, 4) void swaa_fwd_d64_kernel(const FwdParams p) {
    fetch_args<FwdParams>();
    WorkItem wi;
    if (!decode_work(p, wi)) return;
    SeqGeom sg;
    if (!seq_geom(p, wi.b, sg)) return;
    const int hpb = wi.hpb;
    const int rows_per_wg = kFwdWgRows / hpb;
    const int wg_r0 = wi.pt * rows_per_wg;  // first query row of the workgroup
    if (wg_r0 >= sg.nq) return;             // a shorter sequence of a packed batch
    const int Nq = sg.nq, Nk = sg.nk, S = p.S, P = sg.n_prompt;
    const int pos_off = Nk - Nq;  // query row r sits at position pos_off + r

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, l32 = lane & 31, hf = lane >> 5;

    const int head = wi.kvh * p.G + wi.h0 + (wave % hpb);
    const int r0 = wg_r0 + (wave / hpb) * 32;      // first query row of this wave
    const int wg_p0 = pos_off + wg_r0;             // positions of the workgroup's first ...
    const int wg_p1 = pos_off + min(Nq, wg_r0 + rows_per_wg) - 1;  // ... and last valid row
    const int p0 = pos_off + r0;                   // first position of this wave
    const int plast = pos_off + min(r0 + 32, Nq) - 1;  // its last valid one
    const bool wave_active = r0 < Nq;
    const int qpos = p0 + l32;                     // this lane's query column
    const int W = (qpos >= P) ? Nk : p.W;          // a generated token (position >= P) sees its whole prefix

    // ---- this lane's Q fragments (B operand of S^T = K Q^T); they are there before the loop starts, so
    // that no wait inside it covers the tile copies ----
    bf16x8 qf[kKs];
    {
        const __bf16 *qrow = p.q + sg.q_batch * p.q_sb + (long long)head * p.q_sh + (sg.q_row0 + min(r0 + l32, Nq - 1)) * p.q_sn + 8 * hf;
#pragma unroll
        for (int ks = 0; ks < kKs; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(qrow + 16 * ks);
    }

    // ---- the schedule (as in the kernel for head dimension 128): sink halves, then the band's; an odd
    // count is padded with a half past the last row, which no row can see ----
    const int band_lo = (wg_p1 >= P) ? 0 : max(0, wg_p0 - p.W + 1);
    const int hb_lo = band_lo >> 5, hb_hi = wg_p1 >> 5;
    const int n_sink_h = min((min(S, band_lo) + 31) >> 5, hb_lo);
    const int n_halves = n_sink_h + (hb_hi - hb_lo + 1);
    const int J = (n_halves + 1) >> 1;  // tiles
    auto half_of = [&](int i) { return i < n_sink_h ? i : i - n_sink_h + hb_lo; };
    const int wbound = window_bound(p0, 32, p.W, P);

    // ---- HBM -> LDS: waves 0, 1 copy a tile's first half, waves 2, 3 its second; an instruction moves
    // 8 rows of 128 bytes.  Rows past the sequence's last one (and the padding half) repeat it. ----
    const char *kg = reinterpret_cast<const char *>(p.k + sg.k_batch * p.k_sb + (long long)wi.kvh * p.k_sh + sg.k_row0 * p.k_sn);
    const char *vg = reinterpret_cast<const char *>(p.v + sg.k_batch * p.v_sb + (long long)wi.kvh * p.v_sh + sg.k_row0 * p.v_sn);
    const uint32_t k_rsb = (uint32_t)(p.k_sn * 2), v_rsb = (uint32_t)(p.v_sn * 2);  // row strides in bytes
    const int crow = 16 * (wave & 1) + (lane >> 3);  // row of the half that instruction 0 moves in this lane; 1: + 8
    uint32_t cchk[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = crow + 8 * i;
        cchk[i] = (uint32_t)((lane & 7) ^ ((((r >> 1) & 1) << 2) | ((r >> 2) & 3))) << 4;
    }
    auto issue_tile = [&](int j) {
        const int g = min(half_of(2 * j + (wave >> 1)), hb_hi);
        const uint32_t lds = (uint32_t)((j & 1) * kTileB + (wave >> 1) * kHalfB + (wave & 1) * (kHalfB / 2));
        const char *kb = kg + (size_t)(32 * g) * k_rsb, *vb = vg + (size_t)(32 * g) * v_rsb;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t row = (uint32_t)min(crow + 8 * i, Nk - 1 - 32 * g);
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(row * k_rsb + cchk[i]), "s"(kb),
                         "s"(lds + (uint32_t)(1024 * i))
                         : "memory");
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(row * v_rsb + cchk[i]), "s"(vb),
                         "s"(lds + (uint32_t)(2 * kHalfB + 1024 * i))
                         : "memory");
        }
    };
    issue_tile(0);

    // per-lane fragment addresses inside a half (swizzle folded in)
    //  * K fragment, k-step ks: row l32, logical chunk 2 ks + hf:  k_lane ^ (ks << 5)
    //  * V^T fragment, 16-key step st, head-dimension block db: rows 16 st + 4 hf + j16 / 4 (lo) and 8
    //    further (hi), logical chunk 4 db + 2 (grp & 1) + (j16 & 3) / 2:  v_lane ^ (db << 6), + rows
    const uint32_t k_lane = (uint32_t)(l32 * kRowB + ((hf ^ ((((l32 >> 1) & 1) << 2) | ((l32 >> 2) & 3))) << 4));
    const int grp = lane >> 4, j16 = lane & 15;
    const int rr = 4 * hf + (j16 >> 2);
    const int cl = 2 * (grp & 1) + ((j16 & 3) >> 1);
    const uint32_t v_lo = (uint32_t)(rr * kRowB + ((((j16 >> 3) << 2) | (cl ^ hf)) << 4) + 8 * (j16 & 1));
    const uint32_t v_hi = (uint32_t)((rr + 8) * kRowB + ((((j16 >> 3) << 2) | (cl ^ (hf + 2))) << 4) + 8 * (j16 & 1));

    f32x16 oacc[kDb];
#pragma unroll
    for (int db = 0; db < kDb; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[db][e] = 0.f;
    // Row state: the reference (0 while the row has seen no key), the score that moves it (in units of
    // the products: score * c2 > limit), this lane's share of the row sum.
    float mc = 0.f, limit = -INFINITY, l = 0.f;
    // Column sums of the rounded P^T: a P^T fragment (lane l: eight keys of query column l % 32) read as the B
    // operand of a 16x16x32 product is column l % 16, k-group l / 16; against an A operand whose row 0
    // is ones on k-groups 0 and 2 and whose row 1 on 1 and 3, D[0][j] is the sum over the fragment's
    // keys of query column j and D[1][j] of column 16 + j: elements 0 and 1 of lanes 0..15.
    f32x4 lsum = {0.f, 0.f, 0.f, 0.f};
    bf16x8 sel;
    {
        const int m = lane & 15, kg2 = lane >> 4;
        const __bf16 on = round16<kF16>((m == 0 && (kg2 & 1) == 0) || (m == 1 && (kg2 & 1) == 1) ? 1.f : 0.f);
#pragma unroll
        for (int e = 0; e < 8; ++e) sel[e] = on;
    }
    const float c2 = p.scale_log2;

#pragma unroll
    for (int ks = 0; ks < kKs; ++ks) asm volatile("" : "+v"(qf[ks]));  // (waits for the loads here)

    for (int j = 0; j < J; ++j) {
        __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0): this wave's share of tile j has landed, and it has read tile j - 1
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();        // everybody's; and everybody is done with tile j - 1
        asm volatile("" ::: "memory");
        if (j + 1 < J) issue_tile(j + 1);

#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const int k0 = 32 * half_of(2 * j + hh), k_last = k0 + 31;
            const bool in_future = k0 > plast;
            const bool before_band = (plast < P) && (k_last < p0 - p.W + 1) && (k0 >= S);
            if (!wave_active || in_future || before_band) continue;  // (uniform)
            const uint32_t kt = (uint32_t)((j & 1) * kTileB + hh * kHalfB), vt = kt + 2 * kHalfB;

            // ---- S^T = K Q^T : [32 keys] x [32 queries] ----
            f32x16 s;
#pragma unroll
            for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
            for (int ks = 0; ks < kKs; ++ks) s = mfma32<kF16>(lds16(kt + (k_lane ^ (uint32_t)(ks << 5))), qf[ks], s);

            // ---- scores that must not be seen become -inf (edge halves only) ----
            if (!((k_last <= p0) && ((k0 > wbound) || (k_last < S)))) {
                const uint32_t bits = visible_keys(k0, qpos, W, S) >> (4 * hf);
#pragma unroll
                for (int e = 0; e < 16; ++e) s[e] = where_visible(bits, e, s[e]);
            }

            // ---- does a score exceed its row's reference by more than the slack? ----
            float mx = s[0];
#pragma unroll
            for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[e]);
            if (__any(mx * c2 > limit)) {
                mx = half_swap_max(mx);  // (both lanes of a row decide alike)
                const bool move = mx * c2 > limit;
                const float alpha = !move ? 1.f : limit == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mc - mx * c2);
                mc = move ? mx * c2 : mc;
                limit = move ? mc + kSlack : limit;
                l *= alpha;
#pragma unroll
                for (int db = 0; db < kDb; ++db)
#pragma unroll
                    for (int e = 0; e < 16; ++e) oacc[db][e] *= alpha;
                lsum[0] *= __shfl(alpha, lane & 15);
                lsum[1] *= __shfl(alpha, 16 + (lane & 15));
            }

            // ---- P^T = exp2(s c2 - mc), rounded, in B-operand order ----
            bf16x8 pf[2];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float pe = __builtin_amdgcn_exp2f(fmaf(s[e], c2, -mc));
                l += pe;
                pf[e / 8][e % 8] = round16<kF16>(pe);
            }

            // ---- O^T += V^T P^T, and the sums of the rounded P ----
#pragma unroll
            for (int st = 0; st < 2; ++st) {
#pragma unroll
                for (int db = 0; db < kDb; ++db) {
                    const uint32_t off = vt + (uint32_t)(16 * st * kRowB);
                    const s16x4 lo = lds8_tr(off + (v_lo ^ (uint32_t)(db << 6)));
                    const s16x4 hi = lds8_tr(off + (v_hi ^ (uint32_t)(db << 6)));
                    const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                    oacc[db] = mfma32<kF16>(a, pf[st], oacc[db]);
                }
                lsum = mfma16<kF16>(sel, pf[st], lsum);
            }
        }
    }

    // ---- epilogue: O / (sum of the rounded P) -> 16 bit; lse = (mc + log2 l) ln 2 ----
    // (Query columns j and 16 + j share a column of lsum's products, kept apart by zeros, and 0 NaN is NaN: where one
    // of the two rows sees a key that is not a number, the other divides by its own fp32 sum of the unrounded P.)
    l = half_swap_sum(l);
    const float lb_lo = __shfl(lsum[0], l32 & 15), lb_hi = __shfl(lsum[1], l32 & 15);
    const float lb = l32 < 16 ? lb_lo : lb_hi;
    const float inv = 1.f / (non_finite(lb) ? l : lb);
    const int row = r0 + l32;
    if (row >= Nq) return;
    __bf16 *orow = p.out + sg.q_batch * p.o_sb + (long long)head * p.o_sh + (sg.q_row0 + row) * p.o_sn;
#pragma unroll
    for (int db = 0; db < kDb; ++db)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            bf16x4 o4;
#pragma unroll
            for (int e = 0; e < 4; ++e) o4[e] = round16<kF16>(oacc[db][4 * e4 + e] * inv);
            *reinterpret_cast<bf16x4 *>(orow + 32 * db + 8 * e4 + 4 * hf) = o4;
        }
    if (hf == 0)
        p.lse[sg.q_batch * p.lse_sb + (long long)head * p.lse_sh + sg.q_row0 + row] =
            (mc + __builtin_amdgcn_logf(l)) * 0.69314718055994530942f;
}

// ---- short prompts ----
// The kernel above walks a head's 32 rows, or 32 rows of four heads, along their keys in one wave: 765 tokens on 8 heads are 48
// workgroups, and the longest walks 24 halves one behind the other: the chain is the bound.  As at 128 (swaa_fwd_short.hip), a
// workgroup here is 32 rows of ONE head and its four waves take a quarter of the keys each, with a ring of one half of their
// own, no barriers in the loop and a max-based softmax; their results meet in LDS.  (Relative error of O against 64 bits over 12
// calls: 0.00196 where the kernel above has 0.00205, each wave's reference being its own keys' largest score.)
constexpr int kS64Waves = 4, kS64Threads = 64 * kS64Waves, kS64Rows = 32;
constexpr uint32_t kS64Ring = 2 * kHalfB;             // a wave's: K half, then V half; its O at the end
constexpr uint32_t kS64Ml = kS64Waves * kS64Ring;     // [wave][32] of reference, l, l / sum of the rounded P, 0
constexpr int kS64Bytes = kS64Waves * ((int)kS64Ring + 512);
static_assert(kS64Rows * kD64 * 4 == kS64Ring && kS64Bytes <= 64 * 1024, "");

template <bool kF16>
__global__ __launch_bounds__(kS64Threads, 4) void swaa_fwd_d64_short_kernel(const FwdShortParams sp) {
    fetch_args<FwdShortParams>();
    const FwdParams &p = sp.f;
    constexpr int kBelow = kF16 ? 4 : 0;  // terms keep full precision down to 2^-18 of the reference
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int l32 = lane & 31, hf = lane >> 5;
    // Long rows first; the (batch, KV head) pair innermost.
    const unsigned by_pair = fastdiv(blockIdx.x, sp.div_pairs), pair = blockIdx.x - by_pair * (unsigned)sp.pairs;
    const unsigned by_group = fastdiv(by_pair, sp.div_group), g = by_pair - by_group * (unsigned)p.G;
    const int b = (int)fastdiv(pair, p.div_hkv), kvh = (int)pair - b * p.Hkv;
    const int head = kvh * p.G + (int)g;
    const int r0 = kS64Rows * (sp.tiles - 1 - (int)by_group);  // first query row
    const int N = p.Nq, S = p.S;  // (whole prompts: as many keys)
    const int n_prompt = p.n_prompts ? max(p.n_prompts[b], 0) : p.P;
    const int p1 = min(r0 + kS64Rows, N) - 1;  // last row
    const int row = min(r0 + l32, N - 1);      // this lane's column
    const int W = row >= n_prompt ? N : p.W;

    // ---- the schedule, in halves of 32 keys: sinks, then the band; a quarter of them is this wave's ----
    const int band_lo = p1 >= n_prompt ? 0 : max(0, r0 - p.W + 1);
    const int hb_lo = band_lo >> 5, hb_hi = p1 >> 5;
    const int n_sink = min((min(S, band_lo) + 31) >> 5, hb_lo);
    const int n_all = n_sink + (hb_hi - hb_lo + 1);
    const int quarter = (n_all + kS64Waves - 1) / kS64Waves;
    const int h_mine = wave * quarter;
    const int n_mine = max(0, min(quarter, n_all - h_mine));
    auto first_key = [&](int t) __attribute__((always_inline)) {
        const int h = h_mine + t;
        return 32 * (h < n_sink ? h : h - n_sink + hb_lo);
    };

    // ---- HBM -> LDS copies of one half: instruction i moves rows 8 i .. 8 i + 7.  Rows past the end repeat the last one. ----
    const uint32_t k_rsb = (uint32_t)(p.k_sn * 2), v_rsb = (uint32_t)(p.v_sn * 2);
    const char *kg = reinterpret_cast<const char *>(p.k + b * p.k_sb + kvh * p.k_sh);
    const char *vg = reinterpret_cast<const char *>(p.v + b * p.v_sb + kvh * p.v_sh);
    const uint32_t ring = (uint32_t)wave * kS64Ring;
    const int lr = lane >> 3;
    uint32_t cchk[2];  // (the swizzle f(r) of row 8 i + lr depends on i & 1)
#pragma unroll
    for (int i = 0; i < 2; ++i) cchk[i] = (uint32_t)((lane & 7) ^ ((((lr >> 1) & 1) << 2) | ((2 * i + (lr >> 2)) & 3))) << 4;
    auto issue = [&](const char *g0, uint32_t rsb, uint32_t lds, int k0) __attribute__((always_inline)) {
        const char *base = g0 + (size_t)k0 * rsb;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t off = (uint32_t)min(8 * i + lr, N - 1 - k0) * rsb + cchk[i & 1];
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds + (uint32_t)(1024 * i))
                         : "memory");
        }
    };
    if (n_mine > 0) {
        issue(kg, k_rsb, ring, first_key(0));
        issue(vg, v_rsb, ring + kHalfB, first_key(0));
    }
    bf16x8 qf[kKs];
    {
        const __bf16 *qrow = p.q + b * p.q_sb + (long long)head * p.q_sh + (long long)row * p.q_sn + 8 * hf;
#pragma unroll
        for (int ks = 0; ks < kKs; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(qrow + 16 * ks);
    }

    // per-lane fragment addresses in this wave's ring (as above)
    const uint32_t k_lane = ring + (uint32_t)(l32 * kRowB + ((hf ^ ((((l32 >> 1) & 1) << 2) | ((l32 >> 2) & 3))) << 4));
    const int grp = lane >> 4, j16 = lane & 15;
    const int rr = 4 * hf + (j16 >> 2);
    const int cl = 2 * (grp & 1) + ((j16 & 3) >> 1);
    const uint32_t v_lo = (uint32_t)(rr * kRowB + ((((j16 >> 3) << 2) | (cl ^ hf)) << 4) + 8 * (j16 & 1));
    const uint32_t v_hi = (uint32_t)((rr + 8) * kRowB + ((((j16 >> 3) << 2) | (cl ^ (hf + 2))) << 4) + 8 * (j16 & 1));

    f32x16 oacc[kDb];
#pragma unroll
    for (int db = 0; db < kDb; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[db][e] = 0.f;
    RowState rs;
    rs.mc = -INFINITY;
    rs.l = 0.f;
    rs.lb = 0.f;
    const float c2 = p.scale_log2;
    const int wbound = window_bound(r0, kS64Rows, p.W, n_prompt);
#pragma unroll
    for (int ks = 0; ks < kKs; ++ks) asm volatile("" : "+v"(qf[ks]));  // (waits for the loads here)

    for (int t = 0; t < n_mine; ++t) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // half t has landed
        const int k0 = first_key(t);
        // all fragments to registers, then the next half's copy into the same ring, then the arithmetic
        bf16x8 kf[kKs], vf[2][kDb];
#pragma unroll
        for (int ks = 0; ks < kKs; ++ks) kf[ks] = lds16(k_lane ^ (uint32_t)(ks << 5));
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int db = 0; db < kDb; ++db) {
                const uint32_t off = ring + (uint32_t)(kHalfB + 16 * st * kRowB);
                const s16x4 lo = lds8_tr(off + (v_lo ^ (uint32_t)(db << 6)));
                const s16x4 hi = lds8_tr(off + (v_hi ^ (uint32_t)(db << 6)));
                vf[st][db] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (t + 1 < n_mine) {
            issue(kg, k_rsb, ring, first_key(t + 1));
            issue(vg, v_rsb, ring + kHalfB, first_key(t + 1));
        }
        f32x16 s;
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
        for (int ks = 0; ks < kKs; ++ks) s = mfma32<kF16>(kf[ks], qf[ks], s);
        bf16x8 pf[2];
        float alpha;
        if (!((k0 + 31 <= r0) && ((k0 > wbound) || (k0 + 31 < S))))
            softmax_half<true, kF16, kBelow>(s, k0, row, W, S, hf, c2, rs, pf, alpha);
        else
            softmax_half<false, kF16, kBelow>(s, k0, row, W, S, hf, c2, rs, pf, alpha);
        if (__any(alpha != 1.f)) {
#pragma unroll
            for (int db = 0; db < kDb; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) oacc[db][e] *= alpha;
        }
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int db = 0; db < kDb; ++db) oacc[db] = mfma32<kF16>(vf[st][db], pf[st], oacc[db]);
    }

    // ---- the four waves' results through LDS: rows of 256 bytes, 16-byte chunk q of row c at q ^ (c & 15); 16 threads take a row.
    // A wave's O is the sum over the rounded P: it enters scaled by l / (sum of the rounded P). ----
    {
        float l_row, lb_row;
        row_sums(rs, l_row, lb_row);
        const f32x4_t weight = {rs.mc, l_row, lb_row > 0.f ? l_row / lb_row : 0.f, 0.f};  // a row that saw no key: O = 0, l = 0
        if (hf == 0) *(LdsQuads)(uintptr_t)(kS64Ml + (uint32_t)(wave * 512 + l32 * 16)) = weight;
        const uint32_t at = ring + (uint32_t)(l32 * 256 + ((hf ^ (l32 & 15)) << 4));
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            f32x4_t o4;
#pragma unroll
            for (int e = 0; e < 4; ++e) o4[e] = oacc[c / 4][4 * (c % 4) + e];
            *(LdsQuads)(uintptr_t)(at ^ (uint32_t)(c << 5)) = o4;  // head-dimension elements 8 c + 4 hf ..
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int c = 16 * i + (int)(threadIdx.x >> 4), q = (int)(threadIdx.x & 15);
        if (r0 + c >= N) break;
        f32x4_t w[kS64Waves], ox[kS64Waves];
#pragma unroll
        for (int x = 0; x < kS64Waves; ++x) {
            w[x] = *(LdsQuads)(uintptr_t)(kS64Ml + (uint32_t)(x * 512 + c * 16));
            ox[x] = *(LdsQuads)(uintptr_t)((uint32_t)x * kS64Ring + (uint32_t)(c * 256 + ((q ^ (c & 15)) << 4)));
        }
        const float m = fmaxf(fmaxf(w[0][0], w[1][0]), fmaxf(w[2][0], w[3][0])), m_use = m == -INFINITY ? 0.f : m;
        float l = 0.f;
        f32x4_t o4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int x = 0; x < kS64Waves; ++x) {
            const float e2 = __builtin_amdgcn_exp2f(w[x][0] - m_use), wo = e2 * w[x][2];
            l += e2 * w[x][1];
#pragma unroll
            for (int e = 0; e < 4; ++e) o4[e] += ox[x][e] * wo;
        }
        o4 *= 1.f / l;
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = round16<kF16>(o4[e]);
        *reinterpret_cast<bf16x4 *>(p.out + b * p.o_sb + (long long)head * p.o_sh + (long long)(r0 + c) * p.o_sn + 4 * q) = o;
        if (q == 0) p.lse[b * p.lse_sb + (long long)head * p.lse_sh + r0 + c] = (m + __builtin_amdgcn_logf(l)) * 0.69314718055994530942f;
    }
}

// Which of the two?  Four heads in a workgroup's waves, or one head in four parts of its keys (us, bfloat16; full attention
// unless a window is stated):
//    units (of 32 rows)      256           512           1024          1536          2048
//    8 heads on 8        18.6 / 8.4    33.8 / 13.7   63.6 / 31.7   94.1 / 61.2   125 / 105
//      window 1024                     22.1 / 10.8   22.3 / 18.4   29.1 / 25.8   30.0 / 33.3
//    16 heads on 4       11.3 / 5.9    19.1 / 8.8    34.2 / 18.8   49.9 / 34.0   65.3 / 55.6
//      window 1024                                   20.8 / 16.1   28.3 / 23.3   29.0 / 30.3
//    40 heads on 8       6.9 / 4.9     10.0 / 6.7    16.4 / 11.9   29.1 / 18.6   35.8 / 28.1
//    window 128, 32 heads on 8, 1000 tokens, 1024 units: 7.7 / 8.1     32 tokens, 8 on 8: 3.7 / 3.9 (one half: nothing to share out)
// Beyond 1536 units where the longest row's chain is 2.7 times what a resident workgroup gets on average (2048 units above,
// full attention: 4.0; window 1024: 2.1 to 2.9).
bool plan_fwd_d64_short(const FwdParams &p, FwdShortParams &sp) {
    const long long units = (long long)p.B * p.Hq * ((p.Nq + kS64Rows - 1) / kS64Rows);
    if (p.cu_q || p.Nq != p.Nk || p.Nk <= 32 || units > 0x7fffffffLL) return false;
    if (units > 512 && (units > 1536 || longest_row(p) < 256)) {
        if (p.n_prompts) return false;  // (what its rows see is known on the device only)
        if (longest_row(p) < 48 * 32 || !chain_is_the_time(p, 1024, 128, 2.7, 1.7)) return false;
    }
    fill_fwd_short(p, sp);
    return true;
}

}  // namespace

hipError_t launch_fwd_d64(const FwdParams &p, hipStream_t stream) {
    if (p.wg_rows != kFwdWgRows) return hipErrorInvalidValue;  // the plan must be the one for this kernel's workgroups
    FwdShortParams sp;
    if (plan_fwd_d64_short(p, sp)) {
        const dim3 units((unsigned)(sp.pairs * p.G * sp.tiles));
        if (p.fp16)
            hipLaunchKernelGGL(swaa_fwd_d64_short_kernel<true>, units, dim3(kS64Threads), kS64Bytes, stream, sp);
        else
            hipLaunchKernelGGL(swaa_fwd_d64_short_kernel<false>, units, dim3(kS64Threads), kS64Bytes, stream, sp);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)(p.chunk * kXcds));
    if (p.fp16)
        hipLaunchKernelGGL(swaa_fwd_d64_kernel<true>, grid, dim3(kThreads), kSmem64, stream, p);
    else
        hipLaunchKernelGGL(swaa_fwd_d64_kernel<false>, grid, dim3(kThreads), kSmem64, stream, p);
    return hipGetLastError();
}

}  // namespace swaa
