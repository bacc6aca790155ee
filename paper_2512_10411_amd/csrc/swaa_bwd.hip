// Backward pass of the SWA + sink (+ FA Decode rows) attention, gfx950: the
// gradients that SWA-aware fine-tuning (paper Sec. 3.2.2) needs, under the same
// mask as the forward kernels (Sec. 3.2.1 / Fig. 1b, Sec. 3.1.1 / Fig. 1a).
//
// With P_ij = exp(s_ij - lse_i) on the visible pairs and 0 elsewhere:
//
//   delta_i = <dO_i, O_i>                      (= sum_j P_ij dP_ij)
//   dV_j = sum_i P_ij dO_i                     dP_ij = <dO_i, v_j>
//   dS_ij = P_ij (dP_ij - delta_i)
//   dQ_i = scale sum_j dS_ij k_j               dK_j = scale sum_i dS_ij q_i
//
// Three kernels, no atomics, results independent of scheduling:
//   * swaa_bwd_dq_kernel: a workgroup owns 256 query rows (the forward's work
//     decomposition and tile schedule), walks its visible KV tiles, recomputes
//     S^T = K Q^T and dP^T = V dO^T and accumulates dQ^T += K^T dS^T.  It forms delta on the way.
//   * swaa_bwd_dkv_kernel: a workgroup owns 128 keys of one KV head, walks
//     every query head of the GQA group and every 64-row query tile (32-row
//     block) that can see them, recomputes S = Q K^T and dP = dO V^T and accumulates
//     dV^T += dO^T P and dK^T += Q^T dS.  Key tiles that hold sink
//     keys are seen by every later row: their rows beyond the band are cut into
//     segments with a workgroup each, and
//   * swaa_bwd_part_sum_kernel adds the fp32 partial sums of those key tiles.  Where the key tiles are too few for the chip,
//     their steps are cut into pieces with a workgroup each, and all key tiles have partial sums (plan_pieces).
// Each product is a v_mfma_f32_32x32x16_bf16 with the accumulator oriented so
// that the probabilities come out in the B-operand layout of the product that
// consumes them (as in the forward kernels); operands that a product needs
// transposed are read from row-major LDS tiles with ds_read_b64_tr_b16.
// P and dS are rounded to bf16 before the second products, sums are fp32.
// dQ for head dimension 64, in this file, leaves instruction scheduling to the compiler,
// as does dK/dV for head dimension 128 where a key tile is seen by few query tiles (swaa_bwd_dkv_d128_short.h);
// otherwise dQ (swaa_bwd_dq_pipelined.hip) and dK/dV (swaa_bwd_dkv_d128.h) of head dimension 128 and dK/dV of 64
// (swaa_bwd_dkv_d64.h) are pipelined by hand.  Waves per SIMD: two (dQ, short dK/dV) or one (dK/dV) for head
// dimension 128, four (dQ) and two (dK/dV) for 64.
#include <atomic>
#include <cmath>

#include "swaa_bwd.h"

#include <type_traits>

namespace swaa {
namespace {

constexpr int kBq = 64;  // query rows per tile of the dK/dV kernel

__device__ __forceinline__ bf16x8 lds16(uint32_t addr) {
    return *(const bf16x8 __attribute__((address_space(3))) *)(uintptr_t)addr;
}
__device__ __forceinline__ s16x4 lds8_tr(uint32_t addr) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)(uintptr_t)addr);
}

// ---- dQ, head dimension 64 -------------------------------------------------------------
// A workgroup is eight waves of 32 query rows; 128 registers per wave, so that two workgroups share
// a compute unit and one wave's exponentials run under the others' matrix instructions.  (With a
// whole 64-key tile's scores in registers a wave took 208, a compute unit one workgroup, and every
// element of every tile its own mask branches: 95 us for two sequences of 4001 tokens, 16 heads on
// 4, window 1000; in halves 62.)  A tile is two halves of 32 keys, worked through one after the other;
// a wave skips the halves that its rows do not see and masks those on an edge.
// Tiles are copied from memory to LDS without a stop in registers, one ahead, into two buffers with one barrier per tile.  (Through
// registers into one buffer of padded rows, two barriers per tile, the backward of 2048 tokens, 32 heads on 8, full attention
// took 117.8 us, now 109.9; two of 4001 on a window of 1000, 16 heads on 4, 161.0 and 157.8; 16384 on 128 251 and 253.  Three
// buffers, two tiles ahead: 0.3 % slower.  The halves in a loop, operands four at a time: 1.2 % slower.)
namespace dq64 {
constexpr int kD = 64, kKS = kD / 16, kDB = kD / 32;
constexpr int kThreads = 512;
constexpr int kRowB = kD * 2, kHalfB = 32 * kRowB, kTileB = 4 * kHalfB;  // K half 0, K half 1, V half 0, V half 1
constexpr int kBytes = 2 * kTileB;
}  // namespace dq64

__global__ __launch_bounds__(dq64::kThreads, 4) void swaa_bwd_dq_kernel(const BwdParams p) {
    using namespace dq64;
    WorkItem wi;
    if (!decode_work(p.f, wi)) return;
    const int hpb = wi.hpb;
    const int rows_per_wg = kWgRows >> (hpb >> 1);  // (hpb is 1, 2 or 4: shifts, no divisions)
    const int N = p.N, W = p.f.W, S = p.f.S, P = p.f.P;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;

    const int head = wi.kvh * p.f.G + wi.h0 + (wave & (hpb - 1));
    const int wg_p0 = wi.pt * rows_per_wg;
    const int wg_p1 = min(N, wg_p0 + rows_per_wg) - 1;
    const int p0 = wg_p0 + (wave >> (hpb >> 1)) * 32;
    const bool wave_active = p0 < N;
    const int plast = min(p0 + 32, N) - 1;
    const int qpos = p0 + l32;

    // the schedule (as in the forward): sink halves, then the band's; an odd count is padded with a half past the last
    // row, which no row can see
    const int band_lo = (wg_p1 >= P) ? 0 : max(0, wg_p0 - W + 1);
    const int hb_lo = band_lo >> 5, hb_hi = wg_p1 >> 5;
    const int n_sink_h = min((min(S, band_lo) + 31) >> 5, hb_lo);
    const int J = (n_sink_h + (hb_hi - hb_lo + 1) + 1) >> 1;  // tiles
    auto half_of = [&](int i) { return i < n_sink_h ? i : i - n_sink_h + hb_lo; };
    const int wbound = window_bound(p0, 32, W, P);

    // ---- HBM -> LDS: waves 0..3 copy a tile's K, 4..7 its V; the first two of the four its first half, an instruction
    // 8 rows of 128 bytes.  The swizzle of the reads is applied on the global side.  Rows past the sequence's last one
    // (and the padding half) repeat it. ----
    const size_t kv_base = ((size_t)wi.b * p.Hkv + wi.kvh) * (size_t)N * kD;
    const char *src = reinterpret_cast<const char *>((wave < 4 ? p.f.k : p.f.v) + kv_base);
    const int crow = 16 * (wave & 1) + (lane >> 3);  // row of the half that instruction 0 moves in this lane; 1: + 8
    uint32_t cchk[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = crow + 8 * i;
        cchk[i] = (uint32_t)((lane & 7) ^ ((((r >> 1) & 1) << 2) | ((r >> 2) & 3))) << 4;
    }
    const uint32_t lds_copy = (uint32_t)((wave >> 1) * kHalfB + (wave & 1) * (kHalfB / 2));
    auto issue_tile = [&](int j) {
        const int g = min(half_of(2 * j + ((wave >> 1) & 1)), hb_hi);
        const uint32_t lds = lds_copy + (uint32_t)((j & 1) * kTileB);
        const char *base = src + (size_t)(32 * g) * kRowB;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t row = (uint32_t)min(crow + 8 * i, N - 1 - 32 * g);
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(row * kRowB + cchk[i]), "s"(base),
                         "s"(lds + (uint32_t)(1024 * i))
                         : "memory");
        }
    };

    const size_t q_base = ((size_t)wi.b * p.Hq + head) * (size_t)N * kD;
    const size_t r_base = ((size_t)wi.b * p.Hq + head) * (size_t)N;
    // this wave's Q and dO rows as B operands, its rows' lse (log2 units) and delta
    bf16x8 qf[kKS], dof[kKS];
    float lse2, dl;
    {
        const int row = min(qpos, N - 1);
        const __bf16 *qs = p.f.q + q_base + (size_t)row * kD + 8 * hf;
        const __bf16 *ds = p.dout + q_base + (size_t)row * kD + 8 * hf;
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) {
            qf[ks] = *reinterpret_cast<const bf16x8 *>(qs + 16 * ks);
            dof[ks] = *reinterpret_cast<const bf16x8 *>(ds + 16 * ks);
        }
        lse2 = p.f.lse[r_base + row];
        issue_tile(0);  // (behind the loads that the first waits are for)
        dl = row_delta<kKS>(p.out + q_base + (size_t)row * kD + 8 * hf, dof);
        lse2 *= 1.44269504088896340736f;
        if (qpos < N && hf == 0) p.delta[r_base + row] = dl;  // for the dK/dV kernel
    }

    // per-lane fragment addresses inside a half (swizzle folded in)
    //  * row fragment, k-step ks: row l32, logical chunk 2 ks + hf:  row_lane ^ (ks << 5)
    //  * transposed fragment, 16-key step st, head-dimension block db: rows 16 st + 4 hf + j16 / 4 (lo) and 8
    //    further (hi), logical chunk 4 db + 2 (grp & 1) + (j16 & 3) / 2:  col_lane ^ (db << 6), + rows
    const uint32_t row_lane = (uint32_t)(l32 * kRowB + ((hf ^ ((((l32 >> 1) & 1) << 2) | ((l32 >> 2) & 3))) << 4));
    const int grp = lane >> 4, j16 = lane & 15;
    const int rr = 4 * hf + (j16 >> 2);
    const int cl = 2 * (grp & 1) + ((j16 & 3) >> 1);
    const uint32_t col_lo = (uint32_t)(rr * kRowB + ((((j16 >> 3) << 2) | (cl ^ hf)) << 4) + 8 * (j16 & 1));
    const uint32_t col_hi = (uint32_t)((rr + 8) * kRowB + ((((j16 >> 3) << 2) | (cl ^ (hf + 2))) << 4) + 8 * (j16 & 1));

    f32x16 dqacc[kDB];
#pragma unroll
    for (int db = 0; db < kDB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) dqacc[db][e] = 0.f;
    const float c2 = p.f.scale_log2;

#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) asm volatile("" : "+v"(qf[ks]), "+v"(dof[ks]));  // (waits for the loads here)
    asm volatile("" : "+v"(lse2), "+v"(dl));

    for (int j = 0; j < J; ++j) {
        __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0): this wave's share of tile j has landed, and it has read tile j - 1
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();        // everybody's; and everybody is done with tile j - 1
        asm volatile("" ::: "memory");
        if (j + 1 < J) issue_tile(j + 1);

#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const int k0 = 32 * half_of(2 * j + kb), k_last = k0 + 31;
            const bool in_future = k0 > plast;
            const bool before_band = (plast < P) && (k_last < p0 - W + 1) && (k0 >= S);
            if (!wave_active || in_future || before_band) continue;  // (uniform)
            const bool unmasked = (k_last <= p0) && ((k0 > wbound) || (k_last < S));
            const uint32_t kt = (uint32_t)((j & 1) * kTileB + kb * kHalfB), vt = kt + 2 * kHalfB;

            // S^T = K Q^T and dP^T = V dO^T : [32 keys] x [32 queries]
            f32x16 sacc, dpacc;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                sacc[e] = 0.f;
                dpacc[e] = 0.f;
            }
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks) {
                sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds16(kt + (row_lane ^ (uint32_t)(ks << 5))), qf[ks], sacc, 0, 0, 0);
                dpacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds16(vt + (row_lane ^ (uint32_t)(ks << 5))), dof[ks], dpacc, 0, 0, 0);
            }

            // dS^T = P^T (dP^T - delta) with P^T = exp2(s c2 - lse2), packed to bf16; a score that must not
            // be seen becomes -inf, its P an exact 0
            if (!unmasked) {
                const uint32_t bits = qpos < N ? visible_keys(k0, qpos, qpos >= P ? N : W, S) >> (4 * hf) : 0u;
#pragma unroll
                for (int e = 0; e < 16; ++e) sacc[e] = where_visible(bits, e, sacc[e]);
            }
            bf16x8 dsf[2];  // [16-key step]
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float pe = __builtin_amdgcn_exp2f(fmaf(sacc[e], c2, -lse2));
                dsf[e / 8][e % 8] = (__bf16)(pe * (dpacc[e] - dl));
            }

            // dQ^T += K^T dS^T
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
                for (int db = 0; db < kDB; ++db) {
                    const uint32_t off = kt + (uint32_t)(16 * st * kRowB);
                    const s16x4 lo = lds8_tr(off + (col_lo ^ (uint32_t)(db << 6)));
                    const s16x4 hi = lds8_tr(off + (col_hi ^ (uint32_t)(db << 6)));
                    const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                    dqacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, dsf[st], dqacc[db], 0, 0, 0);
                }
        }
    }

    if (qpos >= N) return;
    __bf16 *orow = p.dq + q_base + (size_t)qpos * kD;
#pragma unroll
    for (int db = 0; db < kDB; ++db)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            bf16x4 o4;
#pragma unroll
            for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(dqacc[db][4 * e4 + e] * p.f.scale);
            *reinterpret_cast<bf16x4 *>(orow + 32 * db + 8 * e4 + 4 * hf) = o4;
        }
}

// Short sequences: 32 rows of ONE head per workgroup, whose four waves take a quarter of the keys each with a ring of one half
// of their own and no barriers in the loop (as swaa_bwd_dq_short_kernel of head dimension 128); their sums meet in LDS.
namespace dq64s {
constexpr int kWaves = 4, kThreads = 64 * kWaves, kRows = 32;
constexpr uint32_t kRing = 2 * dq64::kHalfB;  // a wave's: K half, then V half; its dQ at the end
constexpr int kBytes = kWaves * (int)kRing;
static_assert(kRows * dq64::kD * 4 == kRing, "");
}  // namespace dq64s

__global__ __launch_bounds__(dq64s::kThreads, 3) void swaa_bwd_dq64_short_kernel(const BwdParams p) {
    using dq64::kD, dq64::kKS, dq64::kDB, dq64::kRowB, dq64::kHalfB;
    using dq64s::kWaves, dq64s::kRows, dq64s::kRing;
    const int N = p.N, S = p.f.S, P = p.f.P;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l32 = lane & 31, hf = lane >> 5;
    // Long rows first; the (batch, KV head) pair innermost.
    const unsigned by_pair = fastdiv(blockIdx.x, p.div_pairs), pair = blockIdx.x - by_pair * (unsigned)(p.B * p.Hkv);
    const unsigned by_group = fastdiv(by_pair, p.div_group), g = by_pair - by_group * (unsigned)p.f.G;
    const int b = (int)fastdiv(pair, p.div_hkv), kvh = (int)pair - b * p.Hkv;
    const int head = kvh * p.f.G + (int)g;
    const int r0 = kRows * ((N + kRows - 1) / kRows - 1 - (int)by_group);  // first query row
    const int p1 = min(r0 + kRows, N) - 1;  // last row
    const int row = min(r0 + l32, N - 1);   // this lane's column
    const int W = row >= P ? N : p.f.W;

    // the schedule, in halves of 32 keys: sinks, then the band; a quarter of them is this wave's
    const int band_lo = p1 >= P ? 0 : max(0, r0 - p.f.W + 1);
    const int hb_lo = band_lo >> 5, hb_hi = p1 >> 5;
    const int n_sink = min((min(S, band_lo) + 31) >> 5, hb_lo);
    const int n_all = n_sink + (hb_hi - hb_lo + 1);
    const int quarter = (n_all + kWaves - 1) / kWaves;
    const int h_mine = wave * quarter;
    const int n_mine = max(0, min(quarter, n_all - h_mine));
    auto first_key = [&](int t) __attribute__((always_inline)) {
        const int h = h_mine + t;
        return 32 * (h < n_sink ? h : h - n_sink + hb_lo);
    };

    // HBM -> LDS copies of one half: instruction i moves rows 8 i .. 8 i + 7.  Rows past the end repeat the last one.
    const size_t kv_base = ((size_t)b * p.Hkv + kvh) * (size_t)N * kD;
    const char *kg = reinterpret_cast<const char *>(p.f.k + kv_base), *vg = reinterpret_cast<const char *>(p.f.v + kv_base);
    const size_t q_base = ((size_t)b * p.Hq + head) * (size_t)N * kD, r_base = ((size_t)b * p.Hq + head) * (size_t)N;
    const uint32_t ring = (uint32_t)wave * kRing;
    const int lr = lane >> 3;
    uint32_t cchk[2];  // (the swizzle of row 8 i + lr depends on i & 1)
#pragma unroll
    for (int i = 0; i < 2; ++i) cchk[i] = (uint32_t)((lane & 7) ^ ((((lr >> 1) & 1) << 2) | ((2 * i + (lr >> 2)) & 3))) << 4;
    auto issue = [&](const char *g0, uint32_t lds, int k0) __attribute__((always_inline)) {
        const char *base = g0 + (size_t)k0 * kRowB;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t off = (uint32_t)min(8 * i + lr, N - 1 - k0) * kRowB + cchk[i & 1];
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds + (uint32_t)(1024 * i))
                         : "memory");
        }
    };
    if (n_mine > 0) {
        issue(kg, ring, first_key(0));
        issue(vg, ring + kHalfB, first_key(0));
    }
    // this wave's Q and dO rows as B operands, its rows' lse (log2 units) and delta
    bf16x8 qf[kKS], dof[kKS];
    const __bf16 *qs = p.f.q + q_base + (size_t)row * kD + 8 * hf, *ds = p.dout + q_base + (size_t)row * kD + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) {
        qf[ks] = *reinterpret_cast<const bf16x8 *>(qs + 16 * ks);
        dof[ks] = *reinterpret_cast<const bf16x8 *>(ds + 16 * ks);
    }
    const float lse2 = p.f.lse[r_base + row] * 1.44269504088896340736f;
    const float dl = row_delta<kKS>(p.out + q_base + (size_t)row * kD + 8 * hf, dof);
    if (wave == 0 && r0 + l32 < N && hf == 0) p.delta[r_base + row] = dl;  // for the dK/dV kernel

    // per-lane fragment addresses in this wave's ring (as in swaa_bwd_dq_kernel)
    const uint32_t row_lane = ring + (uint32_t)(l32 * kRowB + ((hf ^ ((((l32 >> 1) & 1) << 2) | ((l32 >> 2) & 3))) << 4));
    const int grp = lane >> 4, j16 = lane & 15;
    const int rr = 4 * hf + (j16 >> 2);
    const int cl = 2 * (grp & 1) + ((j16 & 3) >> 1);
    const uint32_t col_lo = ring + (uint32_t)(rr * kRowB + ((((j16 >> 3) << 2) | (cl ^ hf)) << 4) + 8 * (j16 & 1));
    const uint32_t col_hi = ring + (uint32_t)((rr + 8) * kRowB + ((((j16 >> 3) << 2) | (cl ^ (hf + 2))) << 4) + 8 * (j16 & 1));

    f32x16 dqacc[kDB];
#pragma unroll
    for (int db = 0; db < kDB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) dqacc[db][e] = 0.f;
    const float c2 = p.f.scale_log2;
    const int wbound = window_bound(r0, kRows, p.f.W, P);

    for (int t = 0; t < n_mine; ++t) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // half t has landed
        const int k0 = first_key(t);
        // all fragments to registers, then the next half's copies into the same ring, then the arithmetic
        bf16x8 kf[kKS], vf[kKS], ct[2][kDB];
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) {
            kf[ks] = lds16(row_lane ^ (uint32_t)(ks << 5));
            vf[ks] = lds16((row_lane ^ (uint32_t)(ks << 5)) + kHalfB);
        }
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int db = 0; db < kDB; ++db) {
                const s16x4 lo = lds8_tr((col_lo ^ (uint32_t)(db << 6)) + (uint32_t)(16 * st * kRowB));
                const s16x4 hi = lds8_tr((col_hi ^ (uint32_t)(db << 6)) + (uint32_t)(16 * st * kRowB));
                ct[st][db] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (t + 1 < n_mine) {
            issue(kg, ring, first_key(t + 1));
            issue(vg, ring + kHalfB, first_key(t + 1));
        }
        f32x16 sacc, dpacc;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            sacc[e] = 0.f;
            dpacc[e] = 0.f;
        }
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) {
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], sacc, 0, 0, 0);
            dpacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[ks], dof[ks], dpacc, 0, 0, 0);
        }
        if (!((k0 + 31 <= r0) && ((k0 > wbound) || (k0 + 31 < S)))) {
            const uint32_t bits = visible_keys(k0, row, W, S) >> (4 * hf);
#pragma unroll
            for (int e = 0; e < 16; ++e) sacc[e] = where_visible(bits, e, sacc[e]);
        }
        bf16x8 dsf[2];  // [16-key step]
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float pe = __builtin_amdgcn_exp2f(fmaf(sacc[e], c2, -lse2));
            dsf[e / 8][e % 8] = (__bf16)(pe * (dpacc[e] - dl));
        }
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int db = 0; db < kDB; ++db) dqacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ct[st][db], dsf[st], dqacc[db], 0, 0, 0);
    }

    // the four waves' sums: rows of 256 bytes, 16-byte chunk q of row c at q ^ (c & 15); 16 threads take a row
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef f32x4 __attribute__((address_space(3))) *Quads;
    const uint32_t at = ring + (uint32_t)(l32 * 256 + ((hf ^ (l32 & 15)) << 4));
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        f32x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = dqacc[c / 4][4 * (c % 4) + e];
        *(Quads)(uintptr_t)(at ^ (uint32_t)(c << 5)) = o4;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int c = 16 * i + (int)(threadIdx.x >> 4), q = (int)(threadIdx.x & 15);
        if (r0 + c >= N) break;
        const uint32_t from = (uint32_t)(c * 256 + ((q ^ (c & 15)) << 4));
        f32x4 o4 = *(Quads)(uintptr_t)from;
#pragma unroll
        for (int x = 1; x < kWaves; ++x) o4 += *(Quads)(uintptr_t)(from + (uint32_t)x * kRing);
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (__bf16)(o4[e] * p.f.scale);
        *reinterpret_cast<bf16x4 *>(p.dq + q_base + (size_t)(r0 + c) * kD + 4 * q) = o;
    }
}

// Which of the two?  The whole training step, 256 rows together / a head's 32 rows (us; full attention unless a window is stated):
//    units (of 32 rows)     512           1024          1536          2048          3072
//    8 heads on 8       92.7 / 60.3    180 / 131     286 / 226     424 / 369     829 / 798
//      window 1024      69.5 / 48.4   86.8 / 77.9    110 / 109     136 / 140     194 / 194
//    16 heads on 4      61.8 / 44.4    104 / 83.4    161 / 135     241 / 213     444 / 432
//      window 1024                    83.5 / 75.5    107 / 108     122 / 127     187 / 184
//    40 heads on 8      41.7 / 35.9   64.6 / 58.0   99.5 / 91.8    125 / 120     236 / 211
//    window 128, 32 heads on 8, 1000 tokens, 1024 units: 47.5 / 47.8
//    512 generated rows: 8 on 8, 6336, window 1024: 235 / 145   19000: 736 / 434   16 on 4, 8704, window 4096: 717 / 675
// Beyond 1024 units where the longest row's chain is several times what one of the 512 resident workgroups gets on average
// (full attention, 3072 units, 2.7; window 1024, 2048 units, 2.1; the last line's 17, 17 and 2.4).
bool dq64_short(const BwdParams &p) {
    const long long units = (long long)p.B * p.Hq * ((p.N + dq64s::kRows - 1) / dq64s::kRows);
    if (units <= 512 || (units <= 1024 && longest_row(p.f) >= 256)) return true;
    return longest_row(p.f) >= 48 * 32 && chain_is_the_time(p.f, 512, 256, 2.35, 1.95);
}

// ---- dK, dV --------------------------------------------------------------------------
// Which key tile's main workgroup is block `bid` (the blocks before n_extra are sink
// segments)?  Workgroups are dealt to the eight dies round-robin, and each die has its own
// L2: every die gets a contiguous run of the (batch, KV head, key tile) list, so that the
// workgroups running side by side on a die hold neighbouring key tiles, whose query tiles
// largely coincide (tile T is read by key tile kt at its step T - 2 kt).  The Q and dO
// rows then come out of L2 instead of HBM: 0.8 GB instead of 4.6 GB per launch on the
// 16k-token benchmark layer.  The sink segments stay in front, dealt round-robin: a first
// attempt that gave them to one die lost more to the imbalance than the cache gave back.
// The launch rounds the number of main workgroups up to a multiple of the die count; ids
// past the list belong to workgroups that return at once.
// Dies that share a pair take its key tiles in turn where the window is a sixteenth of the sequence or more (plan_bwd): the
// causal key tiles of the last window are shorter than the rest, and with contiguous parts one die has them all.  With
// narrower windows that is little, and neighbours in one L2 save more.  The backward, contiguous parts / in turn (us):
//    window, of the tokens                       1/64           1/32           1/16           1/8            1/2
//    4 heads on 1   65536 tokens             645 / 652     1102 / 1113    2032 / 1875    3943 / 3363
//                  131072                   1979 / 2090    3811 / 3816    7278 / 6880   14361 / 13297
//      D = 64       65536                    347 / 351      615 / 618     1152 / 1035    2266 / 1910
//    8 on 2         16384                    182 / 181      250 / 252      380 / 383      648 / 543
//                   65536                   1185 / 1226    1948 / 1986    3790 / 3687    7329 / 6741
//    16 on 4        16384                    307 / 307      416 / 417      625 / 634     1058 / 970     3780 / 2790
//                   65536                   2291 / 2309    3772 / 3777    7037 / 6937   13808 / 12982
// (n_main: their number, as the launch rounds it up.)
__host__ __device__ __forceinline__ int dkv_main_item(const BwdParams &p, unsigned bid, int n_extra, unsigned n_main, int n_kt) {
    const unsigned xcd = bid % kXcds, slot = (bid - (unsigned)n_extra) / kXcds, dies = 1u << p.die_shift;
    const unsigned per_die = dies > 1 ? (unsigned)n_kt : n_main / kXcds;
    const unsigned off = slot * dies + (xcd & (dies - 1));
    return off < per_die ? (int)((xcd >> p.die_shift) * per_die + off) : 0x7fffffff;
}

// The work list of the dK/dV kernels: first the segments of the sink key tiles (rows beyond the band), then one
// workgroup per key tile of 128 keys (band rows; for key tiles without sinks also the generated rows).  Under a causal mask
// the first key tiles are seen by the most rows.
// Pieces of a key tile (BwdParams::n_split) come in the order key tile, piece, pair: the first key tiles, which are the longest,
// first, and where the pairs are a multiple of eight each die keeps to its own.
struct DkvItem {
    int kt, pair;  // key tile, (batch, KV head)
    int seg;       // -1 for a key tile's main workgroups
    int piece;     // which of them
};
__device__ __forceinline__ bool dkv_item(const BwdParams &p, DkvItem &w) {
    const int n_kt = (p.N + 127) / 128;
    const int n_extra = p.B * p.Hkv * p.n_sink_kt * p.n_seg;
    const unsigned bid = blockIdx.x;
    w.piece = 0;
    if ((int)bid < n_extra) {
        const unsigned tile = fastdiv(bid, p.div_seg);
        w.seg = (int)(bid - tile * (unsigned)p.n_seg);
        w.pair = (int)fastdiv(tile, p.div_sink_kt);
        w.kt = (int)tile - w.pair * p.n_sink_kt;
        return true;
    }
    w.seg = -1;
    if (p.n_split > 1) {
        const unsigned id = bid - (unsigned)n_extra, of_pair = fastdiv(id, p.div_pairs);
        w.pair = (int)(id - of_pair * (unsigned)(p.B * p.Hkv));
        w.kt = (int)fastdiv(of_pair, p.div_split);
        w.piece = (int)of_pair - w.kt * p.n_split;
        return w.kt < n_kt;
    }
    const int id = dkv_main_item(p, bid, n_extra, gridDim.x - (unsigned)n_extra, n_kt);
    if (id >= p.B * p.Hkv * n_kt) return false;  // (the grid is rounded up to a multiple of eight)
    w.pair = (int)fastdiv((unsigned)id, p.div_kt);
    w.kt = id - w.pair * n_kt;
    return true;
}

// A piece's share [from, to) of its key tile's steps (their product is small: few key tiles have pieces, see plan_pieces).
__device__ __forceinline__ int dkv_piece_start(const BwdParams &p, const DkvItem &w, int total, int next) {
    return w.seg >= 0 || p.n_split == 1 ? next * total : (int)fastdiv((unsigned)total * (unsigned)(w.piece + next), p.div_split);
}

// Its tiles of kBq query rows (head dimension 128): the band, then -- if a key is a sink, or there are generated rows --
// the rest.  For a sink key tile the rest is cut into segments, and the main workgroup keeps the band.
struct DkvTiles {
    int lo, n_band;  // the band's first tile, and how many
    int x;           // the first tile of the rest
    int n;           // all of them
    __host__ __device__ __forceinline__ int at(int i) const { return i < n_band ? lo + i : x + (i - n_band); }
};
__host__ __device__ __forceinline__ DkvTiles dkv_tiles(const BwdParams &p, const DkvItem &w) {
    const int N = p.N, k0 = w.kt * 128, k1 = min(k0 + 127, N - 1);
    const int last = (N - 1) / kBq, band_hi = min(N - 1, k1 + p.f.W - 1) / kBq;
    DkvTiles t{k0 / kBq, 0, last + 1, 0};
    t.n_band = band_hi - t.lo + 1;
    int x_end = last;
    if (w.kt < p.n_sink_kt) {
        if (w.seg >= 0) {
            t.n_band = 0;
            t.x = band_hi + 1 + w.seg * p.seg_tiles;
            x_end = min(last, t.x + p.seg_tiles - 1);
        }
    } else if (p.f.P < N) {
        t.x = max(band_hi + 1, p.f.P / kBq);
    }
    t.n = t.n_band + max(0, x_end - t.x + 1);
    return t;
}

}  // namespace
}  // namespace swaa

#include "swaa_bwd_dkv_d128.h"        // dK, dV, head dimension 128
#include "swaa_bwd_dkv_d128_short.h"  // ... of few query tiles per key tile
#include "swaa_bwd_dkv_d64.h"         // dK, dV, head dimension 64

namespace swaa {
namespace {

// dK, dV of the key tiles that have partial sums (all of them, or those with sinks): pieces, then segments, in this order.
template <int D>
__global__ __launch_bounds__(kThreads) void swaa_bwd_part_sum_kernel(const BwdParams p) {
    // one thread per 4 consecutive head-dimension elements of one key
    const int n_kt = p.n_split > 1 ? (p.N + 127) / 128 : p.n_sink_kt;
    const long long per_kt = 128LL * D / 4;
    const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
    const long long total = (long long)p.B * p.Hkv * n_kt * per_kt;
    if (idx >= total) return;
    const int e = (int)(idx % per_kt);
    const long long kt_id = idx / per_kt;  // pair * n_kt + kt
    const int kt = (int)(kt_id % n_kt), pair = (int)(kt_id / n_kt);
    const int key = kt * 128 + e / (D / 4);
    const int d = (e % (D / 4)) * 4;
    if (key >= p.N) return;
    const float *slot = p.partial + (size_t)p.first_part(pair, kt) * (2 * 128 * D) + (size_t)(e / (D / 4)) * D + d;
    float4 sk = {0.f, 0.f, 0.f, 0.f}, sv = {0.f, 0.f, 0.f, 0.f};
    const int n = p.parts(kt);
#pragma unroll 4
    for (int s = 0; s < n; ++s) {
        const float4 a = *reinterpret_cast<const float4 *>(slot + (size_t)s * 2 * 128 * D);
        const float4 c = *reinterpret_cast<const float4 *>(slot + (size_t)s * 2 * 128 * D + 128 * D);
        sk.x += a.x; sk.y += a.y; sk.z += a.z; sk.w += a.w;
        sv.x += c.x; sv.y += c.y; sv.z += c.z; sv.w += c.w;
    }
    const size_t row = ((size_t)pair * p.N + key) * D + d;
    bf16x4 k4 = {(__bf16)(sk.x * p.f.scale), (__bf16)(sk.y * p.f.scale), (__bf16)(sk.z * p.f.scale), (__bf16)(sk.w * p.f.scale)};
    bf16x4 v4 = {(__bf16)sv.x, (__bf16)sv.y, (__bf16)sv.z, (__bf16)sv.w};
    *reinterpret_cast<bf16x4 *>(p.dk + row) = k4;
    *reinterpret_cast<bf16x4 *>(p.dv + row) = v4;
}

// Is a key tile seen by so few query tiles that eight waves with less around their loop, which leave out every block
// without a visible pair, beat one wave per SIMD, whose steps are faster?  Backward of head dimension 128, one wave per
// SIMD / eight waves (us; 32 heads on 8 unless stated):
//    tiles                                   4096 tokens (256 workgroups), window    16384 tokens (1024), window
//    100 tokens   2   42.9 / 39.2             64   3   86.1 / 81.8                    128   4   409 / 390
//    300          5   69.6 / 66.9            256   6  118.6 / 115.9                   256   6   498 / 482
//    384          6   75.9 / 75.9            384   8  138.9 / 138.1                   512  10   672 / 675  (4 sinks 794 / 782)
//    640         10  106.9 / 110.8           512  10  160.0 / 160.2                  1024  18  1032 / 1054
//    (8 heads on 8)                          (8 on 8)                                 (16 heads on 8)
//    500          8   53.8 / 52.0            512  10   71.4 / 69.9                    512  10   377 / 374
//    1000        16   80.1 / 80.1            768  14   84.2 / 83.4                    768  14   469 / 472
// With few workgroups the longest one is the time, and where sinks see many rows that is a segment, in which the eight
// waves keep two busy: 16 heads on 2, 4 sinks, 4096 tokens: window 64 97.8 / 94.9, 128 113 / 112, 256 144 / 148.
// Generated rows see every key, and their blocks have few edges: they count half.
// A piece of a key tile (plan_pieces) has a part of its tiles: 500 tokens in six 63.4 / 61.5, 700 in six 71.7 / 70.8, 1000 in four
// 90.6 / 91.2, 2048 in three 178 / 184; 8 heads on 8, 1000 tokens in two 78.0 / 76.6, 1500 in two 98.3 / 94.1, 2048 120 / 122.
bool dkv_short(const BwdParams &p) {
    const long long n_main = (long long)p.B * p.Hkv * ((p.N + 127) / 128);
    const int G = p.f.G, all = (p.N + kBq - 1) / kBq, band = (p.f.W + 127) / kBq + 1;
    const int tiles = (band < all ? band : all) + (p.N - p.f.P) / (2 * kBq);
    if (p.n_split > 1) return tiles <= (G == 1 ? 12 : 3) * p.n_split;
    if (n_main >= 256) return tiles <= (G <= 2 ? 13 : n_main >= 512 ? 10 : 9);
    return tiles <= (G == 1 ? 12 : p.n_seg > 0 ? 4 : G <= 3 ? 8 : 6);
}

template <int D>
hipError_t launch_bwd_d(const BwdParams &p, hipStream_t stream) {
    // more than 64 KiB of LDS per workgroup has to be requested once per device
    static std::atomic<unsigned long long> configured{0};
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    const unsigned long long bit = 1ull << (dev & 63);
    const bool first_time = !(configured.load(std::memory_order_acquire) & bit);
    if constexpr (D == 128)
        err = launch_bwd_dq_pipelined_d128(p, stream);  // swaa_bwd_dq_pipelined.hip
    else if (dq64_short(p))
        hipLaunchKernelGGL(swaa_bwd_dq64_short_kernel, dim3((unsigned)(p.B * p.Hq * ((p.N + dq64s::kRows - 1) / dq64s::kRows))),
                           dim3(dq64s::kThreads), dq64s::kBytes, stream, p);
    else
        hipLaunchKernelGGL(swaa_bwd_dq_kernel, dim3((unsigned)(p.f.chunk * kXcds)), dim3(dq64::kThreads), dq64::kBytes, stream, p);
    if (err == hipSuccess) err = hipGetLastError();
    if (err != hipSuccess) return err;
    const long long n_kt = (p.N + 127) / 128;
    const long long pairs = (long long)p.B * p.Hkv;
    if (first_time) {
        if constexpr (D == 128) {
            err = hipFuncSetAttribute(reinterpret_cast<const void *>(&swaa_bwd_dkv_dma_kernel),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, dkv128::kBytes);
            if (err == hipSuccess)
                err = hipFuncSetAttribute(reinterpret_cast<const void *>(&swaa_bwd_dkv_dma_short_kernel),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, dkv128short::kBytes);
        } else {
            err = hipFuncSetAttribute(reinterpret_cast<const void *>(&swaa_bwd_dkv_kernel<D>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, dkv64::kBytes);
        }
        if (err != hipSuccess) return err;
        configured.fetch_or(bit, std::memory_order_release);
    }
    // sink segments first (the longest items), then the key tiles' main workgroups, their number
    // rounded up to a multiple of the die count (dkv_main_item)
    const long long n_main = p.n_split > 1 ? pairs * n_kt * p.n_split : (pairs * n_kt + kXcds - 1) / kXcds * kXcds;
    const dim3 dkv_grid((unsigned)(pairs * (long long)p.n_sink_kt * p.n_seg + n_main));
    if constexpr (D == 128) {
        if (dkv_short(p))
            hipLaunchKernelGGL(swaa_bwd_dkv_dma_short_kernel, dkv_grid, dim3(dkv128short::kThreads), dkv128short::kBytes, stream, p);
        else
            hipLaunchKernelGGL(swaa_bwd_dkv_dma_kernel, dkv_grid, dim3(dkv128::kThreads), dkv128::kBytes, stream, p);
    } else
        hipLaunchKernelGGL(swaa_bwd_dkv_kernel<D>, dkv_grid, dim3(dkv64::kThreads), dkv64::kBytes, stream, p);
    err = hipGetLastError();
    if (err != hipSuccess || (p.n_sink_kt == 0 && p.n_split == 1)) return err;
    const long long threads = pairs * (p.n_split > 1 ? n_kt : p.n_sink_kt) * (128LL * D / 4);
    hipLaunchKernelGGL(swaa_bwd_part_sum_kernel<D>, dim3((unsigned)((threads + kThreads - 1) / kThreads)), dim3(kThreads),
                       0, stream, p);
    return hipGetLastError();
}

// The segments of the sink key tiles, about as long as an ordinary key tile's band or a piece of it, but at most 512 of them in
// all, or one to a tile where there are more tiles than that.
void plan_sink_segments(BwdParams &p) {
    const int N = p.N, W = p.f.W, S = p.f.S;
    p.n_sink_kt = 0;
    p.n_seg = 0;
    p.seg_tiles = 1;
    // rows beyond the band of the last sink key: only worth separate workgroups if there are any
    const int tq_last = (N - 1) / kBq;
    const int first_beyond = (min(N - 1, 127 + W - 1)) / kBq + 1;  // of key tile 0, the longest range
    if (S == 0 || first_beyond > tq_last) return;
    p.n_sink_kt = (min(S, N) + 127) / 128;
    const int range = tq_last - first_beyond + 1;
    long long seg = ((W + 127) / kBq + p.n_split) / p.n_split;
    const long long groups = (long long)p.B * p.Hkv * p.n_sink_kt;
    while (seg < range && (range + seg - 1) / seg * groups > 512) seg *= 2;
    p.seg_tiles = (int)seg;
    p.n_seg = (int)((range + seg - 1) / seg);
}

// Into how many pieces are the key tiles' steps cut?  One workgroup runs on a compute unit, so 64 key tiles (1000 tokens on 8
// KV heads) leave three quarters of the chip idle, and causal key tiles differ: the first is seen by all rows, the last by few.
// But every piece leaves 128 KiB of partial sums (head dimension 128) for the last kernel.  The time of a plan, in us: pieces that
// have a compute unit each take as long as the longest; more of them share the chip evenly but for a third of the longest;
// a step takes 1.67 (head dimension 64: 1.13), a workgroup six of them outside its loop; the last kernel 4, and a piece's partial sums
// 0.04 while compute units are idle, then 0.03.  The backward, one piece / as planned / the best of 1 to 8 (us; 4 sinks):
//    head dimension 128           500 tokens        1000              2048              4096              2048, window 512
//      32 heads on 8              94 / 61 / 59      156 / 91 / 91     281 / 174 / 174   594 / 471 / 471   135 / 130 / 125
//      16 heads on 4              95 / 58 / 58      155 / 77 / 77     277 / 136 / 136   528 / 296 / 296   129 / 91 / 91
//      8 heads on 8               54 / 53 / 53      81 / 79 / 77      134 / 122 / 122   240 / 225 / 225   79 / 79 / 79
//    head dimension 64
//      32 heads on 8              65 / 45 / 45      109 / 69 / 69     203 / 124 / 124   409 / 312 / 312   100 / 87 / 82
//      16 heads on 4              65 / 40 / 40      110 / 61 / 61     201 / 103 / 103   386 / 208 / 208   97 / 66 / 64
// With 512 key tiles and more the best of one to four is at most 1 % ahead of whole ones, or behind.  Windows without
// sinks have no partial sums, and callers that know their workspace as delta alone.
int plan_pieces(BwdParams &p, int D) {
    const int n_kt = (p.N + 127) / 128, pairs = p.B * p.Hkv, G = p.f.G;
    if ((long long)pairs * n_kt >= 512 || (p.f.S == 0 && p.f.W < p.N)) return 1;
    const int all = (p.N + kBq - 1) / kBq, generated = (p.N - p.f.P) / kBq;
    const int band = min(all, (p.f.W + 126) / kBq + 1), longest = min(all, band + generated);  // query tiles that see a key tile
    const int full = min(n_kt, (all - band) / 2 + 1);  // key tiles with a whole band; the others have two tiles fewer each time
    const float tiles = (float)(full * band) + (float)(n_kt - full) * (0.5f * (float)band + 1.f) + (float)(n_kt * generated);
    float best = 0.f;
    int pick = 1;
    for (int n = 1; n <= 8 && (n == 1 || pairs * n_kt * n <= 1024); ++n) {
        p.n_split = n;
        plan_sink_segments(p);
        constexpr float kStart = 6.f;
        const int units = pairs * (n_kt * n + p.n_sink_kt * p.n_seg);
        const float seg = p.n_seg ? (float)(p.seg_tiles * G) : 0.f, piece = (float)(longest * G) / (float)n;
        const float one = (seg > piece ? seg : piece) + kStart;
        const float steps = (float)(pairs * G) * (tiles + (float)(p.n_sink_kt * p.n_seg * p.seg_tiles));
        const float shared = (steps + kStart * (float)units) * (1.f / 256.f) + 0.3f * one;
        float t = (D == 128 ? 1.67f : 1.13f) * (units <= 256 || one > shared ? one : shared);
        if (n > 1) t += 4.f + (units <= 256 ? 0.04f : 0.03f) * (float)units * (float)D * (1.f / 128.f);
        // (more pieces than the best so far have to gain 2 %, and any at all 2 us)
        if (n == 1 || t < 0.98f * best - (pick == 1 ? 2.f : 0.f)) {
            best = t;
            pick = n;
        }
    }
    return pick;
}

}  // namespace

void plan_bwd(BwdParams &p, int D, bool pieces) {
    p.die_shift = 16LL * p.f.W >= p.N ? die_shift((long long)p.B * p.Hkv) : 0;  // (dkv_main_item has both sides of the line)
    // (one workgroup of dQ to a compute unit: in the order of their lengths; two sequences of 2048 tokens 275 us folded, 262)
    if (D == 128) p.f.fold = 0x7fffffff;
    p.n_split = pieces ? plan_pieces(p, D) : 1;
    plan_sink_segments(p);
    p.div_kt = make_fastdiv((unsigned)((p.N + 127) / 128));
    p.div_pairs = make_fastdiv((unsigned)(p.B * p.Hkv));
    p.div_hkv = make_fastdiv((unsigned)p.Hkv);
    p.div_group = make_fastdiv((unsigned)(p.Hq / p.Hkv));
    p.div_split = make_fastdiv((unsigned)p.n_split);
    p.div_seg = make_fastdiv((unsigned)p.n_seg);
    p.div_sink_kt = make_fastdiv((unsigned)p.n_sink_kt);
}

long long bwd_workspace_floats(const BwdParams &p, int D) {
    const long long rows = ((long long)p.B * p.Hq * p.N + 3) / 4 * 4;  // the partial sums start 16-byte aligned
    return rows + p.first_part(p.B * p.Hkv, 0) * 2 * 128 * D;
}

hipError_t launch_bwd(const BwdParams &p, int D, hipStream_t stream) {
    return D == 128 ? launch_bwd_d<128>(p, stream) : launch_bwd_d<64>(p, stream);
}

}  // namespace swaa
