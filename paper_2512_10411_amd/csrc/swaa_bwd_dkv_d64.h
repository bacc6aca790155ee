// dK and dV, head dimension 64, gfx950 (formulas and mask: swaa_bwd.hip, which includes this file and holds the
// work list).
//
// A workgroup owns 128 keys; eight waves, two per SIMD: wave w owns the 32 keys 32 (w % 4).., whose K and V rows stay in
// AccVGPRs (B operands of S = Q K^T and dP = dO V^T), and every other block of 32 query rows of the work list (query head, row
// block); the two halves of the list are added through LDS at the end.
//
// Per 32 rows x 32 keys a wave owes the matrix pipe 512 cycles and the vector ALU about 400 (16 exponentials among
// them), and the operands come out of LDS: what matters is that the three run at the same time.  So a wave works on
// three blocks at once, as the forward kernel does (swaa_fwd_pipelined.hip): sub-step n alternates the MFMAs of
// S, dP of block n + 1 and of dV^T += dO^T P, dK^T += Q^T dS of block n - 1, and in their shadow the vector work of block n,
// fixed by hand with scheduling fences; LDS operands are asked for kAhead MFMAs ahead.
// Two sequences of 4001 tokens, 16 heads on 4, window 1000: 126 us with twelve waves, three per SIMD, that took products, vector
// work and products in turn, all in the same phase; now 96.  16384 tokens, 32 heads on 8, window 8192: 1970 -> 1660.  There the matrix
// pipe is busy 47 % of the time, the vector ALU 46 %, LDS 35 %; on the first shape, whose 280 workgroups leave the
// compute units empty for 29 % of it, 30, 33 and 23 % (profiles/swaa_train_d64_sq_counters.txt).  No one thing bounds
// the loop: without the exponentials, the copies, the barrier or a third of the LDS reads it takes 0 to 5 % less.  (Also tried: one wave per
// SIMD on 64 keys, as for head dimension 128: no faster than the twelve waves.)
//
// Blocks travel HBM -> LDS by global_load_lds_dwordx4 into a ring of six buffers per half of the list, two blocks and one
// barrier per step: a step's two sub-steps read four blocks while the next two arrive.  A block lies in LDS as two slices of
// 64 bytes of every row, 16-byte chunk c of the four at chunk c ^ ((r >> 2) & 3): row fragments and transposed ones are
// free of bank conflicts, and two addresses each reach all of them through the instructions' offset fields.
// A block without a visible pair takes part in nothing: its P and dS are cleared, and the products read a buffer of
// zeros in its place, whatever its rows hold.  MFMAs through inline assembly (rules: swaa_tile_d128.h; tests/test_asm_hazards.py
// checks them).  No static LDS: the dynamic LDS starts at address 0.
#ifndef SWAA_BWD_DKV_D64_H_
#define SWAA_BWD_DKV_D64_H_

#include "swaa_bwd.h"
#include "swaa_tile_d128.h"

namespace swaa {
namespace {
namespace dkv64 {

constexpr int kThreads = 512;
constexpr int kD = 64, kKS = kD / 16, kDB = kD / 32, kRowBytes = 2 * kD;
constexpr int kParts = 2;                           // halves of the list
constexpr int kSliceBytes = 32 * 64;                // 64 bytes of every row of a block
constexpr int kBlockBytes = 32 * kRowBytes;         // Q, or dO, of a block: 4 KiB
constexpr int kLseAt = 2 * kBlockBytes;             // behind Q and dO: -lse (log2 units) and -delta of the rows
constexpr int kBufBytes = kLseAt + 2 * 32 * 4;
constexpr int kBufs = 6;
constexpr int kPartBytes = kBufs * kBufBytes;
constexpr int kZero = kParts * kPartBytes;          // a block of zeros, Q and dO
constexpr int kSumBytes = 4 * 32 * kD * 4;          // of the final sums, for dK and for dV, in the rings' place
constexpr int kBytes = kZero + 2 * kBlockBytes;
constexpr int kAhead = 3;                           // MFMAs between an LDS operand read and its use
static_assert(kBytes >= 2 * kSumBytes && kBytes <= 160 * 1024, "one workgroup's LDS");

typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 lds_f4(uint32_t addr) { return *(const f32x4 __attribute__((address_space(3))) *)(uintptr_t)addr; }
// first element handled by chunk c of the vector work: 16 over chunks 0..13
__device__ constexpr int first_elem(int c) { return c >= 14 ? 16 : c * 16 / 14; }

}  // namespace dkv64

template <int D>
__global__ __launch_bounds__(dkv64::kThreads, 2) void swaa_bwd_dkv_kernel(const BwdParams p) {
    using namespace dkv64;
    static_assert(D == dkv64::kD, "the layout below is for rows of 128 bytes");

    const int N = p.N, W = p.f.W, S = p.f.S, P = p.f.P, G = p.f.G;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
    const int kq = wave & 3, part = wave >> 2;
    DkvItem item;
    if (!dkv_item(p, item)) return;
    const int kt = item.kt, pair = item.pair, seg = item.seg;
    const int b = (int)fastdiv((unsigned)pair, p.div_hkv), kvh = pair - b * p.Hkv;
    const int k0 = kt * 128, k1 = min(k0 + 127, N - 1);  // the workgroup's keys
    const int kw0 = k0 + 32 * kq, kw1 = kw0 + 31;         // this wave's keys
    const int key = kw0 + l32;                            // this lane's key column

    // Row blocks (32 rows) with a row that sees one of the workgroup's keys: the band blocks, then
    // -- if a key is a sink, or there are generated rows -- the rest.  For a sink key tile the
    // rest is cut into segments of seg_tiles 64-row tiles, and the main workgroups keep the band.
    const int last_block = (N - 1) / 32;
    const int first = k0 / 32;
    int band_hi = min(N - 1, k1 + W - 1) / 32;
    int x0 = last_block + 1, x1 = last_block;  // second range
    if (kt < p.n_sink_kt) {
        band_hi = min(band_hi | 1, last_block);  // (the segments start at a whole tile)
        if (seg >= 0) {
            x0 = band_hi + 1 + 2 * seg * p.seg_tiles;
            x1 = min(last_block, x0 + 2 * p.seg_tiles - 1);
        }
    } else if (P < N) {
        x0 = max(band_hi + 1, P / 32);
    }
    const int n_band = seg >= 0 ? 0 : band_hi - first + 1;
    const int n_blocks = n_band + max(0, x1 - x0 + 1);  // per query head
    const int all_blocks = G * n_blocks, from = dkv_piece_start(p, item, all_blocks, 0), total = dkv_piece_start(p, item, all_blocks, 1) - from;

    f32x16 acc[2][kDB];  // dV^T, dK^T
#pragma unroll
    for (int w = 0; w < 2; ++w)
#pragma unroll
        for (int db = 0; db < kDB; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[w][db][e] = 0.f;
    asm volatile("s_nop 1" : "+a"(acc[0][0]), "+a"(acc[0][1]), "+a"(acc[1][0]), "+a"(acc[1][1]));

    if (total > 0) {
        // ---- HBM -> LDS copies.  A wave instruction moves 64 bytes of 16 rows: wave kq of a half of the list slice kq / 2 of rows
        // 16 (kq % 2).. of its blocks.  The LDS side is linear in the lane id, the swizzle is applied on the global side.
        // Rows past the end of the sequence repeat its last row (they stay invisible).
        const int lrow = 16 * (kq & 1) + (lane >> 2);
        const uint32_t lchunk = (uint32_t)((kq >> 1) * 64 + (((lane & 3) ^ (lane >> 4)) << 4));
        const uint32_t ring = (uint32_t)(part * kPartBytes), lds_copy = ring + (uint32_t)((kq >> 1) * kSliceBytes + (kq & 1) * 1024);
        auto copy16 = [](uint32_t offset, const __bf16 *base, uint32_t lds) {
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(offset), "s"(base), "s"(lds) : "memory");
        };
        // the next block to ask for: its place in the part's list, in its head's list, and the head's rows
        int rq_at = part, rq_n = (from + part) % n_blocks;
        size_t rq_base = ((size_t)b * p.Hq + kvh * G + (from + part) / n_blocks) * (size_t)N;
        float lreg = 0.f, dlreg = 0.f;
        // block into the buffer at `buf`; its first row, or -32 behind the end of the list
        auto request = [&](uint32_t buf, size_t &rows, int &left) {
            if (rq_at >= total) return -32;
            const int row0 = 32 * (rq_n < n_band ? first + rq_n : x0 + (rq_n - n_band));
            rows = rq_base + (size_t)row0;
            left = N - 1 - row0;
            const uint32_t off = (uint32_t)min(lrow, left) * kRowBytes + lchunk;
            copy16(off, p.f.q + rows * D, lds_copy + buf);
            copy16(off, p.dout + rows * D, lds_copy + buf + kBlockBytes);
            rq_at += kParts;
            rq_n += kParts;
            while (rq_n >= n_blocks && rq_at < total) {
                rq_n -= n_blocks;
                rq_base += N;
            }
            return row0;
        };
        // two blocks, the first only if `both`; the part's first wave asks for their lse and delta, lanes 32.. for the second's
        auto request_two = [&](uint32_t buf0, uint32_t buf1, int &row0, int &row1, bool both) {
            size_t rows0 = 0, rows1 = 0;
            int left0 = 0, left1 = 0;
            row0 = both ? request(buf0, rows0, left0) : -32;
            row1 = request(buf1, rows1, left1);
            if (kq == 0) {  // (first touched in publish; a block that is not there repeats row 0 of the tensors)
                const size_t row = hf ? rows1 + (size_t)min(l32, left1) : rows0 + (size_t)min(l32, left0);
                lreg = p.f.lse[row];
                dlreg = p.delta[row];
            }
        };
        auto publish = [&](uint32_t buf0, uint32_t buf1) {
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's copies, and lse and delta
            if (kq == 0) {
                float __attribute__((address_space(3))) *at =
                    (float __attribute__((address_space(3))) *)(uintptr_t)(ring + (uint32_t)kLseAt + (hf ? buf1 : buf0) + (uint32_t)(l32 * 4));
                at[0] = lreg * -1.44269504088896340736f;
                at[32] = -dlreg;
            }
        };
        auto barrier = [&]() {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };

        // this wave's K and V rows as B operands (rows past the end repeat the last key; they stay invisible)
        bf16x8 kf[kKS], vf[kKS];
        {
            const size_t g = (((size_t)b * p.Hkv + kvh) * (size_t)N + min(key, N - 1)) * D + 8 * hf;
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks) {
                kf[ks] = *reinterpret_cast<const bf16x8 *>(p.f.k + g + 16 * ks);
                vf[ks] = *reinterpret_cast<const bf16x8 *>(p.f.v + g + 16 * ks);
            }
        }
        // the block of zeros: 8 KiB, 16 bytes per thread
        *(u32x4 __attribute__((address_space(3))) *)(uintptr_t)((uint32_t)(kZero + tid * 16)) = u32x4{0u, 0u, 0u, 0u};

        // buffers of blocks n - 1, n, n + 1, .. at the start of a step (n even)
        auto next_buf = [](uint32_t buf) { return buf == (uint32_t)((kBufs - 1) * kBufBytes) ? 0u : buf + (uint32_t)kBufBytes; };
        uint32_t at_m1 = (uint32_t)(5 * kBufBytes), at_0 = 0u;
        int row0, row1, row2, none;  // first rows of blocks n, n + 1, n + 2 (-32: no block)
        request_two(at_m1, at_0, none, row0, false);
        publish(at_m1, at_0);
        request_two((uint32_t)kBufBytes, (uint32_t)(2 * kBufBytes), row1, row2, true);
        publish((uint32_t)kBufBytes, (uint32_t)(2 * kBufBytes));
        asm volatile("s_nop 1" : "+a"(kf[0]), "+a"(kf[1]), "+a"(kf[2]), "+a"(kf[3]), "+a"(vf[0]), "+a"(vf[1]), "+a"(vf[2]), "+a"(vf[3]));
        barrier();

        // ---- per-lane fragment addresses inside a block (swizzle folded in)
        //  * row fragment, k-step ks: row l32, logical chunk 2 ks + hf: even and odd k-steps
        //  * transposed fragment: rows 4 hf + j16/4 (lo) and 8 further (hi), logical chunk 4 db + 2 (grp & 1) + (j16 & 3) / 2
        uint32_t row_lane[2], col_lane[2];
        {
            const uint32_t r = ring + (uint32_t)(l32 * 64 + ((hf ^ ((l32 >> 2) & 3)) << 4));
            row_lane[0] = r;
            row_lane[1] = r ^ 32u;
            const int grp = lane >> 4, j16 = lane & 15, cl = 2 * (grp & 1) + ((j16 & 3) >> 1);
            const uint32_t c = (uint32_t)((4 * hf + (j16 >> 2)) * 64 + 8 * (j16 & 1));
            col_lane[0] = c + (uint32_t)((cl ^ hf) << 4);
            col_lane[1] = c + (uint32_t)(8 * 64 + ((cl ^ hf ^ 2) << 4));
            asm volatile("" : "+v"(row_lane[0]), "+v"(row_lane[1]), "+v"(col_lane[0]), "+v"(col_lane[1]));
        }
        const uint32_t lse_lane = ring + (uint32_t)(kLseAt + 16 * hf);
        const float c2 = p.f.scale_log2;

        f32x16 s[2], dp[2];           // of block n in [n % 2]
        bf16x8 pf[2][2], dsf[2][2];   // [n % 2][16-row step]
        f32x4 nl[4];                  // -lse of the rows of the block whose exponentials are next
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
                for (int e = 0; e < 8; ++e) pf[x][st][e] = dsf[x][st][e] = (__bf16)0.f;

        // Which of the 32 rows from i0 on see this lane's key?  A bit each, moved so that bit 0 is row 4 hf.
        auto visible_rows = [&](int i0) {
            auto below = [](int t) { return t >= 32 ? ~0u : (1u << min(max(t, 0), 31)) - 1u; };  // bits 0 .. t - 1
            const int end = key < S ? N : min(key + W, N);
            uint32_t m = below(end - i0) & ~below(key - i0);
            if (i0 + 31 >= P) m |= below(N - i0) & ~below(max(key, P) - i0);
            return m >> (4 * hf);
        };
        // clears P and dS of the pairs that are not visible
        auto clear_invisible = [&](bf16x8 (&pp)[2], bf16x8 (&dd)[2], uint32_t rows) {
#pragma unroll
            for (int st = 0; st < 2; ++st) {
                u32x4 pb = __builtin_bit_cast(u32x4, pp[st]), db = __builtin_bit_cast(u32x4, dd[st]);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int bit = 16 * st + 8 * (j / 2) + 2 * (j % 2);
                    const uint32_t lo = (uint32_t)((int)(rows << (31 - bit)) >> 31), hi = (uint32_t)((int)(rows << (30 - bit)) >> 31);
                    const uint32_t keep = (lo & 0xffffu) | (hi & 0xffff0000u);
                    pb[j] &= keep;
                    db[j] &= keep;
                }
                pp[st] = __builtin_bit_cast(bf16x8, pb);
                dd[st] = __builtin_bit_cast(bf16x8, db);
            }
            asm volatile("s_nop 1" : "+v"(pp[0]), "+v"(pp[1]), "+v"(dd[0]), "+v"(dd[1]));  // (two wait states in front of the MFMAs)
        };
        // of the 32 x 32 pairs of the rows from i0 on: are all visible, is any?  (rows -32.. are no block: below every key)
        const int full_to = kw1 < S ? N - 32 : min(N - 32, kw0 + W - 32), any_to = kw0 >= N ? -1 : kw0 < S ? N - 1 : kw1 + W - 1;
        auto all_visible = [&](int i0) { return i0 >= kw1 && (i0 <= full_to || (i0 >= P && i0 + 31 < N)); };
        auto any_visible = [&](int i0) { return i0 + 31 >= kw0 && i0 >= 0 && (i0 <= any_to || (i0 + 31 >= P && kw0 < N)); };

        // LDS operand of slot i of a sub-step: even slots S (k-steps 0..3), then dP; odd slots dV and dK in turn
        auto fetch = [&](int i, uint32_t (&row)[2], uint32_t (&col)[2]) {
            if (i % 2 == 0) {
                const int op = i / 2, ks = op % kKS;
                return lds_read16(row[ks % 2] + (uint32_t)((ks / 2) * kSliceBytes + (op < kKS ? 0 : kBlockBytes)));
            }
            const int op = i / 2, st = op / 4, db = (op / 2) % 2;
            const uint32_t off = (uint32_t)((op % 2 == 0 ? kBlockBytes : 0) + db * kSliceBytes + 16 * st * 64);
            const s16x4 lo = lds_read8_tr(col[0] + off), hi = lds_read8_tr(col[1] + off);
            return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        };
        auto load_delta = [&](f32x16 &x, uint32_t buf) {
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
                const f32x4 t = lds_f4(lse_lane + buf + (uint32_t)(32 * e4 + 128));
#pragma unroll
                for (int i = 0; i < 4; ++i) x[4 * e4 + i] = t[i];
            }
        };

        // ---- prologue: S and dP of the first block ----
        {
            uint32_t row[2] = {row_lane[0] + at_0, row_lane[1] + at_0}, col[2] = {0u, 0u};
            load_delta(dp[0], at_0);
            asm volatile("s_nop 1" : "+v"(dp[0]));  // (no copy of theirs right in front of a product)
#pragma unroll
            for (int q = 0; q < 4; ++q) nl[q] = lds_f4(lse_lane + at_0 + (uint32_t)(32 * q));
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks) {
                const bf16x8 qfrag = fetch(2 * ks, row, col), dofrag = fetch(2 * (kKS + ks), row, col);
                if (ks == 0)
                    mfma_s_first(s[0], qfrag, kf[0]);
                else
                    mfma_s(s[0], qfrag, kf[ks]);
                mfma_s(dp[0], dofrag, vf[ks]);
            }
            asm volatile("s_nop 15\n\ts_nop 7" : "+v"(s[0]), "+v"(dp[0]));
        }

        // Sub-step n: S, dP of block n + 1 (buffer at_next) | vector work of block n | dV, dK of block n - 1 (buffer at_prev).
        bool prev_live = false;  // does block n - 1 have a visible pair?
        bf16x8 fr[16 + kAhead];
        auto substep = [&](auto parity, auto first_of_step, int i0, uint32_t at_prev, uint32_t at_next, uint32_t at_after) {
            constexpr int cur = decltype(parity)::value;
            constexpr bool kFirst = decltype(first_of_step)::value;  // of the step's two: its first operands are asked for here
            const uint32_t prev = prev_live ? ring + at_prev : (uint32_t)kZero;
            uint32_t row[2] = {row_lane[0] + at_next, row_lane[1] + at_next}, col[2] = {col_lane[0] + prev, col_lane[1] + prev};
            asm volatile("" : "+v"(row[0]), "+v"(row[1]), "+v"(col[0]), "+v"(col[1]));
            float pe[16], ds[16];
            if constexpr (kFirst) {
#pragma unroll
                for (int i = 0; i < kAhead; ++i) fr[i] = fetch(i, row, col);
            } else {
                // (the rows of the block after next are those of this sub-step; asked for at the end of the last one)
#pragma unroll
                for (int i = 0; i < kAhead; ++i) fr[i] = i % 2 == 0 ? fr[16 + i] : fetch(i, row, col);
            }
            load_delta(dp[1 - cur], at_next);
            uint32_t row_after[2] = {row_lane[0] + at_after, row_lane[1] + at_after};
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int nxt = i + kAhead;
                if (nxt < 16)
                    fr[nxt] = fetch(nxt, row, col);
                else if (kFirst && nxt % 2 == 0)
                    fr[nxt] = fetch(nxt - 16, row_after, col);
                if (i % 2 == 0) {
                    const int op = i / 2, ks = op % kKS;
                    if (op == 0)
                        mfma_s_first(s[1 - cur], fr[i], kf[0]);
                    else if (op < kKS)
                        mfma_s(s[1 - cur], fr[i], kf[ks]);
                    else
                        mfma_s(dp[1 - cur], fr[i], vf[ks]);
                } else {
                    const int op = i / 2, st = op / 4, db = (op / 2) % 2;
                    mfma_acc(acc[op % 2][db], fr[i], op % 2 == 0 ? pf[1 - cur][st] : dsf[1 - cur][st]);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = first_elem(i); e < first_elem(i + 1); ++e) pe[e] = __builtin_amdgcn_exp2f(fmaf(s[cur][e], c2, nl[e / 4][e % 4]));
                if (i >= 1 && i <= 14) {
#pragma unroll
                    for (int e = first_elem(i - 1); e < first_elem(i); ++e) {
                        ds[e] = pe[e] * dp[cur][e];
                        if (e & 1) {
                            pf[cur][e / 8][e % 8 - 1] = (__bf16)pe[e - 1];
                            pf[cur][e / 8][e % 8] = (__bf16)pe[e];
                            dsf[cur][e / 8][e % 8 - 1] = (__bf16)ds[e - 1];
                            dsf[cur][e / 8][e % 8] = (__bf16)ds[e];
                        }
                        if (e % 8 == 7) {
                            pin_p(pf[cur][e / 8]);
                            pin_p(dsf[cur][e / 8]);
                        }
                        // the next block's lse takes the place of this one's
                        if (e % 4 == 3) nl[e / 4] = lds_f4(lse_lane + at_next + (uint32_t)(32 * (e / 4)));
                    }
                }
                if (i == 2 * kKS - 1) asm volatile("s_nop 1" : "+v"(dp[1 - cur]));  // (what arrived, in front of dP's chain)
                __builtin_amdgcn_sched_barrier(0);
            }
            prev_live = true;
            if (__builtin_expect(!all_visible(i0), 0)) {
                prev_live = any_visible(i0);
                clear_invisible(pf[cur], dsf[cur], prev_live ? visible_rows(i0) : 0u);
            }
            __builtin_amdgcn_sched_barrier(0);
        };

        const int steps = ((total + kParts - 1) / kParts + 1) / 2;  // two blocks of either half of the list
        for (int step = 0; step < steps; ++step) {
            const uint32_t at_1 = next_buf(at_0), at_2 = next_buf(at_1), at_3 = next_buf(at_2), at_4 = next_buf(at_3);
            int row3, row4;
            // (these buffers were last read a step ago, in front of its barrier)
            request_two(at_3, at_4, row3, row4, true);
            substep(std::integral_constant<int, 0>{}, std::true_type{}, row0, at_m1, at_1, at_2);
            substep(std::integral_constant<int, 1>{}, std::false_type{}, row1, at_0, at_2, at_2);
            publish(at_3, at_4);
            barrier();
            at_m1 = at_1;
            at_0 = at_2;
            row0 = row2;
            row1 = row3;
            row2 = row4;
        }
        // ---- dV, dK of the last block ----
        {
            const uint32_t prev = prev_live ? ring + at_m1 : (uint32_t)kZero;
            uint32_t row[2] = {0u, 0u}, col[2] = {col_lane[0] + prev, col_lane[1] + prev};
#pragma unroll
            for (int op = 0; op < 8; ++op) {
                const int st = op / 4, db = (op / 2) % 2;
                mfma_acc(acc[op % 2][db], fetch(2 * op + 1, row, col), op % 2 == 0 ? pf[1][st] : dsf[1][st]);
            }
        }
    }
    asm volatile("s_nop 15\n\ts_nop 7" : "+a"(acc[0][0]), "+a"(acc[0][1]), "+a"(acc[1][0]), "+a"(acc[1][1]));
    __syncthreads();

    // ---- add the halves of the list: the waves of part 1 hand their dK to part 0, which hand over their dV,
    // [4 key blocks][D][32 key columns] floats each ----
    const int keep = part == 0 ? 1 : 0;  // as in acc
    auto xbuf = [&](int which, int d) {
        return (float __attribute__((address_space(3))) *)(uintptr_t)(uint32_t)(which * kSumBytes + ((kq * D + d) * 32 + l32) * 4);
    };
    float mine[kDB][16];
#pragma unroll
    for (int db = 0; db < kDB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int d = 32 * db + 8 * (e / 4) + 4 * hf + (e % 4);
            const float v = acc[0][db][e], k = acc[1][db][e];
            mine[db][e] = keep == 1 ? k : v;
            *xbuf(1 - keep, d) = keep == 1 ? v : k;
        }
    __syncthreads();
    const bool partial = p.parts(kt) > 0;
    float *slot = p.partial + ((size_t)(p.first_part(pair, kt) + (seg >= 0 ? p.n_split + seg : item.piece)) * 2 + (1 - keep)) * (size_t)(128 * D) +
                  (size_t)(32 * kq + l32) * D;
    const size_t out_row = (((size_t)b * p.Hkv + kvh) * (size_t)N + key) * D;
    const float factor = keep == 1 ? p.f.scale : 1.f;
#pragma unroll
    for (int db = 0; db < kDB; ++db)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            const int d = 32 * db + 8 * e4 + 4 * hf;
            float x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = mine[db][4 * e4 + e] + *xbuf(keep, d + e);
            if (partial) {  // fp32 partial sums of all 128 key columns (columns past the end hold zeros)
                *reinterpret_cast<float4 *>(slot + d) = float4{x[0], x[1], x[2], x[3]};
            } else if (key < N) {
                bf16x4 x4;
#pragma unroll
                for (int e = 0; e < 4; ++e) x4[e] = (__bf16)(x[e] * factor);
                *reinterpret_cast<bf16x4 *>((keep == 1 ? p.dk : p.dv) + out_row + d) = x4;
            }
        }
}

}  // namespace
}  // namespace swaa

#endif  // SWAA_BWD_DKV_D64_H_
