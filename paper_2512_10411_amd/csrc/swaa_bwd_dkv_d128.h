// dK and dV, head dimension 128, gfx950 (formulas and mask: swaa_bwd.hip, which includes this file
// and holds the work list).
//
// A workgroup owns 128 keys and walks tiles of 64 query rows; four waves, one per SIMD: wave w owns
// the 64 keys 64 (w % 2).. in two units of 32 and the 32 rows 32 (w / 2).. of every tile; the two row
// halves are added through LDS at the end.  It runs at 1.0 PFLOP/s counted by visible pairs, 72 % of what a large product
// reaches on this card (1.06, 77 %, with the masked and dead products of its edges).  The issue rate of the one wave has the
// rest: 3.7 vector, 1.4 scalar and 1.7 LDS instructions per MFMA, the matrix pipe busy 44 % of the cycles at 2.1 GHz, no bank
// conflicts (16384 tokens, window 2048; profiles/swaa_bwd_mid_bwd_sq_counters.txt).
// Eight waves of 32 keys x 32 rows, two per SIMD, drew 48 KiB of operands from LDS for their 32
// MFMAs and were in the same phase (products, exponentials, products) most of the time; a wave of
// 64 keys draws 72 KiB for 64 MFMAs, because a transposed fragment of Q or dO serves both units and
// the K rows of the first stay in registers, and it has the 512 registers that overlapping the phases by hand
// takes: 256 AccVGPRs hold dK^T and dV^T, 256 VGPRs the rest.
//
// A step (one tile) is four phases of 16 MFMAs with eight exponentials' worth of vector work each,
// interleaved by hand, so that matrix and vector pipe are both busy all the time (s: the tile, 0/1:
// the unit of 32 keys, lo/hi: the rows' half of 16):
//     phase  matrix                                      vector
//     1      S, dP of (s, 1)                             P, dS of (s, 0) hi
//     2      S, dP of (s + 1, 0)                         P, dS of (s, 1) lo
//     3      dV^T += dO^T P, dK^T += Q^T dS, rows lo     P, dS of (s, 1) hi
//     4      the same, rows hi                           P, dS of (s + 1, 0) lo
// Measured, 16384 tokens, 32 heads on 8, window 2048, 512 generated rows: 1.36 ms with eight waves, now 1.27
// (1.15 if no step had an edge: 18 % of them do); 4000 tokens, window 2048: the whole backward 847 -> 807 us.  Short
// sequences and narrow windows stay with the eight waves (swaa_bwd_dkv_d128_short.h, dkv_short).  Asking for operands earlier, or for the tiles in another phase, changes nothing.
// S = Q K^T starts from zero, dP = dO V^T from -delta.  An invisible pair's P and dS are cleared
// after packing, in steps with an edge only (a second version of the step).
//
// Tiles travel HBM -> LDS by global_load_lds_dwordx4 into a ring of three buffers, one barrier per
// step.  One wave alone issues at most an instruction in four cycles, seven per MFMA, so that nothing may
// go into addresses: a tile lies in LDS as four slices of 64 bytes of every row, 16-byte chunk c of the
// four at chunk c ^ ((r >> 2) & 3).  Row fragments and transposed ones are free of bank conflicts, and
// two addresses each reach all of them through the instructions' offset fields.  (256-byte rows with a swizzle over
// all 16 chunks need an address per k-step: 57 vector instructions more per step, and 1.61 ms
// where slices gave 1.47 at the time.)  MFMAs through inline assembly (rules: swaa_tile_d128.h;
// tests/test_asm_hazards.py checks them).  No static LDS: the dynamic LDS starts at address 0.
#ifndef SWAA_BWD_DKV_D128_H_
#define SWAA_BWD_DKV_D128_H_

#include "swaa_bwd.h"
#include "swaa_tile_d128.h"

namespace swaa {
namespace {
namespace dkv128 {

constexpr int kThreads = 256;
constexpr int kRows = 64;                          // query rows per tile
constexpr int kTileBytes = kRows * kRowBytes;      // Q, or dO, of a tile: 16 KiB
constexpr int kBufBytes = 2 * kTileBytes;          // Q, then dO
constexpr int kBufs = 3;
constexpr int kSliceBytes = kRows * 64;            // 64 bytes of every row of a tile: 4 KiB
constexpr int kKeys = kBufs * kBufBytes;           // per key block its 64 V rows and the K rows of its second unit
constexpr int kKeysK = 64 * kRowBytes, kKeysBytes = 96 * kRowBytes;
constexpr int kLse = kKeys + 2 * kKeysBytes;       // per buffer: -lse (log2 units) and -delta of the rows
constexpr int kLseBytes = 2 * kRows * 4;
constexpr int kBytes = kLse + kBufs * kLseBytes;
constexpr int kSlots = 16;                         // MFMAs per phase
constexpr int kAhead = 3, kAheadB = 3;             // MFMAs between an LDS operand read and its use: A, B operands
static_assert(kRows == kBq, "the tiles of the work list");
static_assert(kBufBytes % kLseBytes == 0, "a buffer's offset gives that of its lse");
static_assert(kBytes >= 2 * 128 * kD * 4, "the area doubles as the buffer of the final sums");

// S += / dP += with both operands in VGPRs
__device__ __forceinline__ void mfma_vv(f32x16 &s, const bf16x8 a, const bf16x8 b) {
    asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_vv_first(f32x16 &s, const bf16x8 a, const bf16x8 b) {
    asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(a), "v"(b));
}
// The accumulators of dK^T and dV^T take all 256 AccVGPRs.  They are named in the instructions, not
// held in variables: with no register left over the compiler cannot move a variable of this size
// from one place to another, and two versions of a step ask it to (it put 328 registers on the stack).  Every
// product says that it overwrites all of them, so that nothing else is kept there; tests/test_asm_hazards.py
// checks that nothing is on the stack.
#define SWAA_ACC10(x) "a" #x "0", "a" #x "1", "a" #x "2", "a" #x "3", "a" #x "4", "a" #x "5", "a" #x "6", "a" #x "7", "a" #x "8", "a" #x "9"
#define SWAA_ACC100(x) \
    SWAA_ACC10(x##0), SWAA_ACC10(x##1), SWAA_ACC10(x##2), SWAA_ACC10(x##3), SWAA_ACC10(x##4), SWAA_ACC10(x##5), \
        SWAA_ACC10(x##6), SWAA_ACC10(x##7), SWAA_ACC10(x##8), SWAA_ACC10(x##9)
#define SWAA_ALL_ACC \
    SWAA_ACC10(), SWAA_ACC10(1), SWAA_ACC10(2), SWAA_ACC10(3), SWAA_ACC10(4), SWAA_ACC10(5), SWAA_ACC10(6), SWAA_ACC10(7), \
        SWAA_ACC10(8), SWAA_ACC10(9), SWAA_ACC100(1), SWAA_ACC10(20), SWAA_ACC10(21), SWAA_ACC10(22), SWAA_ACC10(23), \
        SWAA_ACC10(24), "a250", "a251", "a252", "a253", "a254", "a255"
// accumulator block: dV (0) or dK (1), unit, head-dimension block
constexpr int acc_block(int which, int u, int db) { return (which * 2 + u) * kDB + db; }
template <int kBlock>
__device__ __forceinline__ void mfma_acc_at(const bf16x8 a, const bf16x8 b) {
    asm volatile("v_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, a[%2:%3]"
                 :: "v"(a), "v"(b), "n"(16 * kBlock), "n"(16 * kBlock + 15) : SWAA_ALL_ACC);
}
template <int kReg>
__device__ __forceinline__ void acc_clear() {
    asm volatile("v_accvgpr_write_b32 a[%0], 0" :: "n"(kReg) : SWAA_ALL_ACC);
}
template <int kReg>
__device__ __forceinline__ float acc_read() {
    float x;
    asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(x) : "n"(kReg) : "memory");
    return x;
}
// f(0), f(1), .. f(n - 1) with the number as a type
template <int kN, int kI = 0, typename F>
__device__ __forceinline__ void unrolled(const F &f) {
    if constexpr (kI < kN) {
        f(std::integral_constant<int, kI>{});
        unrolled<kN, kI + 1>(f);
    }
}
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 lds_f4(uint32_t addr) { return *(const f32x4 __attribute__((address_space(3))) *)(uintptr_t)addr; }

// The lane's number, asked for anew: what edges and the end of the kernel derive from it takes no
// register during the loop.
__device__ __forceinline__ int lane_now() {
    uint32_t zero;
    asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
    return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
}

// Order of a phase's products S (k-steps 0..7) and dP (8..15 here): the chains take turns, dP
// behind, because its accumulator arrives late and its result is needed last.
constexpr int kOrder[kSlots] = {0, 1, 8, 2, 9, 3, 10, 4, 11, 5, 12, 6, 13, 7, 14, 15};
// Slots of the eight elements of a phase's vector work: exponential in slot 3 k / 2, the rest three slots on.
__device__ constexpr int exp_slot(int k) { return 3 * k / 2; }
__device__ constexpr int rest_slot(int k) { return 3 * k / 2 + 3; }

}  // namespace dkv128

__global__ __launch_bounds__(dkv128::kThreads, 1) void swaa_bwd_dkv_dma_kernel(const BwdParams p) {
    using namespace dkv128;
    const int N = p.N, W = p.f.W, S = p.f.S, P = p.f.P, G = p.f.G;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
    const int kq = wave & 1, qb = wave >> 1;  // key block and row half of this wave
    // (dkv_item and dkv_tiles, written out: called, they left this kernel with more scalar registers moved to vector ones, and
    // 3000 to 4096 tokens with sinks took 1 % longer)
    const int n_kt = (N + 127) / 128;
    const int n_extra = p.B * p.Hkv * p.n_sink_kt * p.n_seg;
    const unsigned bid = blockIdx.x;
    int kt, pair, seg, piece = 0;  // seg: -1 for a key tile's main workgroups
    if ((int)bid < n_extra) {
        const unsigned tile = fastdiv(bid, p.div_seg);
        seg = (int)(bid - tile * (unsigned)p.n_seg);
        pair = (int)fastdiv(tile, p.div_sink_kt);
        kt = (int)tile - pair * p.n_sink_kt;
    } else if (p.n_split > 1) {
        const unsigned id = bid - (unsigned)n_extra, of_pair = fastdiv(id, p.div_pairs);
        seg = -1;
        pair = (int)(id - of_pair * (unsigned)(p.B * p.Hkv));
        kt = (int)fastdiv(of_pair, p.div_split);
        piece = (int)of_pair - kt * p.n_split;
        if (kt >= n_kt) return;
    } else {
        const int id = dkv_main_item(p, bid, n_extra, gridDim.x - (unsigned)n_extra, n_kt);
        if (id >= p.B * p.Hkv * n_kt) return;  // (the grid is rounded up to a multiple of eight)
        seg = -1;
        pair = (int)fastdiv((unsigned)id, p.div_kt);
        kt = id - pair * n_kt;
    }
    const bool sink_kt = kt < p.n_sink_kt;
    const int b = (int)fastdiv((unsigned)pair, p.div_hkv), kvh = pair - b * p.Hkv;
    const int k0 = kt * 128, k1 = min(k0 + 127, N - 1);  // the workgroup's keys
    const int kw0 = k0 + 64 * kq;                         // this wave's first key
    const size_t kv_base = ((size_t)b * p.Hkv + kvh) * (size_t)N * kD;

    // query tiles: the band, then -- if a key is a sink, or there are generated rows -- the rest.  For a
    // sink key tile the rest is cut into segments, and the main workgroup keeps the band.
    const int tq_last = (N - 1) / kRows;
    const int tq_band_hi = min(N - 1, k1 + W - 1) / kRows;
    const int tq_lo = k0 / kRows;
    int n_band = tq_band_hi - tq_lo + 1;
    int tq_x = tq_last + 1, tq_x_end = tq_last;  // second range
    if (sink_kt) {
        if (seg >= 0) {
            n_band = 0;
            tq_x = tq_band_hi + 1 + seg * p.seg_tiles;
            tq_x_end = min(tq_last, tq_x + p.seg_tiles - 1);
        }
    } else if (P < N) {
        tq_x = max(tq_band_hi + 1, P / kRows);
    }
    const int n_tiles = n_band + max(0, tq_x_end - tq_x + 1);
    int total = G * n_tiles, from = 0;  // (head, tile) steps, head-major
    if (p.n_split > 1 && seg < 0) {  // (dkv_piece_start)
        from = (int)fastdiv((unsigned)total * (unsigned)piece, p.div_split);
        total = (int)fastdiv((unsigned)total * (unsigned)(piece + 1), p.div_split) - from;
    }
    auto first_row = [&](int n) { return (n < n_band ? tq_lo + n : tq_x + (n - n_band)) * kRows; };

    unrolled<256>([](auto r) { acc_clear<decltype(r)::value>(); });
    asm volatile("s_nop 1" ::: SWAA_ALL_ACC);

    if (total > 0) {
        // ---- HBM -> LDS copies: one wave instruction moves 64 bytes of 16 rows; the LDS side is linear
        // in the lane id, the swizzle is applied on the global side.  Rows past the end of the sequence
        // repeat its last row (they stay invisible), so that the reads stay in bounds.
        // (a lane's row of the 16, and its place in 64 bytes of that row: f(r) = (r >> 2) & 3)
        const uint32_t lane_row = (uint32_t)(lane >> 2), lane_chunk = (uint32_t)(((lane & 3) ^ (lane >> 4)) << 4);
        auto copy16 = [](uint32_t offset, const __bf16 *base, uint32_t lds, auto lds_more) {
            asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(offset), "s"(base), "s"(lds),
                         "n"(decltype(lds_more)::value)
                         : "memory", "scc");
        };
        // The next tile to ask for: its place in its head's list, its first row, its head's rows, where it
        // begins.  Behind the end of the list the last one is asked for again, into buffers that nobody reads any more.
        int rq_left = total, rq_head = from ? from / n_tiles : 0, rq_n = from - rq_head * n_tiles, rq_row = first_row(rq_n);
        size_t rq_base = ((size_t)b * p.Hq + kvh * G + rq_head) * (size_t)N;
        const __bf16 *rq_q = p.f.q + (rq_base + rq_row) * kD, *rq_do = p.dout + (rq_base + rq_row) * kD;
        float lreg = 0.f, dlreg = 0.f;
        uint32_t rq_off = 0;
        // slice j of rows 16 wave .. of Q and of dO
        auto request_slice = [&](auto slice, uint32_t buf_at) {
            constexpr int j = decltype(slice)::value;
            if (j == 0) rq_off = (uint32_t)min(16 * wave + (int)lane_row, N - 1 - rq_row) * kRowBytes + lane_chunk;
            const uint32_t lds = buf_at + (uint32_t)(wave * 1024);
            copy16(rq_off, rq_q, lds, std::integral_constant<int, j * kSliceBytes>{});
            copy16(rq_off, rq_do, lds, std::integral_constant<int, j * kSliceBytes + kTileBytes>{});
            rq_off += 64;
        };
        auto request_end = [&]() {
            if (wave == 0) {  // (first touched in landed, a step later)
                const size_t row = rq_base + min(rq_row + lane_now(), N - 1);
                lreg = p.f.lse[row];
                dlreg = p.delta[row];
            }
            if (--rq_left > 0) {
                ++rq_n;
                if (rq_n == n_band || rq_n == n_tiles) {  // on to the second range, or to the next head
                    if (rq_n == n_tiles) {
                        rq_n = 0;
                        rq_base += N;
                    }
                    rq_row = first_row(rq_n);
                    rq_q = p.f.q + (rq_base + rq_row) * kD;
                    rq_do = p.dout + (rq_base + rq_row) * kD;
                } else {
                    rq_row += kRows;
                    rq_q += kRows * kD;
                    rq_do += kRows * kD;
                }
            }
        };
        // this wave's copies have landed, and the rows' lse and delta are where everybody finds them
        auto landed = [&](uint32_t buf_at) {
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
            if (wave == 0) {
                float __attribute__((address_space(3))) *at =
                    (float __attribute__((address_space(3))) *)(uintptr_t)(kLse + buf_at / (kBufBytes / kLseBytes) + lane_now() * 4);
                at[0] = lreg * -1.44269504088896340736f;
                at[kRows] = -dlreg;
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
            }
        };
        auto barrier = [&]() {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };

        // V rows 32 wave .., and 16 K rows of a second unit
#pragma unroll
        for (int g = 0; g < 3; ++g) {
            const int first = g < 2 ? 32 * wave + 16 * g : 64 * (wave >> 1) + 32 + 16 * (wave & 1);
            const int at = g < 2 ? (2 * (wave & 1) + g) * 1024 : kKeysK + (wave & 1) * 1024;
            const uint32_t off = (uint32_t)min(first + (int)lane_row, N - 1 - k0) * kRowBytes + lane_chunk;
            unrolled<4>([&](auto slice) {
                constexpr int j = decltype(slice)::value;
                const uint32_t lds = (uint32_t)(kKeys + (wave >> 1) * kKeysBytes + at);
                if (g < 2)
                    copy16(off + 64 * j, p.f.v + kv_base + (size_t)k0 * kD, lds, std::integral_constant<int, j * kSliceBytes>{});
                else
                    copy16(off + 64 * j, p.f.k + kv_base + (size_t)k0 * kD, lds, std::integral_constant<int, j * kSliceBytes / 2>{});
            });
        }
        const int row0 = rq_row;
        unrolled<4>([&](auto j) { request_slice(j, 0u); });
        request_end();
        // the K rows of this wave's first unit as B operands
        bf16x8 kf[kKS];
        {
            const __bf16 *kr = p.f.k + kv_base + (size_t)min(kw0 + l32, N - 1) * kD + 8 * hf;
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks) kf[ks] = *reinterpret_cast<const bf16x8 *>(kr + 16 * ks);
        }
        landed(0u);
        barrier();
        const int row1 = rq_row;
        unrolled<4>([&](auto j) { request_slice(j, (uint32_t)kBufBytes); });
        request_end();

        // ---- per-lane fragment addresses (swizzle folded in); the tile's buffer is part of them, and they
        // move on by one buffer per step
        //  * row fragment, k-step ks: row l32, logical chunk 2 ks + hf: even and odd k-steps
        //  * transposed fragment: rows 4 hf + j16/4 (lo) and 8 further (hi), logical chunk 4 db + 2 (grp & 1) + (j16 & 3) / 2
        uint32_t row_at[2], key_at[2], col_lo, col_hi;
        {
            const uint32_t row_lane = (uint32_t)(l32 * 64 + ((hf ^ ((l32 >> 2) & 3)) << 4));
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                row_at[x] = (uint32_t)(32 * qb * 64) + (row_lane ^ (uint32_t)(x << 5));
                key_at[x] = (uint32_t)(kKeys + kq * kKeysBytes) + (row_lane ^ (uint32_t)(x << 5));
                asm volatile("" : "+v"(row_at[x]), "+v"(key_at[x]));
            }
            const int grp = lane >> 4, j16 = lane & 15;
            const int cl = 2 * (grp & 1) + ((j16 & 3) >> 1);
            // (the last buffer: the first step moves them on to buffer 0)
            const uint32_t at = (uint32_t)((kBufs - 1) * kBufBytes + (32 * qb + 4 * hf + (j16 >> 2)) * 64 + 8 * (j16 & 1));
            col_lo = at + (uint32_t)((cl ^ hf) << 4);
            col_hi = at + (uint32_t)(8 * 64 + ((cl ^ hf ^ 2) << 4));
            asm volatile("" : "+v"(col_lo), "+v"(col_hi));
        }
        uint32_t lse_at = (uint32_t)(kLse + (32 * qb + 4 * hf) * 4);
        const float c2 = p.f.scale_log2;

        f32x16 s[2], dp[2];                 // [unit]
        f32x4 nl[2];                        // -lse of the rows whose exponentials are next
        bf16x8 pf[2][2], dsf[2][2];         // [unit][row half]
        auto load_delta = [&](f32x16 &x, int e4, uint32_t at) {  // rows 8 e4 + 4 hf ..
            const f32x4 t = lds_f4(at + (uint32_t)(32 * e4 + kRows * 4));
#pragma unroll
            for (int i = 0; i < 4; ++i) x[4 * e4 + i] = t[i];
        };
        // in front of the dP chain: if the compiler copies what arrived, then here, not right before a product
        auto settle_delta = [](f32x16 &x) { asm volatile("s_nop 1" : "+v"(x)); };
        // slot i of a phase: rows half st of the next phase's, as this one's are used up
        auto load_lse = [&](int i, int st, uint32_t at) {
            if (i == exp_slot(3) + 1) nl[0] = lds_f4(at + (uint32_t)(64 * st));
            if (i == exp_slot(7) + 1) nl[1] = lds_f4(at + (uint32_t)(64 * st + 32));
        };

        // one slot of a phase's vector work on unit u, row half st
        float pe[8], ds[8];
        auto vector_chunk = [&](int i, int u, int st) {
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (exp_slot(k) == i) pe[k] = __builtin_amdgcn_exp2f(fmaf(s[u][8 * st + k], c2, nl[k / 4][k % 4]));
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (rest_slot(k) == i) {
                    ds[k] = pe[k] * dp[u][8 * st + k];
                    if (k & 1) {
                        pf[u][st][k - 1] = (__bf16)pe[k - 1];
                        pf[u][st][k] = (__bf16)pe[k];
                        dsf[u][st][k - 1] = (__bf16)ds[k - 1];
                        dsf[u][st][k] = (__bf16)ds[k];
                    }
                    if (k == 7) {
                        pin_p(pf[u][st]);
                        pin_p(dsf[u][st]);
                    }
                }
        };
        // Which of the 32 rows from i0 on see this lane's key of unit u?  A bit each, moved so that bit 0 is row 4 hf.
        auto visible_rows = [&](int u, int i0) {
            const int ln = lane_now(), key = kw0 + 32 * u + (ln & 31);
            auto below = [](int t) { return t >= 32 ? ~0u : (1u << min(max(t, 0), 31)) - 1u; };  // bits 0 .. t - 1
            const int end = key < S ? N : min(key + W, N);
            uint32_t m = below(end - i0) & ~below(key - i0);
            if (i0 + 31 >= P) m |= below(N - i0) & ~below(max(key, P) - i0);
            return m >> (4 * (ln >> 5));
        };
        // clears P and dS of the pairs that are not visible
        auto clear_invisible = [&](int u, int st, uint32_t rows) {
            u32x4 pb = __builtin_bit_cast(u32x4, pf[u][st]), db = __builtin_bit_cast(u32x4, dsf[u][st]);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int bit = 16 * st + 8 * (j / 2) + 2 * (j % 2);
                const uint32_t lo = (uint32_t)((int)(rows << (31 - bit)) >> 31), hi = (uint32_t)((int)(rows << (30 - bit)) >> 31);
                const uint32_t keep = (lo & 0xffffu) | (hi & 0xffff0000u);
                pb[j] &= keep;
                db[j] &= keep;
            }
            pf[u][st] = __builtin_bit_cast(bf16x8, pb);
            dsf[u][st] = __builtin_bit_cast(bf16x8, db);
            asm volatile("s_nop 1" : "+v"(pf[u][st]), "+v"(dsf[u][st]));  // (two wait states in front of the MFMAs)
        };
        // of the 32 x 32 pairs of the rows from i0 on and a unit's keys: are all visible, is any?
        auto all_visible = [&](int u, int i0) {
            const int ka = kw0 + 32 * u, kb = ka + 31, i1 = i0 + 31;
            return (kb <= i0) & (i1 < N) & ((i1 - ka < W) | (kb < S) | (i0 >= P));
        };
        auto any_visible = [&](int u, int i0) {
            const int ka = kw0 + 32 * u, kb = ka + 31, i1 = i0 + 31;
            return (ka < N) & (i0 < N) & (i1 >= ka) & ((i0 < kb + W) | (ka < S) | (i1 >= P));
        };

        // LDS operands of the MFMA in slot g of a step (four phases of 16; 64.. are the next step's first)
        bf16x8 fa[4 * kSlots + kAhead], fb[4 * kSlots + kAhead];
        uint32_t row_move = 0, col_move = 0;
        auto fetch = [&](int g) {
            const int ph = (g / kSlots) % 4, i = g % kSlots;
            if (ph < 2) {  // S and dP: row fragments
                const int ks = kOrder[i] % kKS;
                if (ph == 1 && kOrder[i] < 2) {  // on to the next tile
                    row_at[ks] += row_move;
                    asm volatile("" : "+v"(row_at[ks]));
                }
                fa[g] = lds_read16(row_at[ks % 2] + (uint32_t)((ks / 2) * kSliceBytes + (kOrder[i] < kKS ? 0 : kTileBytes)));
            } else if (i % 2 == 0) {  // transposed fragments of dO and Q, each for both units
                const int db = i / 4, st = ph - 2;
                const bool of_do = (i / 2) % 2 == 0;
                if (ph == 2 && i == 0) {
                    col_lo += col_move;
                    col_hi += col_move;
                    asm volatile("" : "+v"(col_lo), "+v"(col_hi));
                }
                const uint32_t off = (uint32_t)((of_do ? kTileBytes : 0) + db * kSliceBytes + 16 * st * 64);
                const s16x4 lo = lds_read8_tr(col_lo + off), hi = lds_read8_tr(col_hi + off);
                fa[g] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        };
        auto fetch_b = [&](int g) {
            const int ph = (g / kSlots) % 4, i = g % kSlots;
            if (ph >= 2 || (ph == 1 && kOrder[i] < kKS)) return;
            const int ks = kOrder[i] % kKS;
            const int off = kOrder[i] < kKS ? kKeysK + (ks / 2) * kSliceBytes / 2 : (ks / 2) * kSliceBytes + (ph == 0 ? 1 : 0) * 32 * 64;
            fb[g] = lds_read16(key_at[ks % 2] + (uint32_t)off);
        };
        auto product = [&](int g, int u) {  // phases 1 and 2
            const int op = kOrder[g % kSlots], ks = op % kKS;
            if (op == 0)
                mfma_vv_first(s[u], fa[g], u ? fb[g] : kf[0]);
            else if (op < kKS)
                mfma_vv(s[u], fa[g], u ? fb[g] : kf[ks]);
            else
                mfma_vv(dp[u], fa[g], fb[g]);
        };

        // ---- prologue: S and dP of (0, 0), P and dS of its lower rows ----
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            load_delta(dp[0], e4, lse_at);
            asm volatile("" : "+v"(lse_at));
            load_delta(dp[1], e4, lse_at);
        }
        asm volatile("s_nop 1" : "+v"(dp[0]), "+v"(dp[1]));  // (no copy of theirs right in front of a product)
        nl[0] = lds_f4(lse_at);
        nl[1] = lds_f4(lse_at + 32);
        // this wave's first row of the tile, the next one, the one after it
        int i0 = row0 + 32 * qb, i0n = row1 + 32 * qb;
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) {
            const uint32_t slice = (uint32_t)((ks / 2) * kSliceBytes);
            const bf16x8 qfrag = lds_read16(row_at[ks % 2] + slice), dofrag = lds_read16(row_at[ks % 2] + slice + kTileBytes),
                         vfrag = lds_read16(key_at[ks % 2] + slice);
            if (ks == 0)
                mfma_vv_first(s[0], qfrag, kf[0]);
            else
                mfma_vv(s[0], qfrag, kf[ks]);
            mfma_vv(dp[0], dofrag, vfrag);
        }
        asm volatile("s_nop 15\n\ts_nop 7" : "+v"(s[0]), "+v"(dp[0]));
#pragma unroll
        for (int i = 0; i < kSlots; ++i) {
            vector_chunk(i, 0, 0);
            load_lse(i, 1, lse_at);
        }
        if (!all_visible(0, i0)) clear_invisible(0, 0, visible_rows(0, i0));
        asm volatile("s_nop 1" : "+v"(pf[0][0]), "+v"(dsf[0][0]));
#pragma unroll
        for (int g = 0; g < kAhead; ++g) {
            fetch(g);
            if (g < kAheadB) fetch_b(g);
        }

        uint32_t at_prev = (kBufs - 1) * kBufBytes, at = 0, at_next = kBufBytes;  // the buffers of the tiles around this step
        auto step = [&](auto with_edge, bool more) {
            constexpr bool kEdge = decltype(with_edge)::value;  // not all of the step's pairs are visible
            row_move = at_next - at;
            col_move = at - at_prev;
            const uint32_t lse_move = (uint32_t)((int)row_move / (kBufBytes / kLseBytes));
            uint32_t lse_next = lse_at + lse_move;
            asm volatile("" : "+v"(lse_next));
            bool live[2] = {true, true};  // does the unit see any of the rows?
            if constexpr (kEdge) {
                live[0] = any_visible(0, i0);
                live[1] = any_visible(1, i0);
            }
            // phase 1: S, dP of (this, 1); P, dS of (this, 0) hi
            unrolled<kSlots>([&](auto slot) {
                constexpr int i = decltype(slot)::value;
                fetch(i + kAhead);
                fetch_b(i + kAheadB);
                product(i, 1);
                __builtin_amdgcn_sched_barrier(0);
                vector_chunk(i, 0, 1);
                if (i == 1) {
                    // the next tile has landed; the buffer of the one after it was last read a step ago
                    if (more) landed(at_next);
                    barrier();
                }
                load_lse(i, 0, lse_at);
                if (i == 1) settle_delta(dp[1]);
                if (i == 4) load_delta(dp[0], 0, lse_next);
                if (i == 6) load_delta(dp[0], 1, lse_next);
                if (i == rest_slot(3) + 1) load_delta(dp[0], 2, lse_next);
                if (i == rest_slot(7)) load_delta(dp[0], 3, lse_next);
                if constexpr (i == 5 || i == 11) request_slice(std::integral_constant<int, i / 8>{}, at_prev);
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (kEdge)
                if (live[0] && !all_visible(0, i0)) clear_invisible(0, 1, visible_rows(0, i0));
            __builtin_amdgcn_sched_barrier(0);
            // phase 2: S, dP of (next, 0); P, dS of (this, 1) lo
            unrolled<kSlots>([&](auto slot) {
                constexpr int i = decltype(slot)::value;
                fetch(kSlots + i + kAhead);
                fetch_b(kSlots + i + kAheadB);
                product(kSlots + i, 0);
                __builtin_amdgcn_sched_barrier(0);
                vector_chunk(i, 1, 0);
                load_lse(i, 1, lse_at);
                if (i == 1) settle_delta(dp[0]);
                if constexpr (i == 5 || i == 11) request_slice(std::integral_constant<int, 2 + i / 8>{}, at_prev);
                __builtin_amdgcn_sched_barrier(0);
            });
            const int row2 = rq_row;
            request_end();
            if constexpr (kEdge)
                if (live[1] && !all_visible(1, i0)) clear_invisible(1, 0, visible_rows(1, i0));
            __builtin_amdgcn_sched_barrier(0);
            lse_at = lse_next;
            // phases 3 and 4: dV^T, dK^T; P, dS of (this, 1) hi and of (next, 0) lo.  A unit that sees none of the
            // rows takes nothing from them, whatever they hold.
            auto sums = [&](auto half, auto live0, auto live1) {
                constexpr int st = decltype(half)::value;
                unrolled<kSlots>([&](auto slot) {
                    constexpr int i = decltype(slot)::value, db = i / 4, u = i % 2;
                    const int g = (2 + st) * kSlots + i;
                    fetch(g + kAhead);
                    fetch_b(g + kAheadB);
                    if constexpr (u == 0 ? decltype(live0)::value : decltype(live1)::value) {
                        if constexpr ((i / 2) % 2 == 0)
                            mfma_acc_at<acc_block(0, u, db)>(fa[g - u], pf[u][st]);
                        else
                            mfma_acc_at<acc_block(1, u, db)>(fa[g - u], dsf[u][st]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    vector_chunk(i, 1 - st, 1 - st);
                    load_lse(i, st, lse_at);
                    if (st == 1 && i < 8 && i % 2 == 0) load_delta(dp[1], i / 2, lse_at);
                    __builtin_amdgcn_sched_barrier(0);
                });
            };
            auto sums_of_live = [&](auto half) {
                if (!kEdge || (live[0] && live[1]))
                    sums(half, std::true_type{}, std::true_type{});
                else if constexpr (kEdge) {
                    if (live[0])
                        sums(half, std::true_type{}, std::false_type{});
                    else if (live[1])
                        sums(half, std::false_type{}, std::true_type{});
                    else
                        sums(half, std::false_type{}, std::false_type{});
                }
            };
            sums_of_live(std::integral_constant<int, 0>{});
            if constexpr (kEdge)
                if (live[1] && !all_visible(1, i0)) clear_invisible(1, 1, visible_rows(1, i0));
            __builtin_amdgcn_sched_barrier(0);
            sums_of_live(std::integral_constant<int, 1>{});
            if constexpr (kEdge)
                if (!all_visible(0, i0n)) clear_invisible(0, 0, visible_rows(0, i0n));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < kAhead; ++g) {
                fa[g] = fa[4 * kSlots + g];
                if (g < kAheadB) fb[g] = fb[4 * kSlots + g];
            }
            i0 = i0n;
            i0n = row2 + 32 * qb;
            at_prev = at;
            at = at_next;
            at_next = at_next == (kBufs - 1) * kBufBytes ? 0 : at_next + kBufBytes;
        };
        // All pairs of both units are visible, in one comparison per bound (if the window's end or the sinks' lies between the
        // units, the answer is no).
        const int lean_from = kw0 + 63, lean_to = min(N - 32, kw0 + 63 < S ? N : kw0 + W - 32);
        auto lean = [&](int first) { return first >= lean_from && (first <= lean_to || (first >= P && first + 31 < N)); };
        // (Steps without an edge loop among themselves: where the two versions of the step meet, what they keep in different
        // registers is moved, 59 instructions that every step paid.  The whole backward, 16384 tokens, 32 heads on 8, window
        // 2048, 512 generated rows: 2182 -> 2140 us; 8192 tokens, full attention: 1720 -> 1662.)
        int left = total;
        bool lean_now = lean(i0);
        while (left > 0) {
            if (lean_now && lean(i0n)) {
                do {
                    step(std::false_type{}, left > 1);
                    --left;
                } while (left > 0 && lean(i0n));  // (behind the last tile: never used)
            } else {
                step(std::true_type{}, left > 1);
                --left;
                lean_now = lean(i0);
            }
        }
    }

    // ---- add the two row halves through LDS, [2 key blocks][D][64 keys] floats of dK, then of dV: the waves of
    // rows 32.. hand over dK and keep dV, the others the other way round ----
    asm volatile("s_nop 15\n\ts_nop 7" ::: "memory", SWAA_ALL_ACC);  // (the last MFMAs have no MFMA behind them)
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the copies asked for last
    const int keep = qb == 0 ? 1 : 0;  // as in acc_block
    const int ln = lane_now(), col32 = ln & 31, row4 = 4 * (ln >> 5);
    const uint32_t lane_at = (uint32_t)((kq * kD * 64 + col32) * 4);
    const uint32_t take = (uint32_t)(keep * 128 * kD * 4) + lane_at;
    float mine[2][kDB][16];
    // this wave's sums of `which` to registers, of the other to LDS
    auto hand_over = [&](auto which) {
        constexpr int kWhich = decltype(which)::value;
        const uint32_t give = (uint32_t)((1 - kWhich) * 128 * kD * 4) + lane_at;
        unrolled<2 * kDB * 16>([&](auto r) {
            constexpr int x = decltype(r)::value, u = x / (16 * kDB), db = x / 16 % kDB, e = x % 16;
            const int d = 32 * db + 8 * (e / 4) + row4 + (e % 4);
            *(float __attribute__((address_space(3))) *)(uintptr_t)(give + (uint32_t)((d * 64 + 32 * u) * 4)) =
                acc_read<16 * acc_block(1 - kWhich, u, db) + e>();
            mine[u][db][e] = acc_read<16 * acc_block(kWhich, u, db) + e>();
        });
    };
    __syncthreads();
    if (keep == 1)
        hand_over(std::integral_constant<int, 1>{});
    else
        hand_over(std::integral_constant<int, 0>{});
    __syncthreads();
    const bool partial = p.parts(kt) > 0;
    float *slot = p.partial + ((size_t)(p.first_part(pair, kt) + (seg >= 0 ? p.n_split + seg : piece)) * 2 + (1 - keep)) * (size_t)(128 * kD);
    const float factor = keep == 1 ? p.f.scale : 1.f;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int col = 64 * kq + 32 * u + col32, key = k0 + col;
#pragma unroll
        for (int db = 0; db < kDB; ++db)
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
                const int d = 32 * db + 8 * e4 + row4;
                float x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    x[e] = mine[u][db][4 * e4 + e] +
                           *(const float __attribute__((address_space(3))) *)(uintptr_t)(take + (uint32_t)(((d + e) * 64 + 32 * u) * 4));
                if (partial) {  // fp32 partial sums of all 128 key columns (columns past the end hold zeros)
                    const float4 x4 = {x[0], x[1], x[2], x[3]};
                    *reinterpret_cast<float4 *>(slot + (size_t)col * kD + d) = x4;
                } else if (key < N) {
                    bf16x4 x4;
#pragma unroll
                    for (int e = 0; e < 4; ++e) x4[e] = (__bf16)(x[e] * factor);
                    *reinterpret_cast<bf16x4 *>((keep == 1 ? p.dk : p.dv) + kv_base + (size_t)key * kD + d) = x4;
                }
            }
    }
}

}  // namespace
}  // namespace swaa

#endif  // SWAA_BWD_DKV_D128_H_
