// dK and dV, head dimension 128, where a key tile is seen by few query tiles: short sequences and narrow
// windows (dkv_short in swaa_bwd.hip, which includes this file and holds the work list).
//
// Eight waves, two per SIMD (one wave's exponentials overlap the other's MFMAs): wave w owns
// the 32 keys 32*(w%4).. of the workgroup's 128 and the 32 rows 32*(w/4).. of every 64-row
// query tile; the two row halves are added through LDS at the end.  A block of 32 rows x 32 keys without a
// visible pair costs nothing, where the kernel of one wave per SIMD (swaa_bwd_dkv_d128.h) forms S and dP of it all the
// same, and there is little to do before the first tile and after the last (64 tokens, 32 heads on 8: 12.3 us, 17.3 the other; 16384
// tokens on a window of 128: 195 us, 213; measured on both sides of the line in dkv_short).
// K, V (once per workgroup) and the query
// tile's Q and dO (per step, two buffers each) travel HBM -> LDS with global_load_lds_dwordx4,
// no register staging and no store phase: one barrier per step.  Rows are 256
// bytes without padding; 16-byte chunk c of row r lies at chunk c ^ g(r), g(r) = ((r & 3) << 2)
// | ((r >> 2) & 3), applied on the global side of the copy.  That one layout serves both read
// patterns without bank conflicts: 16 consecutive rows reading the same logical chunk
// (ds_read_b128 row fragments: g takes 16 different values) and 4 consecutive rows reading the
// same 64 bytes (ds_read_b64_tr_b16 transposed fragments: the upper two bits of g differ).
// This kernel declares no static LDS: its dynamic LDS starts at address 0 and all LDS accesses
// below use plain byte addresses.
#ifndef SWAA_BWD_DKV_D128_SHORT_H_
#define SWAA_BWD_DKV_D128_SHORT_H_

#include "swaa_bwd.h"
#include "swaa_tile_d128.h"

namespace swaa {
namespace {
namespace dkv128short {

constexpr int kThreads = 512;
constexpr int kAhead = 2;  // MFMAs between an LDS operand read and its use
constexpr int kKeyTileBytes = 128 * kRowBytes;  // 32 KiB: the workgroup's K rows, or V rows
constexpr int kQTileBytes = kBq * kRowBytes;    // 16 KiB
constexpr int kK = 0, kV = kKeyTileBytes, kQ = 2 * kKeyTileBytes, kDO = kQ + 2 * kQTileBytes, kL = kDO + 2 * kQTileBytes,
              kDl = kL + 2 * kBq * 4, kBytes = kDl + 2 * kBq * 4;
static_assert(2 * kKeyTileBytes >= 4 * 32 * kD * 4, "the K/V area doubles as the buffer of the final sum");

}  // namespace dkv128short

__global__ __launch_bounds__(dkv128short::kThreads, 1) void swaa_bwd_dkv_dma_short_kernel(const BwdParams p) {
    using namespace dkv128short;
    constexpr int D = kD, KS = kKS, DB = kDB;

    const int N = p.N, W = p.f.W, S = p.f.S, P = p.f.P, G = p.f.G;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
    const int kq = wave & 3, qb = wave >> 2;  // key block and row half of this wave
    DkvItem item;
    if (!dkv_item(p, item)) return;
    const int kt = item.kt, pair = item.pair, seg = item.seg;
    const int b = (int)fastdiv((unsigned)pair, p.div_hkv), kvh = pair - b * p.Hkv;
    const int k0 = kt * 128;                             // the workgroup's first key
    const int kw0 = k0 + 32 * kq, kw1 = kw0 + 31;         // this wave's keys
    const int key = kw0 + l32;                            // this lane's key column
    const bool wave_active = kw0 < N;

    // ---- HBM -> LDS copies: one wave instruction moves 64 x 16 bytes = 4 rows; the LDS side
    // is linear in the lane id, LDS address = M0 + 16 * lane.  Rows past the end of the
    // sequence repeat its last row (they stay invisible), so that the reads stay in bounds.
    const int lrow = lane >> 4, lchk = lane & 15;
    auto copy16 = [](const char *g, uint32_t lds) {
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(lds) : "memory");
    };
    // rows [4 ii, 4 ii + 4) of a tile whose first row is row `first` of a [N][D] matrix
    auto copy_rows = [&](const __bf16 *mat, int first, int ii, uint32_t tile) {
        const int r = 4 * ii + lrow;
        const int g = (lrow << 2) | (ii & 3);  // g(r): r & 3 = lrow, (r >> 2) & 3 = ii & 3
        const char *src = reinterpret_cast<const char *>(mat + (size_t)min(first + r, N - 1) * D) + ((lchk ^ g) << 4);
        copy16(src, tile + (uint32_t)(ii * 1024));
    };
    {
        const size_t kv_base = ((size_t)b * p.Hkv + kvh) * (size_t)N * D;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            copy_rows(p.f.k + kv_base, k0, 4 * wave + i, kK);
            copy_rows(p.f.v + kv_base, k0, 4 * wave + i, kV);
        }
    }
    f32x16 dkacc[DB], dvacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            dkacc[db][e] = 0.f;
            dvacc[db][e] = 0.f;
        }

    const DkvTiles tiles = dkv_tiles(p, item);
    const int n_tiles = tiles.n;
    const int from = dkv_piece_start(p, item, G * n_tiles, 0);  // this workgroup's (head, tile) steps, head-major
    const int total = dkv_piece_start(p, item, G * n_tiles, 1) - from;

    const float c2 = p.f.scale_log2;
    float lreg = 0.f, dlreg = 0.f;
    // the next step = (head, query tile) to ask for, its head's rows, and the step being computed.  (Counted
    // on: with a division and a remainder for both in every step the backward of four sequences of 2048 tokens on a window of
    // 128, 16 heads on 4, took 149 us, 146 now; 32 heads on 8, 4001 tokens, 144 and 141.)
    const int first_head = from ? from / n_tiles : 0;
    int rq_n = from - first_head * n_tiles, at_n = rq_n;
    size_t base = ((size_t)b * p.Hq + kvh * G + first_head) * (size_t)N;
    // its Q and dO rows into buffer `buf`, its lse and delta into registers
    auto request_tile = [&](int buf) {
        const int tq = tiles.at(rq_n);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            copy_rows(p.f.q + base * D, tq * kBq, 2 * wave + i, (uint32_t)(kQ + buf * kQTileBytes));
            copy_rows(p.dout + base * D, tq * kBq, 2 * wave + i, (uint32_t)(kDO + buf * kQTileBytes));
        }
        // (asked for here, first touched in publish_rows at the end of the step: any arithmetic on
        // them right away would make this wave wait for the loads, and with them for the copies above)
        if (tid < kBq) {
            const int row = min(tq * kBq + tid, N - 1);
            lreg = p.f.lse[base + row];
            dlreg = p.delta[base + row];
        }
        if (++rq_n == n_tiles) {
            rq_n = 0;
            base += N;
        }
    };
    auto publish_rows = [&](int buf) {
        if (tid < kBq) {
            *(float __attribute__((address_space(3))) *)(uintptr_t)(kL + buf * kBq * 4 + tid * 4) = lreg * 1.44269504088896340736f;
            *(float __attribute__((address_space(3))) *)(uintptr_t)(kDl + buf * kBq * 4 + tid * 4) = dlreg;
        }
    };

    // per-lane fragment addresses inside a tile (swizzle folded in)
    //  * row fragment, k-step ks: row 32 rb + l32, logical chunk 2 ks + hf:  row_lane ^ (ks << 5), + 32 rb rows
    //  * transposed fragment, 16-row step st, head-dimension block db: rows 32 rb + 16 st + 4 hf + j16/4 (lo)
    //    and 8 further (hi), logical chunk 4 db + 2 (grp & 1) + (j16 & 3) / 2:  col_lane ^ (db << 6), + rows
    const int gl = ((l32 & 3) << 2) | ((l32 >> 2) & 3);
    const uint32_t row_lane = (uint32_t)(l32 * kRowBytes + ((hf ^ gl) << 4));
    const int grp = lane >> 4, j16 = lane & 15;
    const int rr = 4 * hf + (j16 >> 2);
    const int cl = 2 * (grp & 1) + ((j16 & 3) >> 1);
    const uint32_t col_lo = (uint32_t)(rr * kRowBytes + ((((rr & 3) << 2) | (cl ^ hf)) << 4) + 8 * (j16 & 1));
    const uint32_t col_hi = (uint32_t)((rr + 8) * kRowBytes + ((((rr & 3) << 2) | (cl ^ (hf + 2))) << 4) + 8 * (j16 & 1));
    auto row_frag_at = [&](uint32_t tile, int rb, int ks) {
        return lds16(tile + (uint32_t)(32 * rb * kRowBytes) + (row_lane ^ (uint32_t)(ks << 5)));
    };
    auto col_frag_at = [&](uint32_t tile, int rb, int st, int db) {
        const uint32_t off = tile + (uint32_t)((32 * rb + 16 * st) * kRowBytes);
        const s16x4 lo = lds8_tr(off + (col_lo ^ (uint32_t)(db << 6)));
        const s16x4 hi = lds8_tr(off + (col_hi ^ (uint32_t)(db << 6)));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    if (total > 0) {
        request_tile(0);
        publish_rows(0);
    }
    __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0): this wave's copies have landed
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    for (int step = 0; step < total; ++step) {
        const int buf = step & 1;
        const bool has_next = step + 1 < total;
        // the other buffers were last read one step ago, before the barrier that ended it
        if (has_next) request_tile(buf ^ 1);

        const uint32_t Qs = (uint32_t)(kQ + buf * kQTileBytes), dOs = (uint32_t)(kDO + buf * kQTileBytes);
        const int tq = tiles.at(at_n);
        if (++at_n == n_tiles) at_n = 0;
        const int i0 = tq * kBq + 32 * qb, i1 = i0 + 31;  // this wave's rows of the tile
        // can any of them see any key of this wave?
        const bool sees = (i0 < N) && (i1 >= kw0) && ((i0 < kw1 + W) || (kw0 < S) || (i1 >= P));
        if (wave_active && sees) {
            // all 32 x 32 pairs visible: rows at or below the keys' diagonal, inside every row's window
            // (or the keys are sinks, or the rows are generated tokens), and no row past the end
            const bool unmasked = (kw1 <= i0) && (i1 < N) && ((i1 - kw0 < W) || (kw1 < S) || (i0 >= P));

            // S = Q K^T and dP = dO V^T : [32 queries] x [32 keys]
            f32x16 sacc, dpacc;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                sacc[e] = 0.f;
                dpacc[e] = 0.f;
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row_frag_at(Qs, qb, ks), row_frag_at(kK, kq, ks), sacc, 0, 0, 0);
                dpacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row_frag_at(dOs, qb, ks), row_frag_at(kV, kq, ks), dpacc, 0, 0, 0);
            }
            // operand reads run kAhead MFMAs ahead of their use (two reads per MFMA)
            __builtin_amdgcn_sched_group_barrier(0x100, 2 * kAhead, 0);
#pragma unroll
            for (int i = 0; i < 2 * KS; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            }

            // P and dS in the accumulator layout (row 8 (e/4) + 4 hf + e%4, column = this lane's key)
            bf16x8 pf[2], dsf[2];  // [16-row step]
            // (one uniform branch per tile, none per element: a bit for each of the 32 rows that sees this lane's key)
            auto softmax_stage = [&](auto masked) {
                const int i32 = tq * kBq + 32 * qb;
                const uint32_t rows = !decltype(masked)::value ? 0u
                                      : (keys_below(N - i32) & ~keys_below(key - i32) &
                                         (keys_below(key < S ? 32 : key + W - i32) | ~keys_below(P - i32))) >> (4 * hf);
#pragma unroll
                for (int e4 = 0; e4 < 4; ++e4) {
                    const int r4 = 32 * qb + 8 * e4 + 4 * hf;
                    typedef float f32x4 __attribute__((ext_vector_type(4)));
                    const f32x4 l4 = *(const f32x4 __attribute__((address_space(3))) *)(uintptr_t)(kL + buf * kBq * 4 + r4 * 4);
                    const f32x4 d4 = *(const f32x4 __attribute__((address_space(3))) *)(uintptr_t)(kDl + buf * kBq * 4 + r4 * 4);
                    const float lv[4] = {l4[0], l4[1], l4[2], l4[3]};
                    const float dv4[4] = {d4[0], d4[1], d4[2], d4[3]};
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const int e = 4 * e4 + x;
                        float pe = __builtin_amdgcn_exp2f(fmaf(sacc[e], c2, -lv[x]));
                        if (decltype(masked)::value)
                            pe = __uint_as_float((uint32_t)((int)(rows << (31 - (8 * e4 + x))) >> 31) & __float_as_uint(pe));
                        pf[e / 8][e % 8] = (__bf16)pe;
                        dsf[e / 8][e % 8] = (__bf16)(pe * (dpacc[e] - dv4[x]));
                    }
                }
            };
            if (unmasked)
                softmax_stage(std::false_type{});
            else
                softmax_stage(std::true_type{});

            // dV^T += dO^T P,  dK^T += Q^T dS
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    dvacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(col_frag_at(dOs, qb, st, db), pf[st], dvacc[db], 0, 0, 0);
                    dkacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(col_frag_at(Qs, qb, st, db), dsf[st], dkacc[db], 0, 0, 0);
                }
            __builtin_amdgcn_sched_group_barrier(0x100, 2 * kAhead, 1);
#pragma unroll
            for (int i = 0; i < 4 * DB; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 1);
            }
        }

        if (has_next) publish_rows(buf ^ 1);
        // the next tile has landed (this wave's part, then everybody's), this one is free afterwards
        __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }

    // ---- add the two row halves: waves 4..7 hand their sums to waves 0..3 through LDS
    // (the K/V area, which nobody reads any more), first dK, then dV ----
    // [4 key blocks][D][32 key columns] floats from LDS address 0
#pragma unroll
    for (int which = 0; which < 2; ++which) {
        if (which) __syncthreads();
        if (qb == 1) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int d = 32 * db + 8 * (e / 4) + 4 * hf + (e % 4);
                    *(float __attribute__((address_space(3))) *)(uintptr_t)(((kq * D + d) * 32 + l32) * 4) =
                        which == 0 ? dkacc[db][e] : dvacc[db][e];
                }
        }
        __syncthreads();
        if (qb == 0) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int d = 32 * db + 8 * (e / 4) + 4 * hf + (e % 4);
                    const float other = *(const float __attribute__((address_space(3))) *)(uintptr_t)(((kq * D + d) * 32 + l32) * 4);
                    if (which == 0)
                        dkacc[db][e] += other;
                    else
                        dvacc[db][e] += other;
                }
        }
    }
    if (qb != 0) return;

    if (p.parts(kt) > 0) {
        // fp32 partial sums of all 128 key columns (columns past the end hold zeros)
        float *slot = p.partial + (size_t)(p.first_part(pair, kt) + (seg >= 0 ? p.n_split + seg : item.piece)) * (2 * 128 * D);
        float *pk = slot + (size_t)(32 * kq + l32) * D, *pv = pk + 128 * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
                const float4 k4 = {dkacc[db][4 * e4], dkacc[db][4 * e4 + 1], dkacc[db][4 * e4 + 2], dkacc[db][4 * e4 + 3]};
                const float4 v4 = {dvacc[db][4 * e4], dvacc[db][4 * e4 + 1], dvacc[db][4 * e4 + 2], dvacc[db][4 * e4 + 3]};
                *reinterpret_cast<float4 *>(pk + 32 * db + 8 * e4 + 4 * hf) = k4;
                *reinterpret_cast<float4 *>(pv + 32 * db + 8 * e4 + 4 * hf) = v4;
            }
    } else if (key < N) {
        const size_t row = (((size_t)b * p.Hkv + kvh) * (size_t)N + key) * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
                bf16x4 k4, v4;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    k4[e] = (__bf16)(dkacc[db][4 * e4 + e] * p.f.scale);
                    v4[e] = (__bf16)dvacc[db][4 * e4 + e];
                }
                *reinterpret_cast<bf16x4 *>(p.dk + row + 32 * db + 8 * e4 + 4 * hf) = k4;
                *reinterpret_cast<bf16x4 *>(p.dv + row + 32 * db + 8 * e4 + 4 * hf) = v4;
            }
    }
}

}  // namespace
}  // namespace swaa

#endif  // SWAA_BWD_DKV_D128_SHORT_H_
