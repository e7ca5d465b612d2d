// fp32 products of the paper's first listing (Section 2) on the bf16 matrix
// cores, any operand layout with 16-byte aligned rows.  Each operand value is
// the sum of three bf16 terms (split3_pair in common.hpp) and a product eight of
// the nine bf16 products, all but ll (2^-32 of the product): eight MFMAs of 1024
// FLOP per cycle and SIMD for one of 64, so twice the fp32 matrix rate.  The terms
// are formed in registers, from fp32 tiles in LDS: nothing but the operands is
// read from memory and no copy of the terms is written.
//
// Eight and not six: without ml and lm a product is off by up to 2^-24 of itself
// before the result is rounded, so a sum that holds one non-zero product (a
// diagonal scaling, a selection) is off by up to 1.68 half units in the last place
// and 4 % of such results are not the nearest; with them 1.004 and 0.15 % (the fp32
// instructions: 1 and none).  They cost a tenth of the time (2048x1024x1024 32.9 ->
// 35.9 us, 1536x1536x1536 63.5 -> 67, 2048x4096x4096 379 -> 430).
//
// What bounds it: forming the terms takes 13 vector instructions per two
// values, 52 per MFMA operand block, so a wave of 2 x 2 blocks issues about 230
// vector instructions (920 cycles) for 32 MFMAs (1024 cycles): the two have to
// run side by side.  So:
//   * a wave owns 64 x 64 of the tile and one 16-deep step of each K tile; the
//     other waves on its SIMD take other K steps of the same block (WK), so no
//     value is split more often than the 2 x 2 block needs, and their MFMAs
//     fill each other's gaps.  The WK sums are added through LDS at the end;
//   * of the four operand blocks of a step one is split while the eight MFMAs of
//     a block pair run: (A0,B0) with A1, (A1,B0) with B1, (A0,B1) with B0 of
//     the next K tile, (A1,B1) with A0 of the next.  Four split blocks are live
//     at a time, as many as one step needs;
//   * the seven small products have an accumulator of their own, added at the end:
//     a result is rounded once per 16 values of K at its full size, where the
//     fp32 matrix instructions round at least 8 times, so the error against
//     64 bits is smaller than theirs (2048x1024x1024: 9.8e-8 of the result's norm
//     against 5.7e-7, 512x512x4096 1.1e-7 against 5.7e-7).
// Per call, fp32, us (this kernel / the fp32 tile kernel): 2048x1024x1024 NT 38 /
// 48, 1536x768x3072 TN 64 / 145, 1536x1536x1536 TN 69 / 123, 1000^3 25 / 34,
// 512x512x4096 29 / 36, 4096x512x512 22.5 / 27.4, 8192x256x256 15.9 / 15.6.  With the whole
// chip busy it runs at 1.25 PFLOP/s of bf16 products, the rate at which random
// values are held by power.  Terms by masks instead of conversions cost the same
// time and, truncated, more error.
// The copies into an LDS ring and the K slices summed by the last arrival are
// those of the bf16 kernel (gemm_ring.hpp).  K tiles are 32 deep per sub-block
// (a K-contiguous row is one 128-byte line, as 64 bf16 values are there); rows
// along M or N are read one value per lane, rows k and k + 8 (the two halves of
// a wave) 32 banks apart.
//
// Range: the operands are scaled by 2^24 while they are split, so the terms of every
// value down to the smallest denormal (2^-149) are normal bf16 numbers and exact,
// whatever stands beside it in its row; unscaled, a value below about 2^-109 loses
// its low terms, and 2^-120 times 2^27 came out with 14 good bits.  The sums are
// scaled back by 2^-48 at the end; products of values below 2^28 stay under 2^104
// scaled, so 2^23 of them can be added.  The scaling costs two of the 13 vector
// instructions per pair (2048x1024x1024 36.2 -> 37.6 us, 1536x1536x1536 66 -> 68).  A value of
// 2^28 or more (an infinity among them) is not split: a wave that reads one scales
// its sums back and goes on with fp32 matrix instructions for the rest of its K
// steps, on the same LDS tiles and barriers, so such values cost at most what they
// cost the fp32 tile kernel.  A whole column of 1e30, us (first K tile / last /
// none / tile kernel): 2048x1024x1024 45 / 39 / 39 / 46, 1536x1536x1536 88 / 70 / 71 / 124,
// 512x512x4096 32 / 29 / 29 / 37; forming the tile again afterwards took 245, 750 and 220.
// The check needs the tile's fp32 blocks in registers before its first MFMA; it
// stands at the end of the loop so that the loop has one exit (a second one made
// the compiler copy and spill accumulators: 81 us for 39).
#pragma once

#include "gemm_ring.hpp"

namespace isam {

constexpr float kF32xScale = 0x1p24f;     // on both operands while they are split
constexpr float kF32xUnscale = 0x1p-48f;  // on the sums
constexpr float kF32xLimit = 0x1p28f;     // values from here on take the fp32 instructions

// One fp32 operand of a workgroup's tile: ROWS values of M / N x 32 SUB of K.
template <int ROWS, bool KC, int NW, int SUB>
struct F32xOperand {
    static constexpr int SUB_BYTES = ROWS * 128, BYTES = SUB_BYTES * SUB;
    static constexpr int INSTR = BYTES / 1024 / NW;  // copies per wave and K tile
    static_assert(INSTR >= 1 && INSTR * NW * 1024 == BYTES, "whole copies per wave");
    static_assert(ROWS % 64 == 0, "bank swizzle");
    __amdgpu_buffer_rsrc_t rs;
    uint32_t base[INSTR];
    int kq[INSTR];
    uint32_t kstep;
    int wid;

    __device__ __forceinline__ F32xOperand(const void* p, uint32_t bytes, int64_t ld, int64_t rows, int64_t r0,
                                           int wid_, int lane)
        : wid(wid_) {
        rs = make_rsrc(p, bytes);
        kstep = KC ? 4u : (uint32_t)(ld * 4);
#pragma unroll
        for (int q = 0; q < INSTR; ++q) {
            const int unit = (wid * INSTR + q) * 64 + lane;  // 16-byte LDS unit of the stage
            const int sub = unit / (ROWS * 8), u = unit % (ROWS * 8);
            int64_t off;
            bool ok;
            if constexpr (KC) {
                const int r = u >> 3;
                kq[q] = sub * 32 + ((u & 7) ^ dma_a_swz(r)) * 4;
                ok = r0 + r < rows;
                off = (r0 + r) * ld + kq[q];
            } else {
                constexpr int UPR = ROWS / 4;
                const int k = u / UPR;
                const int64_t n = r0 + ((u % UPR) ^ (k & 8)) * 4;
                kq[q] = sub * 32 + k;
                ok = n < rows;
                off = kq[q] * ld + n;
            }
            base[q] = (uint32_t)(off * 4);
            if (!ok) kq[q] = 0x40000000;
        }
    }
    template <int Q>
    __device__ __forceinline__ void copy(int k0, int kend, uint32_t lds) const {
        const uint32_t off = kq[Q] + k0 < kend ? base[Q] + (uint32_t)k0 * kstep : kOob;
        dma16(rs, __builtin_amdgcn_readfirstlane(lds + (uint32_t)((wid * INSTR + Q) * 1024)), off);
    }
    // The lane's 8 consecutive K values of row r0 + lane % 32, K step ks.
    __device__ __forceinline__ static void read(float (&x)[8], const char* s, int r0, int ks, int lane) {
        s += (ks >> 1) * SUB_BYTES;
        if constexpr (KC) {
            const int c = (ks & 1) * 4 + (lane >> 5) * 2;
            const float4 a = *reinterpret_cast<const float4*>(s + dma_a_off(r0 + (lane & 31), c));
            const float4 b = *reinterpret_cast<const float4*>(s + dma_a_off(r0 + (lane & 31), c + 1));
            x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w; x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
        } else {
            const int k = (ks & 1) * 16 + (lane >> 5) * 8, n = r0 + (lane & 31);
            const char* p = s + k * (ROWS * 4) + (n ^ (4 * (k & 8))) * 4;
            static_for<8>([&](auto e) { x[e] = *reinterpret_cast<const float*>(p + e * (ROWS * 4)); });
        }
    }
};

// The three terms of a lane's 8 values, as MFMA operands.
struct F32xTerms {
    uint32_t t[3][4];
    __device__ __forceinline__ uint4 op(int i) const { return make_uint4(t[i][0], t[i][1], t[i][2], t[i][3]); }
};

// The largest magnitude of top and a lane's pair P (a NaN drops out of the maximum
// and stays one in the terms).
template <int P>
__device__ __forceinline__ void f32x_top(float& top, const float (&x)[8]) {
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(top) : "v"(x[2 * P]), "v"(x[2 * P + 1]));
}
// Pair P of a block, scaled, into terms.
template <int P>
__device__ __forceinline__ void f32x_split(F32xTerms& o, const float (&x)[8]) {
    uint32_t w[3];
    split3_pair(x[2 * P] * kF32xScale, x[2 * P + 1] * kF32xScale, w);
    static_for<3>([&](auto i) { o.t[i][P] = w[i]; });
}

template <int BM, int BN, bool TA, bool TB, int WM, int WN, int WK, int ST, int OCC>
__global__ __launch_bounds__(64 * WM * WN * WK, OCC) void gemm_f32x_kernel(GemmArgs a, RingArgs t) {
    gemm_batch_offset(a);
    constexpr int NB = WM * WN, NW = NB * WK, KT = 16 * WK, SUB = KT / 32;
    static_assert(BM == 64 * WM && BN == 64 * WN && WK % 2 == 0, "64 x 64 per wave, whole 32-deep sub-blocks");
    using OpA = F32xOperand<BM, !TA, NW, SUB>;
    using OpB = F32xOperand<BN, TB, NW, SUB>;
    constexpr int STAGE = OpA::BYTES + OpB::BYTES, PER_TILE = OpA::INSTR + OpB::INSTR;
    constexpr int SUMS = (WK - 1) * NB * 16384, EPI = NB * 32 * (64 * 4 + 16);
    static_assert(ST >= 2 && ST * PER_TILE < 64, "vmcnt range");
    static_assert(SUMS + EPI <= ST * STAGE, "the K steps' sums and the epilogue staging must fit in LDS");
    __shared__ __attribute__((aligned(1024))) char smem[ST * STAGE];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wid / NB, wb = wid % NB, wm = wb / WN, wn = wb % WN;
    const int x = (int)blockIdx.x % t.xcds, i = (int)blockIdx.x / t.xcds;
    const int split = i / t.per_xcd, tile = x * t.per_xcd + (i - split * t.per_xcd);
    if (tile >= t.tiles_m * t.tiles_n) return;
    int tm, tn;
    {
        TileMapArgs m{};
        m.tiles_m = t.tiles_m;
        m.tiles_n = t.tiles_n;
        m.group_m = t.group_m;
        tile_coords(m, tile, tm, tn);
    }
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    const int kbeg = split * t.k_per_split, kend = min((int)a.K, kbeg + t.k_per_split);
    const int nk = (kend - kbeg + KT - 1) / KT;  // at least one: the host leaves no slice empty
    const OpA oa(a.A, t.a_bytes, a.lda, a.M, m0, wid, lane);
    const OpB ob(a.B, t.b_bytes, a.ldb, a.N, n0, wid, lane);
    const uint32_t sbase = lds_addr_of(smem);

    f32x16_t acc[2][2], low[2][2];  // hh; the seven small products
    static_for<2>([&](auto i_) {
        static_for<2>([&](auto j) {
            static_for<16>([&](auto v) { acc[i_][j][decltype(v)::value] = low[i_][j][decltype(v)::value] = 0.0f; });
        });
    });

    // Tiles past the end are copied too (every offset out of range: zeros).
    auto copy_part = [&](int tt, int st, auto qc) {
        constexpr int q = decltype(qc)::value;
        const int k0 = kbeg + tt * KT;
        if constexpr (q < OpA::INSTR) oa.template copy<q>(k0, kend, sbase + (uint32_t)(st * STAGE));
        else ob.template copy<q - OpA::INSTR>(k0, kend, sbase + (uint32_t)(st * STAGE + OpA::BYTES));
    };
    static_for<ST>([&](auto s) {
        static_for<PER_TILE>([&](auto q) { copy_part(decltype(s)::value, decltype(s)::value, q); });
    });

    float ra[2][8], rb[2][8];   // fp32 blocks
    F32xTerms ta[2], tb[2];     // split blocks
    float top = 0.0f;  // largest magnitude seen
    auto read_a = [&](auto b, const char* s) { OpA::read(ra[b], s, wm * 64 + b * 32, wk, lane); };
    auto read_b = [&](auto b, const char* s) { OpB::read(rb[b], s + OpA::BYTES, wn * 64 + b * 32, wk, lane); };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    // Smallest terms first: (A, B) = (l,m) (m,l) (m,m) (l,h) (h,l) (m,h) (h,m), then (h,h).
    auto block = [&](auto ic, auto jc, F32xTerms& o, const float (&src)[8], auto&& extra) {
        constexpr int TI[8] = {2, 1, 1, 2, 0, 1, 0, 0}, TJ[8] = {1, 2, 1, 0, 2, 0, 1, 0};
        static_for<8>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            mfma32_bf16(m < 7 ? low[ic][jc] : acc[ic][jc], ta[ic].op(TI[m]), tb[jc].op(TJ[m]));
            if constexpr (m % 2 == 0) f32x_split<m / 2>(o, src);
            else if constexpr (m == 1 || m == 5) extra(std::integral_constant<int, m / 5>{});
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    vm_wait<(ST - 1) * PER_TILE>();
    block_sync();
    read_a(C0{}, smem);
    read_b(C0{}, smem);
    read_a(C1{}, smem);
    read_b(C1{}, smem);
    static_for<4>([&](auto p) {
        f32x_split<decltype(p)::value>(ta[0], ra[0]);
        f32x_split<decltype(p)::value>(tb[0], rb[0]);
    });
    int cur = 0, next = 1, tt = 0;
    auto advance = [&] {
        cur = next;
        next = next + 1 == ST ? 0 : next + 1;
    };
    auto arrive = [&] {
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave holds its part of tile tt, in fp32
        vm_wait<(ST - 2) * PER_TILE>();      // and its share of tile tt + 1 has landed
        block_sync();                        // the same for every wave: tile tt's stage is free
    };
    auto large = [&] {
        static_for<4>([&](auto p) {
            static_for<2>([&](auto b) {
                f32x_top<decltype(p)::value>(top, ra[b]);
                f32x_top<decltype(p)::value>(top, rb[b]);
            });
        });
        return __builtin_amdgcn_ballot_w64(top >= kF32xLimit) != 0;
    };
    arrive();
    bool fp32 = large();
    if (!fp32) do {
        const char* sn = smem + next * STAGE;
        block(C0{}, C0{}, ta[1], ra[1], [&](auto e) {
            if constexpr (e == 0) read_b(C0{}, sn);
            else read_a(C0{}, sn);
        });
        block(C1{}, C0{}, tb[1], rb[1], [&](auto e) {
            constexpr int h = PER_TILE / 2;
            static_for<h>([&](auto q) { copy_part(tt + ST, cur, std::integral_constant<int, e * h + decltype(q)::value>{}); });
        });
        block(C0{}, C1{}, tb[0], rb[0], [&](auto e) {
            if constexpr (e == 0) read_a(C1{}, sn);
        });
        block(C1{}, C1{}, ta[0], ra[0], [&](auto e) {
            if constexpr (e == 0) read_b(C1{}, sn);
        });
        advance();
        ++tt;
        arrive();
        fp32 = large();
    } while (tt < nk && !fp32);
    static_for<2>([&](auto i_) {
        static_for<2>([&](auto j) { acc[i_][j] = (acc[i_][j] + low[i_][j]) * kF32xUnscale; });
    });
    // The rest of the wave's K steps from tile tt on in fp32 (v_mfma_f32_32x32x2_f32:
    // lane half = K index, so instruction e takes values e and 8 + e of the step).
    // The other waves keep their own pace: both loops meet the same barriers.
    if (tt < nk) {
        auto fp32_step = [&](const float (&xa)[2][8], const float (&xb)[2][8]) {
            static_for<PER_TILE>([&](auto q) { copy_part(tt + ST, cur, q); });
            static_for<8>([&](auto e) {
                static_for<2>([&](auto i_) {
                    static_for<2>([&](auto j) {
                        acc[i_][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(xa[i_][e], xb[j][e], acc[i_][j], 0, 0, 0);
                    });
                });
            });
        };
        fp32_step(ra, rb);
        while (++tt < nk) {
            advance();
            float xa[2][8], xb[2][8];
            const char* s = smem + cur * STAGE;
            static_for<2>([&](auto b) {
                OpA::read(xa[b], s, wm * 64 + b * 32, wk, lane);
                OpB::read(xb[b], s + OpA::BYTES, wn * 64 + b * 32, wk, lane);
            });
            arrive();
            fp32_step(xa, xb);
        }
        advance();
        arrive();
    }
    vm_wait<0>();  // copies of tiles past the end still write (zeros) into LDS
    __syncthreads();
    auto piece = [&](int k, auto c) { return reinterpret_cast<f32x4_t*>(smem + (k * NB + wb) * 16384 + c * 1024 + lane * 16); };
    if (wk) {
        static_for<16>([&](auto c) {
            constexpr int cc = decltype(c)::value;
            const f32x16_t& v = acc[cc / 8][cc / 4 % 2];
            *piece(wk - 1, c) = f32x4_t{v[4 * (cc % 4)], v[4 * (cc % 4) + 1], v[4 * (cc % 4) + 2], v[4 * (cc % 4) + 3]};
        });
    }
    __syncthreads();
    if (!wk) {
        static_for<WK - 1>([&](auto k) {
            static_for<16>([&](auto c) {
                constexpr int cc = decltype(c)::value;
                const f32x4_t p = *piece(k, c);
                static_for<4>([&](auto e) { acc[cc / 8][cc / 4 % 2][4 * (cc % 4) + decltype(e)::value] += p[decltype(e)::value]; });
            });
        });
    }
    if (t.splits > 1) {
        uint64_t* const line = t.arrive + (size_t)tile * 8;
        uint64_t old = 0;
        if (tid == 0) old = __hip_atomic_load(line, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // under the stores
        if (!wk) partial_store<2, 2>(acc, partial_rsrc<BM, BN>(a.partial, tile * t.splits + split), wb, lane);
        __syncthreads();  // every wave's partial sums are in L2
        int* word = reinterpret_cast<int*>(smem);
        if (tid == 0) {
            bool mixed = t.mixed != 0;
            const bool last = ring_arrive(line, old, t.epoch, t.splits, &mixed);
            *word = (last ? 1 : 0) | (mixed ? 2 : 0);
        }
        __syncthreads();
        const int state = __builtin_amdgcn_readfirstlane(*word);
        if (!(state & 1) || wk) return;
        if (!(state & 2)) {
            ring_sum<2, 2, BM * BN * 4>(acc, make_rsrc(reinterpret_cast<char*>(a.partial) + (size_t)tile * t.splits * (BM * BN * 4),
                                                       (uint32_t)(t.splits * (BM * BN * 4))), t.splits, wb, lane);
        } else {
            // Slices on several XCDs (see gemm_ring.hpp): all of K here, from memory, in fp32.
            static_for<2>([&](auto i_) {
                static_for<2>([&](auto j) { static_for<16>([&](auto v) { acc[i_][j][decltype(v)::value] = 0.0f; }); });
            });
            const int64_t am = m0 + wm * 64 + (lane & 31), bn = n0 + wn * 64 + (lane & 31);
            for (int k0 = 0; k0 < (int)a.K; k0 += 2) {
                const int64_t k = k0 + (lane >> 5);
                float va[2], vb[2];
                static_for<2>([&](auto b) {
                    const int64_t m = am + b * 32, n = bn + b * 32;
                    const uint32_t oa_ = (uint32_t)((TA ? k * a.lda + m : m * a.lda + k) * 4);
                    const uint32_t ob_ = (uint32_t)((TB ? n * a.ldb + k : k * a.ldb + n) * 4);
                    va[b] = __uint_as_float(buf_load4(oa.rs, k < a.K && m < a.M ? oa_ : kOob));
                    vb[b] = __uint_as_float(buf_load4(ob.rs, k < a.K && n < a.N ? ob_ : kOob));
                });
                static_for<2>([&](auto i_) {
                    static_for<2>([&](auto j) {
                        acc[i_][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[i_], vb[j], acc[i_][j], 0, 0, 0);
                    });
                });
            }
        }
    }
    if (wk) return;
    // staging past the K steps' sums, which slower waves may still be reading
    store_acc_tile<2, 2, 64, 64, NB, true>(a, acc, smem + SUMS, m0, n0, wm, wn, wb, lane);
}

}  // namespace isam
