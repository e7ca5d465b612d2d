// Mid-size bf16 products of the paper's first listing (Section 2): grids of at
// most a few output tiles per compute unit, any operand layout (A [M][K] or
// [K][M], B [K][N] or [N][K]) with 16-byte aligned rows.
//
// Such products are bound by the copies into LDS and by latency, not by the
// matrix cores: a CU holds one or two output tiles, and a 128x128x64 step moves
// 32 KB into LDS (about 770 cycles at the 24 cycles a CU takes per 1 KB copy)
// for 512 cycles of MFMAs.  So:
//   * the operands are copied straight into an LDS ring of ST stages of
//     64-deep K tiles; ST - 1 tiles are in flight (3, 4 and 5 stages time the
//     same, so the latency is covered), with one barrier per tile, and tile
//     t + 1 is read into registers under the MFMAs of tile t;
//   * an operand whose rows run along K is read with ds_read_b128, one whose
//     rows run along M or N with the transposing ds_read_b64_tr_b16, so a
//     transposed A ([K][M], weight gradients) needs no copy in memory first;
//   * K is split over S workgroups per tile when the tiles alone leave CUs
//     idle.  The slices of a tile run on one XCD (workgroup b runs on XCD b %
//     xcds); each leaves its fp32 partial sums in the workspace, in that XCD's
//     L2, and counts itself in; the last to arrive adds the S partial sums in
//     slice order (the same sum whoever is last) and writes C.  Nobody waits,
//     so the form needs no co-residency and no second kernel; the counting word
//     also collects the XCDs, and slices that ran on several (a stream with a CU
//     mask, another partition) make the last arrival form the tile by itself.
// Per call against the plans it replaces (register-staged 128x64 / 64x64 tiles, a
// transposing copy of A, split-K with a reduction kernel): the table above plan_ring
// in api.cpp.  Ablations on 2048x2048x8192 (75 us): MFMAs alone 35 us, copies alone
// 47, LDS reads alone 26 (tr) to 53 (b128); 53 us on zeros, so long products of random
// values are held by power.
// LDS layouts and swizzles are those of the large direct-to-LDS kernel
// (gemm_dma.hpp); rows of 64 M / N values (128 bytes) swizzle their 32-byte
// blocks by 2 * ((k >> 1) & 1): the four K rows of a transpose read are two
// 256-byte bank lines, so rows k and k + 2 have to differ.
#pragma once

#include "gemm_dma.hpp"

namespace isam {

struct RingArgs {
    int tiles_m, tiles_n, group_m;
    int xcds, per_xcd;     // tiles per XCD (the last XCDs' ranges may be short or empty)
    int splits;            // K slices per tile
    int k_per_split;       // multiple of 64
    int fold;              // K tiles (even) whose products are summed before they join the total
    int mixed;             // 1: treat every tile's slices as spread over XCDs (test hook)
    uint32_t a_bytes, b_bytes;  // extents of A and B (per problem of a batch)
    uint64_t epoch;        // arrival words of this launch: epoch (not 0) in the upper 40 bits
    uint64_t* arrive;      // one 64-byte line per tile
};

// One operand of a workgroup's tile: ROWS values of M / N x 64 of K.  KC: rows
// along K (128 bytes of K per row); otherwise K rows of ROWS values.
template <int ROWS, bool KC, int NW>
struct RingOperand {
    static constexpr int BYTES = ROWS * 128;
    static constexpr int INSTR = BYTES / 1024 / NW;  // copies per wave and tile
    static_assert(INSTR >= 1, "tile too small for one copy per wave");
    static_assert(KC || ROWS == 64 || ROWS >= 128, "transpose-read swizzle");
    __amdgpu_buffer_rsrc_t rs;
    uint32_t base[INSTR];  // byte offset of the copy's chunk in the K tile at k = 0
    int kq[INSTR];         // first K index of the chunk in the tile; beyond any K outside M / N
    uint32_t kstep;        // bytes per K value step
    int wid;

    __device__ __forceinline__ static int swz(int k) { return ROWS == 64 ? 2 * ((k >> 1) & 1) : 2 * (k & 3); }

    __device__ __forceinline__ RingOperand(const void* p, uint32_t bytes, int64_t ld, int64_t rows, int64_t r0,
                                           int wid_, int lane)
        : wid(wid_) {
        rs = make_rsrc(p, bytes);
        kstep = KC ? 2u : (uint32_t)(ld * 2);
#pragma unroll
        for (int q = 0; q < INSTR; ++q) {
            const int unit = (wid * INSTR + q) * 64 + lane;  // 16-byte LDS unit of the stage
            int64_t off;
            bool ok;
            if constexpr (KC) {
                const int r = unit >> 3, pc = unit & 7;
                kq[q] = (pc ^ dma_a_swz(r)) * 8;
                ok = r0 + r < rows;
                off = (r0 + r) * ld + kq[q];
            } else {
                constexpr int UPR = ROWS / 8;
                const int k = unit / UPR, u = unit % UPR;
                const int64_t n = r0 + ((u >> 1) ^ swz(k)) * 16 + (u & 1) * 8;
                kq[q] = k;
                ok = n < rows;
                off = k * ld + n;
            }
            base[q] = (uint32_t)(off * 2);
            if (!ok) kq[q] = 0x40000000;
        }
    }
    // Copy instruction Q of the K tile at k0 (values at kend and beyond arrive as zeros).
    template <int Q>
    __device__ __forceinline__ void copy(int k0, int kend, uint32_t lds) const {
        const uint32_t off = kq[Q] + k0 < kend ? base[Q] + (uint32_t)k0 * kstep : kOob;
        dma16(rs, __builtin_amdgcn_readfirstlane(lds + (uint32_t)((wid * INSTR + Q) * 1024)), off);
    }
    // The lane's 8 K values from k of row r, from memory (rows and K values outside: zeros).
    __device__ __forceinline__ static uint4 direct(__amdgpu_buffer_rsrc_t rs, int64_t ld, int64_t rows, int64_t K, int64_t r, int k) {
        if constexpr (KC) {
            return buf_load16(rs, r < rows && k < K ? (uint32_t)((r * ld + k) * 2) : kOob);
        } else {
            uint32_t h[8];
            static_for<8>([&](auto e) { h[e] = buf_load2(rs, r < rows && k + e < K ? (uint32_t)(((k + e) * ld + r) * 2) : kOob) & 0xffffu; });
            return make_uint4(h[0] | h[1] << 16, h[2] | h[3] << 16, h[4] | h[5] << 16, h[6] | h[7] << 16);
        }
    }
    // MFMA operand block (32 rows from r0, K step ks) of the stage at s.
    __device__ __forceinline__ static uint4 frag(const char* s, int r0, int ks, int lane) {
        if constexpr (KC) {
            return *reinterpret_cast<const uint4*>(s + dma_a_off(r0 + (lane & 31), ks * 2 + (lane >> 5)));
        } else {
            const int g = lane >> 4, li = lane & 15;
            const int n = r0 + (g & 1) * 16 + 4 * (li & 3), k = ks * 16 + (g >> 1) * 8 + (li >> 2);
            uint2 h[2];
            static_for<2>([&](auto rc) {
                constexpr int rr = decltype(rc)::value;
                const int kk = k + rr * 4;
                const char* p = s + kk * (ROWS * 2) + (((n >> 4) ^ swz(kk)) * 32) + (n & 15) * 2;
                h[rr] = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)p));
            });
            return make_uint4(h[0].x, h[0].y, h[1].x, h[1].y);
        }
    }
};

// Counts a slice's workgroup in on its tile; true for the last of `splits`.
// The word holds epoch (40 bits), the XCDs seen (one bit each, 16 bits) and
// the count (8 bits); whatever an earlier launch or another program left there
// differs in the epoch and counts as zero.  The last arrival clears the word, so
// a captured launch (the same epoch on every replay) starts from zero too.  Sets
// *mixed if slices ran on several XCDs.
// `old`: a recent reading of the word (a stale one costs another round trip).
__device__ __forceinline__ bool ring_arrive(uint64_t* word, uint64_t old, uint64_t epoch, int splits, bool* mixed) {
    const unsigned xcc = __builtin_amdgcn_s_getreg((20) | (0 << 6) | (31 << 11)) & 0xfu;  // HW_REG_XCC_ID
    const uint64_t bit = 1ull << (8 + xcc);
    for (;;) {
        const uint64_t cur = (old >> 24) == epoch ? old : epoch << 24;
        const uint64_t next = (cur + 1) | bit;
        if (__hip_atomic_compare_exchange_strong(word, &old, next, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT)) {
            const uint64_t seen = (next >> 8) & 0xffff;
            if (seen & (seen - 1)) *mixed = true;
            const bool last = (int)(next & 0xff) == splits;
            if (last) __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return last;
        }
    }
}

// acc = sum over the tile's `splits` partial-sum tiles (consecutive in rp) in
// slice order.  The loads of up to 128 registers' worth of slices go out
// together: the sum is a chain of L2 round trips otherwise.
template <int MI, int NI, int TILE_BYTES>
__device__ __forceinline__ void ring_sum(f32x16_t (&acc)[MI][NI], __amdgpu_buffer_rsrc_t rp, int splits, int wid,
                                         int lane) {
    constexpr int PIECES = MI * NI * 4, GROUP = 32 / PIECES;  // slices loaded together
    const int vo = lane * 16 + wid * PIECES * 1024;
    for (int s0 = 0; s0 < splits; s0 += GROUP) {
        f32x4_t p[GROUP][PIECES];
        static_for<GROUP>([&](auto g) {
            static_for<PIECES>([&](auto c) {
                // slices past the last lie beyond the record count: zeros
                p[g][c] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(
                                                          rp, vo, (s0 + g) * TILE_BYTES + c * 1024, 17));
            });
        });
        __builtin_amdgcn_sched_barrier(0);  // every load issued before the first add
        static_for<GROUP>([&](auto g) {
            static_for<PIECES>([&](auto c) {
                constexpr int cc = decltype(c)::value;
                f32x16_t& v = acc[cc / 4 / NI][cc / 4 % NI];
                static_for<4>([&](auto e) {
                    constexpr int ee = decltype(e)::value, i = 4 * (cc % 4) + ee;
                    v[i] = g == 0 && s0 == 0 ? p[g][cc][ee] : v[i] + p[g][cc][ee];
                });
            });
        });
    }
}

template <int BM, int BN, bool TA, bool TB, int WM, int WN, int ST, int OCC>
__global__ __launch_bounds__(64 * WM * WN, OCC) void gemm_ring_kernel(GemmArgs a, RingArgs t) {
    gemm_batch_offset(a);
    constexpr int NW = WM * WN, WTM = BM / WM, WTN = BN / WN, MI = WTM / 32, NI = WTN / 32;
    using OpA = RingOperand<BM, !TA, NW>;
    using OpB = RingOperand<BN, TB, NW>;
    constexpr int STAGE = OpA::BYTES + OpB::BYTES, PER_TILE = OpA::INSTR + OpB::INSTR;
    static_assert(ST >= 2 && ST * PER_TILE < 64, "vmcnt range");
    static_assert(NW * 32 * (WTN * 4 + 16) <= ST * STAGE, "epilogue staging must fit in LDS");
    __shared__ __attribute__((aligned(1024))) char smem[ST * STAGE];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wid / WN, wn = wid % WN;
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
    const int nk = (kend - kbeg + 63) / 64;  // at least one: the host leaves no slice empty
    const OpA oa(a.A, t.a_bytes, a.lda, a.M, m0, wid, lane);
    const OpB ob(a.B, t.b_bytes, a.ldb, a.N, n0, wid, lane);
    const uint32_t sbase = lds_addr_of(smem);

    // A wave of one 32x32 block has a second accumulator for odd 16-deep K steps:
    // half as many additions one after the other.  Every t.fold K tiles the accumulators
    // join a total and start from zero, so a slice of n K tiles is summed in two
    // short chains (about 2 sqrt(n) additions each for 128x128) instead of one of
    // 4 n, whose error grows with the root of its length.  Error of the norm, fp32
    // out (one chain / the plan replaced, up to eight slices / two chains), and us:
    // 2608x1032x4472 TN 4.2e-7 / 1.8e-7 / 1.3e-7, 41.5 / 81 / 41.9; 1024x2048x8192
    // 4.0e-7 / 1.9e-7 / 1.2e-7, 48.6 / 53 / 49.5; 1024^3 1.3e-7 / 1.8e-7 / 7.7e-8, 9.0 /
    // 15.7 / 9.0.  The folds stand between loops and not in one under a condition, which cost
    // 10 to 35 %.
    constexpr int ODD = MI * NI == 1 ? 1 : 0;
    f32x16_t acc[MI][NI], odd[MI][NI], total[MI][NI];
    auto each = [&](auto&& f) {
        static_for<MI>([&](auto i_) { static_for<NI>([&](auto j) { f(total[i_][j], acc[i_][j], odd[i_][j]); }); });
    };
    auto zero = [](f32x16_t& x) { static_for<16>([&](auto v) { x[decltype(v)::value] = 0.0f; }); };
    auto fold = [&] {
        each([&](f32x16_t& s, f32x16_t& x, f32x16_t& y) {
            if constexpr (ODD) x += y;
            s += x;
            zero(x);
            zero(y);
        });
    };
    each([&](f32x16_t& s, f32x16_t& x, f32x16_t& y) { zero(s); zero(x); zero(y); });

    // Tiles past the end are copied too (every offset out of range: zeros, no
    // memory read), so the number of copies in flight is the same in each step.
    auto copy_part = [&](int tt, int st, auto qc) {
        constexpr int q = decltype(qc)::value;
        const int k0 = kbeg + tt * 64;
        if constexpr (q < OpA::INSTR) oa.template copy<q>(k0, kend, sbase + (uint32_t)(st * STAGE));
        else ob.template copy<q - OpA::INSTR>(k0, kend, sbase + (uint32_t)(st * STAGE + OpA::BYTES));
    };
    static_for<ST>([&](auto s) {
        static_for<PER_TILE>([&](auto q) { copy_part(decltype(s)::value, decltype(s)::value, q); });
    });
    // All fragments of a K tile (four 16-deep steps) in registers; tile tt + 1
    // is read while the MFMAs of tile tt run, so neither the LDS latency nor
    // the barrier stands between MFMA groups.
    struct Frags {
        uint4 a[4][MI], b[4][NI];
    };
    constexpr int READS = 4 * (MI + NI), SLOTS = 4 * MI * NI;
    auto read_part = [&](Frags& f, const char* sa, auto rc) {
        constexpr int r = decltype(rc)::value, ks = r / (MI + NI), o = r % (MI + NI);
        if constexpr (o < MI) f.a[ks][o] = OpA::frag(sa, wm * WTM + o * 32, ks, lane);
        else f.b[ks][o - MI] = OpB::frag(sa + OpA::BYTES, wn * WTN + (o - MI) * 32, ks, lane);
    };
    // MFMAs of `f` (tile tt) with the reads of tile tt + 1 (stage `next`) into
    // `g` and the copies of tile tt + ST into tile tt's stage spread over them
    // (a CU takes 16-20 copies and then stalls further issue at about 24
    // cycles per copy, and a wave stalled on a copy issues no MFMAs).
    int cur = 0, next = 1;
    auto step = [&](const Frags& f, Frags& g, int tt) {
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave holds all of tile tt
        vm_wait<(ST - 2) * PER_TILE>();      // and its share of tile tt + 1 has landed
        block_sync();                        // the same for every wave: tile tt's stage is free
        const char* sn = smem + next * STAGE;
        static_for<SLOTS>([&](auto mc) {
            constexpr int m = decltype(mc)::value, ks = m / (MI * NI), o = m % (MI * NI);
            mfma32_bf16(ks & ODD ? odd[o / NI][o % NI] : acc[o / NI][o % NI], f.a[ks][o / NI], f.b[ks][o % NI]);
            constexpr int rlo = m * READS / SLOTS, rhi = (m + 1) * READS / SLOTS;
            static_for<rhi - rlo>([&](auto d) { read_part(g, sn, std::integral_constant<int, rlo + decltype(d)::value>{}); });
            constexpr int lo = m * PER_TILE / SLOTS, hi = (m + 1) * PER_TILE / SLOTS;
            static_for<hi - lo>([&](auto d) { copy_part(tt + ST, cur, std::integral_constant<int, lo + decltype(d)::value>{}); });
            __builtin_amdgcn_sched_barrier(0);
        });
        cur = next;
        next = next + 1 == ST ? 0 : next + 1;
    };
    Frags f0, f1;
    vm_wait<(ST - 1) * PER_TILE>();
    block_sync();
    static_for<READS>([&](auto r) { read_part(f0, smem, r); });
    int tt = 0;
    for (const int even = nk & ~1;;) {
        for (const int stop = min(even, tt + t.fold); tt < stop; tt += 2) {
            step(f0, f1, tt);
            step(f1, f0, tt + 1);
        }
        if (tt >= even) break;
        fold();
    }
    if (nk & 1) step(f0, f1, tt);
    vm_wait<0>();  // copies of tiles past the end still write (zeros) into LDS
    fold();
    each([](f32x16_t& s, f32x16_t& x, f32x16_t&) { x = s; });
    __syncthreads();
    if (t.splits > 1) {
        uint64_t* const line = t.arrive + (size_t)tile * 8;
        uint64_t old = 0;
        if (tid == 0) old = __hip_atomic_load(line, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // under the stores
        partial_store<MI, NI>(acc, partial_rsrc<BM, BN>(a.partial, tile * t.splits + split), wid, lane);
        __syncthreads();  // every wave's partial sums are in L2
        int* word = reinterpret_cast<int*>(smem);
        if (tid == 0) {
            bool mixed = t.mixed != 0;
            const bool last = ring_arrive(line, old, t.epoch, t.splits, &mixed);
            *word = (last ? 1 : 0) | (mixed ? 2 : 0);
        }
        __syncthreads();
        const int state = __builtin_amdgcn_readfirstlane(*word);
        if (!(state & 1)) return;
        __syncthreads();
        if (!(state & 2)) {
            ring_sum<MI, NI, BM * BN * 4>(acc, make_rsrc(reinterpret_cast<char*>(a.partial) + (size_t)tile * t.splits * (BM * BN * 4),
                                                              (uint32_t)(t.splits * (BM * BN * 4))), t.splits, wid, lane);
        } else {
            // Slices on several XCDs (workgroups are dealt to them in turn, so never
            // seen) cannot read each other's sums, which are in their own L2: all of K
            // here, straight from memory (the way above in a loop cost every product
            // 2 %).
            static_for<MI>([&](auto i_) {
                static_for<NI>([&](auto j) { static_for<16>([&](auto v) { acc[i_][j][decltype(v)::value] = 0.0f; }); });
            });
            for (int k0 = 0; k0 < (int)a.K; k0 += 16) {
                const int k = k0 + (lane >> 5) * 8;
                uint4 fa[MI], fb[NI];
                static_for<MI>([&](auto i_) { fa[i_] = OpA::direct(oa.rs, a.lda, a.M, a.K, m0 + wm * WTM + i_ * 32 + (lane & 31), k); });
                static_for<NI>([&](auto j) { fb[j] = OpB::direct(ob.rs, a.ldb, a.N, a.K, n0 + wn * WTN + j * 32 + (lane & 31), k); });
                static_for<MI>([&](auto i_) { static_for<NI>([&](auto j) { mfma32_bf16(acc[i_][j], fa[i_], fb[j]); }); });
            }
        }
    }
    store_acc_tile<MI, NI, WTM, WTN, NW, true>(a, acc, smem, m0, n0, wm, wn, wid, lane);
}

typedef void (*GemmRingFn)(GemmArgs, RingArgs);

hipError_t ring_args(const GemmArgs& a, const RingPlan& r, const RingPadded& pad, int es, int cus, RingArgs* out);

}  // namespace isam
