// Instantiations and launch of the LDS-ring kernel for mid-size bf16 products.
#include "gemm_ring.hpp"

namespace isam {

namespace {

template <int BM, int BN, int WM, int WN, int ST, int OCC>
GemmRingFn ring_fn(int ta, int tb) {
    if (ta) return tb ? gemm_ring_kernel<BM, BN, true, true, WM, WN, ST, OCC> : gemm_ring_kernel<BM, BN, true, false, WM, WN, ST, OCC>;
    return tb ? gemm_ring_kernel<BM, BN, false, true, WM, WN, ST, OCC> : gemm_ring_kernel<BM, BN, false, false, WM, WN, ST, OCC>;
}

}  // namespace

void gemm_ring_dims(int ring, int* bm, int* bn) {
    *bm = ring == 2 ? 64 : 128;
    *bn = ring == 1 ? 128 : 64;
}

size_t gemm_ring_ws_bytes(const RingPlan& r, int64_t M, int64_t N) {
    if (!r.ring || r.splits <= 1) return 0;
    int bm, bn;
    gemm_ring_dims(r.ring, &bm, &bn);
    const size_t tiles = (size_t)((M + bm - 1) / bm) * (size_t)((N + bn - 1) / bn);
    return tiles * ((size_t)r.splits * bm * bn * 4 + 64);
}

// What a launch of either ring kernel (es: bytes per operand value) passes besides the operands.
hipError_t ring_args(const GemmArgs& a, const RingPlan& r, const RingPadded& pad, int es, int cus, RingArgs* out) {
    int bm, bn;
    gemm_ring_dims(r.ring, &bm, &bn);
    RingArgs t{};
    t.tiles_m = (int)((a.M + bm - 1) / bm);
    t.tiles_n = (int)((a.N + bn - 1) / bn);
    t.group_m = 8;
    t.mixed = r.mixed;
    t.xcds = cus % 32 == 0 ? cus / 32 : 1;
    const int64_t tiles = (int64_t)t.tiles_m * t.tiles_n;
    t.per_xcd = (int)((tiles + t.xcds - 1) / t.xcds);
    const int64_t nk = (a.K + 63) / 64;
    const int want = a.batch > 1 || r.splits < 1 ? 1 : r.splits;
    t.k_per_split = (int)(((nk + want - 1) / want) * 64);
    t.splits = (int)((a.K + t.k_per_split - 1) / t.k_per_split);  // no slice is empty
    // K tiles per fold: about half the root of a slice's K tiles makes the two chains of
    // additions equal; fewer than four cost time and gain nothing over the plans that
    // cut K into more slices.  Up to K = 4096, 128x128 tiles stand in for plans of one
    // slice, whose error they have in one chain of up to 2048 of K (3072x1024x2048 TN
    // accumulating 22.2 us, 22.8 with folds).
    t.fold = 4;
    while (4 * t.fold * t.fold < t.k_per_split / 64) t.fold += 2;
    if (r.ring == 1 && a.K < 4096 && t.k_per_split <= 2048) t.fold = 32;
    if (t.splits > 255 || (t.splits > 1 && ((uintptr_t)a.partial & 255))) return hipErrorInvalidValue;
    const int64_t a_rows = a.trans_a ? a.K : a.M, a_cols = a.trans_a ? a.M : a.K;
    const int64_t b_rows = a.trans_b ? a.N : a.K, b_cols = a.trans_b ? a.K : a.N;
    t.a_bytes = (uint32_t)((pad.a ? a_rows * a.lda : (a_rows - 1) * a.lda + a_cols) * es);
    t.b_bytes = (uint32_t)((pad.b ? b_rows * a.ldb : (b_rows - 1) * a.ldb + b_cols) * es);
    t.epoch = next_fixup_epoch() & ((1ull << 40) - 1);
    if (!t.epoch) t.epoch = 1;
    t.arrive = reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(a.partial) + (size_t)tiles * t.splits * bm * bn * 4);
    *out = t;
    return hipSuccess;
}

hipError_t launch_gemm_ring(const GemmArgs& a, const RingPlan& r, const RingPadded& pad, int cus, hipStream_t s) {
    if (a.ab_type != kBF16 || (r.ring != 1 && r.ring != 2) || a.K <= 0) return hipErrorInvalidValue;
    // 128x128: 8 waves of 64x32, four stages (128 KB), one workgroup per CU;
    // 64x64: 4 waves of 32x32, four stages (64 KB), two workgroups per CU.
    const int threads = r.ring == 1 ? 512 : 256;
    const GemmRingFn fn = r.ring == 1 ? ring_fn<128, 128, 2, 4, 4, 2>(a.trans_a, a.trans_b)
                                      : ring_fn<64, 64, 2, 2, 4, 2>(a.trans_a, a.trans_b);
    RingArgs t{};
    hipError_t e = ring_args(a, r, pad, 2, cus, &t);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)(t.xcds * t.per_xcd * t.splits), 1, (unsigned)(a.batch > 1 ? a.batch : 1));
    hipLaunchKernelGGL(fn, grid, dim3(threads), 0, s, a, t);
    return hipGetLastError();
}

}  // namespace isam
