// Instantiations and launch of the fp32 kernel on bf16 terms.
#include "gemm_f32x.hpp"

namespace isam {

namespace {

template <int BM, int BN, int WM, int WN, int WK, int ST, int OCC>
GemmRingFn f32x_fn(int ta, int tb) {
    if (ta) return tb ? gemm_f32x_kernel<BM, BN, true, true, WM, WN, WK, ST, OCC> : gemm_f32x_kernel<BM, BN, true, false, WM, WN, WK, ST, OCC>;
    return tb ? gemm_f32x_kernel<BM, BN, false, true, WM, WN, WK, ST, OCC> : gemm_f32x_kernel<BM, BN, false, false, WM, WN, WK, ST, OCC>;
}

}  // namespace

hipError_t launch_gemm_f32x(const GemmArgs& a, const RingPlan& r, const RingPadded& pad, int cus, hipStream_t s) {
    if (a.ab_type != kF32 || r.ring < 1 || r.ring > 3 || a.K <= 0) return hipErrorInvalidValue;
    // 128x128: 8 waves, 2 x 2 blocks of 64x64 x 2 K steps, four stages (128 KB);
    // 64x64: 4 waves, one block x 4 K steps, four stages (128 KB).
    // 128x64: 8 waves, 2 blocks x 4 K steps, three stages (144 KB).
    const int threads = r.ring == 2 ? 256 : 512;
    const GemmRingFn fn = r.ring == 1   ? f32x_fn<128, 128, 2, 2, 2, 4, 2>(a.trans_a, a.trans_b)
                          : r.ring == 2 ? f32x_fn<64, 64, 1, 1, 4, 4, 1>(a.trans_a, a.trans_b)
                                        : f32x_fn<128, 64, 2, 1, 4, 3, 2>(a.trans_a, a.trans_b);
    RingArgs t{};
    hipError_t e = ring_args(a, r, pad, 4, cus, &t);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)(t.xcds * t.per_xcd * t.splits), 1, (unsigned)(a.batch > 1 ? a.batch : 1));
    hipLaunchKernelGGL(fn, grid, dim3(threads), 0, s, a, t);
    return hipGetLastError();
}

}  // namespace isam
