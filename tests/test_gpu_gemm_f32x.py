"""fp32 products on bf16 terms formed in registers: against 64-bit products, also out of the terms' range."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1810_09958_amd as isam


def _tol(K):
    # Of sum |a||b|: the terms the kernels drop (at most 2^-23), the 32-bit sums (one rounding per 16
    # values of K, the small products' far below, at most 24 when the K steps and slices are added)
    # and the result's.
    return 2.0 ** -23 + (K / 16 + 26) * 2.0 ** -24


def _operands(M, N, K, ta, tb, pad, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def make(r, c):
        w = torch.full((r, c + pad), float("nan"), device="cuda")
        w[:, :c] = torch.randn((r, c), generator=g, device="cuda")
        return w[:, :c]

    return make(K, M) if ta else make(M, K), make(N, K) if tb else make(K, N)


def _check(A, B, ta, tb, acc=False, ct=torch.float32, workspace=None):
    A64, B64 = (A.t() if ta else A).double().contiguous(), (B.t() if tb else B).double().contiguous()
    K = A64.shape[1]
    C = torch.randn((A64.shape[0], B64.shape[1]), device="cuda").to(ct)
    ref = A64 @ B64 + (C.double() if acc else 0)
    S = A64.abs() @ B64.abs() + (C.double().abs() if acc else 0)
    isam.gemm(A, B, C, trans_a=bool(ta), trans_b=bool(tb), accumulate=acc, workspace=workspace)
    tol = _tol(K) + (2.0 ** -8 if ct == torch.bfloat16 else 0)
    fin = S < 3e38  # the others overflow or hold an infinity or a NaN: the same value in both
    assert bool(((C.double() - ref).abs()[fin] <= tol * S[fin] + K * 2.0 ** -126).all())  # products below 2^-126 may be flushed
    want = ref.float()[~fin]
    same = (C.float()[~fin] == want) | (torch.isnan(want) & torch.isnan(C.float()[~fin]))
    assert bool(same.all())
    return C


# Edges of the tiles, K of one tile and less, ragged K tiles, more slices than K tiles.
@pytest.mark.parametrize("ring", [1, 2, 3])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K,rs", [(4, 4, 4, 1), (128, 64, 64, 2), (132, 68, 36, 1), (64, 260, 640, 4),
                                      (260, 132, 652, 5), (128, 128, 2048, 16), (388, 520, 200, 3)])
def test_f32x_forced(ring, ta, tb, M, N, K, rs, monkeypatch):
    monkeypatch.setenv("ISAM_GEMM_CONFIG", f"f32x={ring},rs={rs},skinny=0,small=0")
    _check(*_operands(M, N, K, ta, tb, 0, M + K), ta, tb)
    _check(*_operands(M, N, K, ta, tb, 4, N + K), ta, tb, acc=True, ct=torch.bfloat16)


# Slices that ran on several XCDs (forced from the host): the last arrival forms the whole tile, with
# and without values that take the fp32 instructions.
@pytest.mark.parametrize("ring", [1, 2, 3])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
def test_f32x_slices_on_several_xcds(ring, ta, tb, monkeypatch):
    monkeypatch.setenv("ISAM_GEMM_CONFIG", f"f32x={ring},rs=3,rmix=1,skinny=0,small=0")
    A, B = _operands(260, 200, 652, ta, tb, 4, ring)
    _check(A, B, ta, tb, acc=True)
    (A.t() if ta else A)[7, 300] = math.inf
    _check(A, B, ta, tb)


# As planned: aligned and odd sizes (operands copied into padded rows), with too little
# workspace for slices or copies, and the strided batch of a convolution.
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(1024, 512, 2048), (999, 1001, 1003), (2052, 516, 516)])
def test_f32x_planned(ta, tb, M, N, K, monkeypatch):
    monkeypatch.delenv("ISAM_GEMM_CONFIG", raising=False)
    A, B = _operands(M, N, K, ta, tb, 0, M)
    _check(A, B, ta, tb)
    _check(A, B, ta, tb, workspace=torch.empty(256, device="cuda", dtype=torch.uint8))
    x, w = torch.randn((3, 700, 256), device="cuda"), torch.randn((5, 256, 384), device="cuda") / 36
    y = isam.conv1d(x, w).double()
    ref = sum(x.double()[:, d:d + 696].reshape(-1, 256).contiguous() @ w[d].double() for d in range(5))
    S = sum(x.double().abs()[:, d:d + 696].reshape(-1, 256).contiguous() @ w[d].double().abs() for d in range(5))
    assert bool(((y.reshape(-1, 384) - ref).abs() <= _tol(5 * 256) * S).all())


# An XCD runs whole tiles with all their slices: a plan may not give a full one more rounds of
# workgroups than the chip has on average (84 tiles of 64x64 in three slices did: 33 on 32 CUs).
@pytest.mark.parametrize("M,N,K,ta,tb", [(128, 2688, 3456, 0, 1), (2600, 68, 3232, 1, 0), (1536, 768, 3072, 1, 0), (200, 2000, 4000, 1, 0)])
def test_f32x_plan_counts_rounds_per_xcd(M, N, K, ta, tb, monkeypatch, capfd):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("counts for 8 XCDs of 32 CUs")
    monkeypatch.delenv("ISAM_GEMM_CONFIG", raising=False)
    monkeypatch.setenv("ISAM_LOG", "1")
    _check(*_operands(M, N, K, ta, tb, 0, K), ta, tb)
    plan = capfd.readouterr().err.split("ring kernel: ")[1]
    bm, bn = (int(x) for x in plan.split(" ")[0].split("x"))
    slices, tiles = int(plan.split(" K slices")[0].split(" ")[-1]), -(-M // bm) * -(-N // bn)
    assert -(-(-(-tiles // 8) * slices) // 32) == -(-tiles * slices // 256)


# Products that the split copies (any alignment) served: with bases and leading dimensions off 16
# bytes and the queried workspace they run on the terms too, not element by element.
@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("off_a,off_b", [(1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(2048, 1024, 1024), (1144, 1776, 928)])
def test_fp32_unaligned_operands_run_on_terms(tb, off_a, off_b, M, N, K, monkeypatch, capfd):
    monkeypatch.delenv("ISAM_GEMM_CONFIG", raising=False)
    monkeypatch.setenv("ISAM_LOG", "1")
    A, B = _operands(M, N, K, 0, tb, 0, 3)

    def shift(x, off):  # rows one value longer, from an odd address
        if not off:
            return x
        w = torch.zeros(x.shape[0] * (x.shape[1] + 1) + 1, device="cuda")[1:].view(x.shape[0], x.shape[1] + 1)[:, : x.shape[1]]
        w.copy_(x)
        return w

    _check(shift(A, off_a), shift(B, off_b), 0, tb)
    log = capfd.readouterr().err
    assert "ring kernel" in log or "fp32 split into bf16 terms" in log, log


# Values that do not split into bf16 terms (infinities, NaNs, magnitudes from 2^28: the waves that
# read them go on in fp32), and rows and columns of tiny values.
@pytest.mark.parametrize("ring,rs", [(1, 1), (1, 3), (2, 1), (2, 4), (3, 2)])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
def test_f32x_range(ring, rs, ta, tb, monkeypatch):
    monkeypatch.setenv("ISAM_GEMM_CONFIG", f"f32x={ring},rs={rs},skinny=0,small=0")
    A, B = _operands(260, 200, 328, ta, tb, 0, 9)
    Am, Bm = (A.t() if ta else A), (B.t() if tb else B)
    Am[3] *= 2.0 ** 100
    Am[7] *= 2.0 ** -100
    Am[130, 200] = math.inf
    Am[131, 327] = -math.inf
    Am[200, 5] = math.nan
    Bm[:, 150] *= 2.0 ** -110
    Bm[17, 2] = 1e37
    C = _check(A, B, ta, tb)
    assert bool(torch.isinf(C[130]).any()) and bool(torch.isnan(C[200]).all())


def test_f32x_error_is_below_the_fp32_instructions(monkeypatch):
    # Against 64 bits, over the products that moved from the fp32 tile kernel: no larger.
    for M, N, K, tb in [(2048, 1024, 1024, 1), (512, 512, 4096, 0), (8192, 256, 256, 0)]:
        A, B = _operands(M, N, K, 0, tb, 0, K)
        ref = A.double() @ (B.t() if tb else B).double().contiguous()
        err = {}
        for env in ("", "f32x=0,f32split=0"):
            monkeypatch.setenv("ISAM_GEMM_CONFIG", env)
            C = isam.gemm(A, B, trans_b=bool(tb))
            err[env] = float((C.double() - ref).norm() / ref.norm())
        assert err[""] <= err["f32x=0,f32split=0"], err


# One non-zero product per result (a diagonal operand): the fp32 product rounded once, as the fp32
# instructions give it, but for the dropped ll and the roundings of the small products' sum, each
# below 2^-8 of a half unit in the last place.
@pytest.mark.parametrize("ring,rs", [(1, 1), (2, 3), (3, 1)])
def test_f32x_single_products(ring, rs, monkeypatch):
    monkeypatch.setenv("ISAM_GEMM_CONFIG", f"f32x={ring},rs={rs},skinny=0,small=0")
    _, B = _operands(256, 512, 256, 0, 0, 0, 4)
    d = torch.randn(256, device="cuda", generator=torch.Generator(device="cuda").manual_seed(7))
    ref = d.double()[:, None] * B.double()
    for C in (isam.gemm(torch.diag(d), B), isam.gemm(B.t().contiguous(), torch.diag(d)).t()):
        assert bool(((C.double() - ref).abs() <= 1.01 * 2.0 ** -24 * ref.abs()).all())


# Tiny values beside ordinary ones in the same row, where the ordinary ones meet zeros: down to
# denormals, and up to the largest values that are split.  The tolerance is that of ordinary values
# (no allowance for products below 2^-126: there are none).
@pytest.mark.parametrize("ring,rs", [(1, 1), (2, 3), (3, 1)])
@pytest.mark.parametrize("small", [-100, -115, -126, -140])
def test_f32x_tiny_beside_ordinary(ring, rs, small, monkeypatch):
    monkeypatch.setenv("ISAM_GEMM_CONFIG", f"f32x={ring},rs={rs},skinny=0,small=0")
    A, B = _operands(132, 136, 200, 0, 0, 0, -small)
    A.clamp_(-4, 4).mul_(2.0 ** small)
    B.clamp_(-4, 4).mul_(2.0 ** 25)
    A[:, ::7] = 1.0
    B[::7] = 0.0
    for C, ref, S in ((isam.gemm(A, B), A.double() @ B.double(), A.double().abs() @ B.double().abs()),
                      (isam.gemm(B.t().contiguous(), A.t().contiguous()), B.double().t().contiguous() @ A.double().t().contiguous(),
                       B.double().abs().t().contiguous() @ A.double().abs().t().contiguous())):
        assert bool(((C.double() - ref).abs() <= _tol(200) * S).all())


# One large value (just split, the first that is not, and far out) in the first, a middle or the last
# K tile of a slice: the waves that read it change to fp32 instructions there.
@pytest.mark.parametrize("ring,rs", [(1, 1), (2, 2), (3, 1)])
@pytest.mark.parametrize("k", [0, 15, 16, 70, 130, 235, 251])
def test_f32x_large_values(ring, rs, k, monkeypatch):
    monkeypatch.setenv("ISAM_GEMM_CONFIG", f"f32x={ring},rs={rs},skinny=0,small=0")
    for v in (math.nextafter(2.0 ** 28, 0), 2.0 ** 28, -3e36):
        A, B = _operands(132, 136, 252, 0, 0, 0, k)
        A[5, k] = v
        A[:, :k][A[:, :k].abs() < 0.1] = 0.0
        _check(A, B, 0, 0)
        _check(B.t().contiguous(), A.t().contiguous(), 0, 0)


def test_f32x_large_values_cost_no_second_pass(monkeypatch):
    # Large values everywhere in a column of A: the fp32 instructions run once, at about the speed of
    # the fp32 tile kernel (measured: 1.2 times the time without; 6.5 times when the tiles were formed
    # again).
    monkeypatch.delenv("ISAM_GEMM_CONFIG", raising=False)

    def best(A, B):
        C, ms = isam.gemm(A, B, trans_b=True), []
        for _ in range(8):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(10):
                isam.gemm(A, B, C, trans_b=True)
            e1.record()
            torch.cuda.synchronize()
            ms.append(e0.elapsed_time(e1))
        return min(ms)

    A, B = _operands(2048, 1024, 1024, 0, 1, 0, 3)
    plain = best(A, B)
    A[:, 0] = 1e30
    assert best(A, B) <= 2.5 * plain


# Streaming kernel on fp32 (N <= 256, K <= 128, B in registers): ragged last 32-row tile, K off the
# MFMA step, N off a wave's 32 columns, padded leading dimensions.
@pytest.mark.parametrize("M,N,K", [(33, 8, 8), (100, 40, 36), (257, 256, 128), (64, 100, 100), (95, 256, 4),
                                   (1, 4, 64), (300, 12, 124), (20000, 132, 64)])
def test_stream_fp32(M, N, K, monkeypatch):
    monkeypatch.setenv("ISAM_GEMM_CONFIG", "stream=1,skinny=0,small=0,f32x=0")
    _check(*_operands(M, N, K, 0, 0, 0, M), 0, 0)
    _check(*_operands(M, N, K, 0, 0, 4, N), 0, 0, acc=True, ct=torch.bfloat16)
    A, B = _operands(M, N, K, 0, 0, 0, M)
    A[M // 2, K - 1], B[K - 1, 1] = math.inf, 0.0
    _check(A, B, 0, 0)
