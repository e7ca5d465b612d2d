"""LDS-ring kernel of mid-size bf16 products: every element against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests._util import TOL_BF16, bits, norm_err, to_gpu, to_host_f64

pytestmark = pytest.mark.gpu

import paper_1810_09958_amd as isam

# fp32 outputs of bf16 products are exact products summed in fp32: sums of at most 4200 terms
# in any order stay within 4200 * 2^-24 = 2.5e-4 of sum |a||b|; bf16 outputs add half an ulp
# (2^-9 of the result).
TOL_SUM = 2.5e-4


def _check(M, N, K, ta, tb, ct="f32", acc=False, pad=0, shift=0, seed=0, workspace=None):
    Am, Bm = synth.uniform(seed, 80, (M, K), -1, 1), synth.uniform(seed, 81, (K, N), -1, 1)
    A_h, B_h = bits(np.ascontiguousarray(Am.T) if ta else Am), bits(np.ascontiguousarray(Bm.T) if tb else Bm)

    def place(h):
        # rows padded with NaN patterns and a base off 16 bytes by `shift` values
        w = np.full((h.shape[0], h.shape[1] + pad), 0x7FC0, h.dtype)
        w[:, : h.shape[1]] = h
        flat = to_gpu(np.concatenate([np.full(shift, 0x7FC0, h.dtype), w.ravel()]))
        return flat[shift:].view(w.shape)[:, : h.shape[1]]

    A, B = place(A_h), place(B_h)
    out_t = torch.bfloat16 if ct == "bf16" else torch.float32
    C_in = None
    if acc:
        c0 = synth.uniform(seed, 82, (M, N), -1, 1)
        C = to_gpu(bits(c0) if ct == "bf16" else c0)
        C_in = to_host_f64(C)
        isam.gemm(A, B, C, trans_a=bool(ta), trans_b=bool(tb), accumulate=True, workspace=workspace)
    else:
        C = isam.gemm(A, B, trans_a=bool(ta), trans_b=bool(tb), out_dtype=out_t, workspace=workspace)
    torch.cuda.synchronize()
    ref, S = oracle.gemm(A_h, B_h, M, N, K, ta, tb, C_in=C_in)
    assert norm_err(to_host_f64(C), ref, S) <= (TOL_BF16 if ct == "bf16" else TOL_SUM)
    return A, B, C


# Edges of the tiles (one row, one over, one under), K of one tile and less, ragged K tiles,
# more slices than K tiles, and the slice counts around the groups the sum loads together.
@pytest.mark.parametrize("ring", ["1", "2"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K,rs", [(8, 8, 8, 1), (128, 64, 64, 2), (136, 120, 72, 1), (64, 264, 640, 4),
                                      (264, 72, 648, 5), (72, 136, 1152, 9), (128, 128, 2048, 16), (392, 520, 200, 3)])
def test_ring_forced(ring, ta, tb, M, N, K, rs, monkeypatch):
    monkeypatch.setenv("ISAM_GEMM_CONFIG", f"ring={ring},rs={rs},skinny=0,small=0")
    _check(M, N, K, ta, tb, seed=M + K + rs)
    _check(M, N, K, ta, tb, ct="bf16", acc=True, pad=8, seed=M + N + rs)


# Slices that ran on several XCDs (forced from the host): the last arrival forms the whole tile.
@pytest.mark.parametrize("ring", ["1", "2"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K,rs", [(136, 120, 648, 3), (264, 72, 2000, 7), (128, 128, 128, 2)])
def test_ring_slices_on_several_xcds(ring, ta, tb, M, N, K, rs, monkeypatch):
    monkeypatch.setenv("ISAM_GEMM_CONFIG", f"ring={ring},rs={rs},rmix=1,skinny=0,small=0")
    _check(M, N, K, ta, tb, seed=M + K + rs)
    _check(M, N, K, ta, tb, ct="bf16", acc=True, pad=8, seed=M + N + rs)


# Odd sizes: operands copied into padded rows, C rows that are not 16-byte aligned.
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(1000, 1537, 1023), (89, 170, 800), (131, 67, 1573), (700, 12, 312), (65, 71, 100)])
def test_ring_odd_sizes(ta, tb, M, N, K, monkeypatch):
    monkeypatch.delenv("ISAM_GEMM_CONFIG", raising=False)
    _check(M, N, K, ta, tb, seed=K)
    _check(M, N, K, ta, tb, ct="bf16", acc=True, seed=K + 1)


# Bases and leading dimensions off 16 bytes, with and without a workspace that holds the copies.
@pytest.mark.parametrize("room", [0, 16 << 20])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
def test_ring_unaligned_operands(ta, tb, room, monkeypatch):
    monkeypatch.delenv("ISAM_GEMM_CONFIG", raising=False)
    ws = torch.empty(max(room, 1), device="cuda", dtype=torch.uint8)
    _check(520, 648, 1032, ta, tb, pad=3, shift=1, seed=5, workspace=ws)


# Against 64 bits, no larger an error than the plans the kernel stands in for, which cut deep K into
# up to eight slices: K from one fold of the accumulators to many, an odd number of K tiles, and a
# short last one.
@pytest.mark.parametrize("M,N,K,ta,tb", [(2608, 1032, 4472, 1, 0), (2048, 1024, 4096, 0, 1), (1024, 2048, 8192, 0, 0),
                                         (512, 512, 16384, 0, 0), (64, 960, 1024, 1, 0), (568, 208, 936, 1, 0),
                                         (144, 3864, 4152, 0, 0), (3072, 1024, 2048, 1, 0), (2304, 1408, 3080, 0, 0)])
def test_ring_error_is_no_larger_than_with_more_slices(M, N, K, ta, tb, monkeypatch):
    g = torch.Generator(device="cuda").manual_seed(K)
    A = torch.randn((K, M) if ta else (M, K), device="cuda", generator=g).bfloat16()
    B = torch.randn((N, K) if tb else (K, N), device="cuda", generator=g).bfloat16()
    ref = (A.t() if ta else A).double().contiguous() @ (B.t() if tb else B).double().contiguous()
    err = {}
    for env in ("", "ring=0"):
        monkeypatch.setenv("ISAM_GEMM_CONFIG", env)
        err[env] = float((isam.gemm(A, B, trans_a=bool(ta), trans_b=bool(tb)).double() - ref).norm() / ref.norm())
    assert err[""] <= err["ring=0"], err


# A workspace of the queried size that starts anywhere has room for the planned K slices, and one of
# half the size for fewer; nothing outside it is written.
@pytest.mark.parametrize("off", [0, 2, 16, 100, 255])
def test_ring_workspace_at_any_address(off, monkeypatch, capfd):
    monkeypatch.delenv("ISAM_GEMM_CONFIG", raising=False)
    monkeypatch.setenv("ISAM_LOG", "1")
    M, N, K = 512, 512, 4096
    slices = {}
    for part in (1, 2):
        need = isam.gemm_workspace_size(M, N, K, 1, 0) if part == 1 else 64 * (2 * 64 * 64 * 4 + 64) + 255
        buf = torch.full((off + need + 512,), 0xA5, device="cuda", dtype=torch.uint8)
        _check(M, N, K, 0, 0, workspace=buf[off : off + need])
        slices[part] = int(capfd.readouterr().err.split(" K slices")[0].split()[-1])
        assert bool((buf[:off] == 0xA5).all()) and bool((buf[off + need :] == 0xA5).all())
    assert slices == {1: 4, 2: 2}


def test_ring_deterministic_and_captured(monkeypatch):
    # K slices summed by whichever workgroup arrives last: the same bits every time, on a
    # workspace that holds anything, and when one captured launch is replayed.
    monkeypatch.setenv("ISAM_GEMM_CONFIG", "ring=2,rs=7")
    M, N, K = 200, 328, 4096
    ws = torch.full((isam.gemm_workspace_size(M, N, K, 1, 0),), 255, device="cuda", dtype=torch.uint8)
    A, B, C = _check(M, N, K, 0, 0, workspace=ws)
    for _ in range(5):
        assert torch.equal(isam.gemm(A, B, workspace=ws), C)
    out = torch.zeros_like(C)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        isam.gemm(A, B, out, workspace=ws)
    for _ in range(4):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, C)
        assert torch.equal(isam.gemm(A, B, workspace=ws), C)


def test_ring_batched_conv1d(monkeypatch):
    # short sequences: a strided batch of small tiles on the ring kernel
    monkeypatch.delenv("ISAM_GEMM_CONFIG", raising=False)
    nb, L, Ki, D, Ko = 5, 77, 72, 3, 200
    A_h, B_h = bits(synth.normal(1, 83, (nb, L, Ki))), bits(synth.uniform(1, 84, (D, Ki, Ko), -0.1, 0.1))
    C = isam.conv1d(to_gpu(A_h), to_gpu(B_h))
    torch.cuda.synchronize()
    ref, S = oracle.conv1d(A_h, B_h)
    assert norm_err(to_host_f64(C), ref, S) <= TOL_SUM
