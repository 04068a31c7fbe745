"""Kernel-level parity of the projection kernels (twist_gemm_raw) against the plain matrix product in fp64 on the
same inputs: <= 5e-3 with bf16 operands and output (fp32 accumulation), <= 1e-4 when the output is fp32."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from helpers import rel_fro, to_numpy

pytestmark = pytest.mark.gpu

SHAPES = [  # (M, N, K): several tiles with ragged edges, a tiny one, k not a multiple of the k-tile
    (300, 200, 136), (129, 257, 64), (8, 8, 8), (513, 384, 1000), (256, 256, 4096), (1000, 72, 520), (260, 580, 72),
]


@pytest.mark.parametrize("tile", [128, 256, "plain"])
@pytest.mark.parametrize("layout", [0, 1, 2])
def test_bf16_projection_matches_fp64_product(lib, layout, tile):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG3))
    if tile == "plain":
        ctx.twist_set_kernel_choice(plain_only=True)          # the fall-back kernel for unaligned bf16 operands
    else:
        ctx.twist_set_kernel_choice(gemm_tile=tile)
    for M, N, K in SHAPES:
        a_shape = (K, M) if layout == 2 else (M, K)
        b_shape = (N, K) if layout == 0 else (K, N)
        A = si.to_bf16_grid(si.normal(M + N, f"A{layout}", a_shape))
        B = si.to_bf16_grid(si.normal(K, f"B{layout}", b_shape, 0.05))
        want = (A.T if layout == 2 else A) @ (B.T if layout == 0 else B)
        At, Bt = (torch.tensor(x, dtype=torch.float64).to(torch.bfloat16).cuda() for x in (A, B))
        for out_dtype, tol in ((torch.bfloat16, 5e-3), (torch.float32, 1e-4)):
            out = torch.full((M, N), float("nan"), dtype=out_dtype, device="cuda")
            guard = torch.zeros(64, dtype=out_dtype, device="cuda")       # allocated right after: must stay zero
            ctx.twist_gemm_raw(layout, M, N, K, At, Bt, out, alpha=0.5)
            torch.cuda.synchronize()
            assert rel_fro(to_numpy(out), 0.5 * want) <= tol, (layout, tile, M, N, K, out_dtype)
            assert not guard.any()


# rows padded to 16 bytes whose last chunk is partly used: the last k row (layout 2) or the last row (layout 1) of the operand ends in it
@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("layout,M,N,K", [(2, 129, 64, 40), (2, 33, 257, 64), (1, 40, 64, 1003), (1, 257, 136, 129)])
def test_bf16_projection_uses_a_partly_filled_last_chunk(lib, tile, layout, M, N, K):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG3))
    ctx.twist_set_kernel_choice(gemm_tile=tile)
    up = lambda n: (n + 7) // 8 * 8
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    a_rows, a_cols = (K, M) if layout == 2 else (M, K)
    A, B = torch.zeros((a_rows, up(a_cols)), device="cuda").bfloat16()[:, :a_cols], torch.zeros((K, up(N)), device="cuda").bfloat16()[:, :N]
    A.copy_(torch.randn(A.shape, generator=gen, device="cuda"))
    B.copy_(torch.randn(B.shape, generator=gen, device="cuda"))
    want = (A.double().T if layout == 2 else A.double()) @ B.double()
    out = torch.full((M, N), float("nan"), device="cuda")
    ctx.twist_gemm_raw(layout, M, N, K, A, B, out)
    torch.cuda.synchronize()
    # fp32 sums of exact products: an element that misses one of K products is off by 1 / sqrt(K)
    rows = (out.double() - want).norm(dim=1) / want.norm(dim=1)
    assert float(rows.max()) <= 1e-5 and float((out.double() - want).norm() / want.norm()) <= 1e-5


def test_fp32_projection(lib):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG1))
    for layout in (0, 1, 2):
        M, N, K = 150, 70, 90
        a_shape = (K, M) if layout == 2 else (M, K)
        b_shape = (N, K) if layout == 0 else (K, N)
        A, B = si.normal(1, "a", a_shape), si.normal(2, "b", b_shape)
        A, B = A.astype(np.float32).astype(np.float64), B.astype(np.float32).astype(np.float64)
        want = (A.T if layout == 2 else A) @ (B.T if layout == 0 else B)
        out = torch.empty((M, N), dtype=torch.float32, device="cuda")
        ctx.twist_gemm_raw(layout, M, N, K, torch.tensor(A, dtype=torch.float32).cuda(), torch.tensor(B, dtype=torch.float32).cuda(), out)
        assert rel_fro(to_numpy(out), want) <= 1e-4


# By size: the first shapes take the 32x32 tiles, the last four the 64x64 tiles; edges of both, contractions shorter than, ending in and
# filling a slice (128 and 64 long) and fewer slices than the four stages
@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(8, 8, 8), (1, 40, 120), (31, 33, 136), (33, 64, 264), (128, 768, 1032), (65, 200, 3080),
                                   (500, 2300, 136), (513, 2304, 8), (449, 2305, 56), (520, 2048, 648)])
def test_small_bf16_projection_edges(lib, layout, M, N, K):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG3))
    assert {ctx.twist_gemm_kernel(layout, M, N, K, f32)[0] for f32 in (False, True)} == {64 if M >= 449 else 32}
    up = lambda n: (n + 7) // 8 * 8
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, B = ((torch.randn((r, up(c)), generator=gen, device="cuda").bfloat16()[:, :c]) for r, c in
            ((K, M) if layout == 2 else (M, K), (N, K) if layout == 0 else (K, N)))      # rows 16 bytes apart
    want = (A.double().T if layout == 2 else A.double()) @ (B.double().T if layout == 0 else B.double())
    for dt, tol in ((torch.bfloat16, 5e-3), (torch.float32, 1e-5)):
        buf = torch.full((M * N + 64,), float("nan"), dtype=dt, device="cuda")            # what lies behind the result must stay
        out = buf[:M * N].view(M, N)
        ctx.twist_gemm_raw(layout, M, N, K, A, B, out, alpha=0.5)
        torch.cuda.synchronize()
        assert float((out.double() - 0.5 * want).norm() / (0.5 * want).norm()) <= tol
        assert torch.isnan(buf[M * N:]).all()


# fp32 kernels: tiles of 32 (by size), 64 (pinned by 256) and 128 (pinned), ragged edges, contractions that end
# inside a slice of 32 or 64, strides that allow 16-byte loads and strides that do not (odd K, M or N)
@pytest.mark.parametrize("tile", [0, 128, 256])
@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (64, 64, 32), (65, 63, 33), (132, 260, 100), (300, 200, 136), (127, 129, 31), (40, 72, 1028)])
def test_fp32_projection_edges(lib, tile, layout, M, N, K):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG1))
    ctx.twist_set_kernel_choice(gemm_tile=tile)
    assert ctx.twist_gemm_kernel(layout, M, N, K, True)[0] == {0: 32, 128: 128, 256: 64}[tile]
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn((K, M) if layout == 2 else (M, K), generator=gen, device="cuda")
    B = torch.randn((N, K) if layout == 0 else (K, N), generator=gen, device="cuda")
    want = (A.double().T if layout == 2 else A.double()) @ (B.double().T if layout == 0 else B.double())
    buf = torch.full((M * N + 64,), float("nan"), device="cuda")            # what lies behind the result must stay
    out = buf[:M * N].view(M, N)
    ctx.twist_gemm_raw(layout, M, N, K, A, B, out, alpha=0.5)
    torch.cuda.synchronize()
    # K products of one rounding each and K additions: 2^-24 sqrt(2 K) at most about 3e-6 here
    assert float((out.double() - 0.5 * want).norm() / (0.5 * want).norm()) <= 3e-6
    assert torch.isnan(buf[M * N:]).all()


# the tiles on the bf16 instruction: operands of very different sizes, and values that their three terms cannot stand for (infinities, NaNs, the largest
# floats, which round to infinity in bf16) give what the plain kernel gives; rows and columns without such a value stay finite and exact
@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("layout", [0, 1, 2])
def test_fp32_projection_with_values_beyond_the_terms(lib, tile, layout):
    M, N, K = 260, 140, 200
    ctx = lib.Context(lib.desc_from_cfg(si.CFG1))
    gen = torch.Generator(device="cuda").manual_seed(layout)
    A, B = torch.randn((M, K), generator=gen, device="cuda"), torch.randn((N, K), generator=gen, device="cuda")
    A *= 10.0 ** torch.randint(-12, 12, (M, 1), generator=gen, device="cuda")
    for special in (None, float("inf"), float("-inf"), float("nan"), 3.4e38):
        a, b = A.clone(), B.clone()
        if special is not None:
            a[70, 50], b[100, 7] = special, special
            a[70, 51:] = 0.0
        want = (a.double() @ b.double().T).float()                        # 64 bits: overflows where fp32 does
        a_, b_ = (a.T.contiguous() if layout == 2 else a), (b if layout == 0 else b.T.contiguous())
        out = torch.empty((M, N), device="cuda")
        ctx.twist_set_kernel_choice(gemm_tile=tile)
        ctx.twist_gemm_raw(layout, M, N, K, a_, b_, out)
        torch.cuda.synchronize()
        ok = torch.isfinite(want)
        assert torch.equal(torch.isfinite(out), ok) and torch.equal(torch.isnan(out), torch.isnan(want)), special
        err = torch.where(ok, (out.double() - want.double()).abs(), 0.0)
        # 2^-24 sqrt(2 K) of the row's and column's norms, three times that for the largest of 36000 entries; terms near 3.4e38 leave nothing of others
        bound = 4e-6 * a.double().nan_to_num(0, 0, 0).norm(dim=1)[:, None] * b.double().nan_to_num(0, 0, 0).norm(dim=1)[None, :]
        assert bool((err <= bound).all()), special


# ... and operands down to the smallest float, whose lower terms would be below the smallest bf16, against as large ones on the other side (the largest
# overflow as terms).  Bound: K products summed in fp32 in any order, 2^-24 sqrt(K) of the result's norm
@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("up,down", [(90, -100), (90, -112), (90, -120), (90, -126), (95, -135), (118, -135), (-20, -100)])
def test_fp32_projection_of_tiny_operands(lib, tile, layout, up, down):
    M, N, K = 260, 140, 200
    ctx = lib.Context(lib.desc_from_cfg(si.CFG1))
    gen = torch.Generator(device="cuda").manual_seed(layout)
    A, B = torch.randn((M, K), generator=gen, device="cuda"), torch.randn((N, K), generator=gen, device="cuda")
    for ea, eb in ((up, down), (down, up)):
        a, b = (A.double() * 2.0 ** ea).float(), (B.double() * 2.0 ** eb).float()
        want = a.double() @ b.double().T
        a_, b_ = (a.T.contiguous() if layout == 2 else a), (b if layout == 0 else b.T.contiguous())
        out = torch.empty((M, N), device="cuda")
        ctx.twist_set_kernel_choice(gemm_tile=tile)
        ctx.twist_gemm_raw(layout, M, N, K, a_, b_, out)
        torch.cuda.synchronize()
        assert float((out.double() - want).norm() / want.norm()) <= 2.0 ** -24 * K ** 0.5


# tiles of 64 whose rows are padded to 16 bytes, NaNs in the padding: contractions that end at and beside a wave's step of 16 and the waves' round of
# 64 or 128, rows and columns that end inside a tile; one tile per CU (eight waves) and more (four)
@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(64, 64, 1), (1, 3, 17), (65, 63, 15), (127, 130, 16), (193, 62, 127), (66, 64, 128), (64, 129, 131), (61, 190, 525),
                                   (1089, 1027, 50), (1100, 1026, 64), (1027, 1089, 67), (1030, 1091, 243)])
def test_fp32_projection_leaves_padding_out(lib, layout, M, N, K):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG1))
    ctx.twist_set_kernel_choice(gemm_tile=256)
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)

    def padded(rows, cols):
        x = torch.full((rows, (cols + 3) // 4 * 4), float("nan"), device="cuda")
        x[:, :cols] = torch.randn((rows, cols), generator=gen, device="cuda")
        return x[:, :cols]
    A, B = padded(*((K, M) if layout == 2 else (M, K))), padded(*((N, K) if layout == 0 else (K, N)))
    want = (A.double().T if layout == 2 else A.double()) @ (B.double().T if layout == 0 else B.double())
    buf = torch.full((M * N + 64,), float("nan"), device="cuda")
    out = buf[:M * N].view(M, N)
    ctx.twist_gemm_raw(layout, M, N, K, A, B, out, alpha=0.5)
    torch.cuda.synchronize()
    # K products of one rounding each and K additions against the sum of the products' sizes; a product left out or counted twice is 1 / K of that on
    # average, and more than 10 times the bound
    size = (A.double().abs().T if layout == 2 else A.double().abs()) @ (B.double().abs().T if layout == 0 else B.double().abs())
    assert float(((out.double() - 0.5 * want).abs() / (0.5 * size)).max()) <= 2.0 ** -24 * (K + 2)
    assert torch.isnan(buf[M * N:]).all()


# tiles of 64 (eight waves to a tile, and four) sum no coarser than tiles of 128, whose waves share every slice: contractions of a few steps of 16 to a
# wave, where the additions of the waves' sums are most of the error.  (2 % for the norm over a million outputs)
@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("size", [1024, 2048])
@pytest.mark.parametrize("K", [48, 56, 64, 96, 128, 192, 320, 768])
def test_fp32_tiles_of_64_sum_as_finely_as_tiles_of_128(lib, layout, size, K):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG1))
    gen = torch.Generator(device="cuda").manual_seed(K)
    A = torch.randn((K, size) if layout == 2 else (size, K), generator=gen, device="cuda")
    B = torch.randn((size, K) if layout == 0 else (K, size), generator=gen, device="cuda")
    want = (A.double().T if layout == 2 else A.double()) @ (B.double().T if layout == 0 else B.double())
    err = []
    for pin in (128, 256):
        ctx.twist_set_kernel_choice(gemm_tile=pin)
        out = torch.empty((size, size), device="cuda")
        ctx.twist_gemm_raw(layout, size, size, K, A, B, out)
        torch.cuda.synchronize()
        err.append(float((out.double() - want).norm() / want.norm()))
    assert err[1] <= 1.02 * err[0], err


# contractions below 320 in tiles of 64 keep the kernel whose waves share every slice, the one of rows that are not aligned: the same bits.  (Not where one
# tile a CU has a last slice of 64 that is half empty, and not from 320 on)
@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("M,N,K,same", [(264, 328, 64, True), (1000, 772, 48, True), (1024, 768, 128, True), (1028, 772, 244, True), (2048, 1028, 96, True), (1500, 1540, 316, True),
                                        (1024, 768, 96, False), (1028, 772, 320, False), (1500, 1540, 320, False)])
def test_fp32_short_contractions_in_tiles_of_64(lib, layout, M, N, K, same):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG1))
    ctx.twist_set_kernel_choice(gemm_tile=256)
    assert ctx.twist_gemm_kernel(layout, M, N, K, True)[0] == 64
    gen = torch.Generator(device="cuda").manual_seed(K)
    A = torch.randn((K, M) if layout == 2 else (M, K), generator=gen, device="cuda")
    B = torch.randn((N, K) if layout == 0 else (K, N), generator=gen, device="cuda")
    odd = lambda x: torch.cat((x[:, :1], x), 1)[:, 1:]
    bufs = [torch.full((M * N + 64,), float("nan"), device="cuda") for _ in range(2)]
    outs = [buf[:M * N].view(M, N) for buf in bufs]
    ctx.twist_gemm_raw(layout, M, N, K, odd(A), odd(B), outs[0])
    ctx.twist_gemm_raw(layout, M, N, K, A, B, outs[1])
    torch.cuda.synchronize()
    want = (A.double().T if layout == 2 else A.double()) @ (B.double().T if layout == 0 else B.double())
    assert torch.equal(*outs) == same and all(torch.isnan(buf[M * N:]).all() for buf in bufs)
    assert float((outs[1].double() - want).norm() / want.norm()) <= 1e-6


# ... and some that tiles of 128 would take go to the waves of tiles of 64 (last steps, rounds and columns that are not whole): no coarser than on tiles of 128, which
# rows that are not aligned run on.  (2 % for the norm over a million outputs)
@pytest.mark.parametrize("layout,M,N,K", [(0, 4095, 763, 160), (0, 8190, 771, 100), (0, 3001, 3071, 244), (0, 1827, 5515, 316), (1, 4093, 764, 132), (1, 3001, 3076, 252), (1, 2599, 2340, 96),
                                          (2, 4092, 764, 163), (2, 3712, 3700, 283), (2, 50252, 764, 257)])
def test_fp32_short_contractions_by_waves_of_whole_tiles(lib, layout, M, N, K):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG1))
    assert ctx.twist_gemm_kernel(layout, M, N, K, True) == (64, 64, 1)
    gen = torch.Generator(device="cuda").manual_seed(K)
    A = torch.randn((K, M) if layout == 2 else (M, K), generator=gen, device="cuda")
    B = torch.randn((N, K) if layout == 0 else (K, N), generator=gen, device="cuda")
    want = (A.double().T if layout == 2 else A.double()) @ (B.double().T if layout == 0 else B.double())
    odd = lambda x: torch.cat((x[:, :1], x), 1)[:, 1:]
    buf = torch.full((M * N + 64,), float("nan"), device="cuda")
    out, err = buf[:M * N].view(M, N), []
    for a, b in ((odd(A), odd(B)), (A, B)):
        ctx.twist_gemm_raw(layout, M, N, K, a, b, out)
        torch.cuda.synchronize()
        err.append(float((out.double() - want).norm() / want.norm()))
    assert err[1] <= 1.02 * err[0] and torch.isnan(buf[M * N:]).all(), err


# aligned operands take kernels of their own: their sums are no coarser than those of the same product on rows that are not aligned.  Products that the
# fp32 instruction, a shorter cut of the contraction or fewer waves to a tile would give a larger error for (1.3 to 3.7 times), and some where the
# kernels agree.  (3 % for the norm over 1e5 outputs and more)
@pytest.mark.parametrize("layout,M,N,K", [(2, 2908, 316, 92), (1, 4696, 164, 68), (1, 276, 500, 1272), (0, 2972, 200, 256), (0, 1136, 604, 320), (2, 332, 5892, 160),
                                          (1, 248, 1008, 1408), (2, 2176, 80, 2032), (1, 464, 1056, 5884), (1, 740, 848, 8704), (2, 1504, 448, 9024), (2, 768, 384, 1024),
                                          (2, 1500, 1500, 2000), (1, 1024, 768, 1536)])
def test_fp32_projection_of_aligned_operands_sums_as_finely(lib, layout, M, N, K):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG1))
    gen = torch.Generator(device="cuda").manual_seed(K)
    A = torch.randn((K, M) if layout == 2 else (M, K), generator=gen, device="cuda")
    B = torch.randn((N, K) if layout == 0 else (K, N), generator=gen, device="cuda")
    want = (A.double().T if layout == 2 else A.double()) @ (B.double().T if layout == 0 else B.double())
    scratch = torch.empty(1 << 24, device="cuda")
    odd = lambda x: torch.cat((x[:, :1], x), 1)[:, 1:]
    err = []
    for a, b in ((odd(A), odd(B)), (A, B)):
        out = torch.empty((M, N), device="cuda")
        ctx.twist_gemm_raw_cut(layout, M, N, K, a, b, out, scratch)
        torch.cuda.synchronize()
        err.append(float((out.double() - want).norm() / want.norm()))
    assert err[1] <= 1.03 * err[0], err


# a tile that an infinity or a NaN reaches is formed a second time, on the fp32 instruction (measured: twice as long in all).  A loop over k
# per output in its place took 34 to 115 times as long
@pytest.mark.parametrize("layout,M,N,K", [(0, 1024, 20000, 768), (0, 1024, 1536, 768), (1, 1024, 768, 1536), (2, 2048, 2048, 768)])
def test_fp32_projection_of_nans_keeps_its_speed(lib, layout, M, N, K):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG1))
    assert ctx.twist_gemm_kernel(layout, M, N, K)[0] >= 64
    A, B = torch.randn((K, M) if layout == 2 else (M, K), device="cuda"), torch.randn((N, K) if layout == 0 else (K, N), device="cuda")
    out = torch.empty((M, N), device="cuda")

    def fastest(passes):
        times = []
        for _ in range(passes):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                ctx.twist_gemm_raw(layout, M, N, K, A, B, out)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    plain = fastest(6)
    A.fill_(float("nan"))
    assert fastest(3) <= 8 * plain and bool(torch.isnan(out).all())


@pytest.mark.parametrize("M,N,K,tile", [(3000, 2900, 72, 64), (4000, 3900, 72, 128)])
def test_fp32_projection_by_size_takes_the_larger_tiles(lib, M, N, K, tile):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG1))
    assert ctx.twist_gemm_kernel(0, M, N, K, True)[0] == tile
    gen = torch.Generator(device="cuda").manual_seed(1)
    A, B = torch.randn((M, K), generator=gen, device="cuda"), torch.randn((N, K), generator=gen, device="cuda")
    out = torch.full((M, N), float("nan"), device="cuda")
    ctx.twist_gemm_raw(0, M, N, K, A, B, out)
    want = A.double() @ B.double().T
    assert float((out.double() - want).norm() / want.norm()) <= 3e-6


def test_raw_rejects_bad_strides(lib):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG3))
    A = torch.zeros(16, 8, dtype=torch.bfloat16, device="cuda")
    out = torch.zeros(16, 16, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(lib.TwistError):
        ctx.twist_gemm_raw(0, 16, 16, 32, A, A, out)      # K larger than the row stride
    with pytest.raises(lib.TwistError):
        ctx.twist_set_kernel_choice(gemm_tile=64)         # only 0, 128 and 256 exist


# y = x W^T on the ping-pong kernel: contractions around the length of its ring of five sub-tiles of 32, odd and even counts of them,
# edges of a tile, and more tiles than workgroups (a second tile through the same stages)
@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("M,N,K", [(1, 1, 8), (255, 130, 32), (257, 260, 40), (300, 64, 64), (256, 256, 96), (31, 300, 136), (520, 136, 168), (256, 129, 328),
                                   (4360, 4100, 72)])
def test_bf16_nt_projection_edges(lib, tile, M, N, K):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG3))
    ctx.twist_set_kernel_choice(gemm_tile=tile)
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, B = (torch.randn((r, K), generator=gen, device="cuda").bfloat16() for r in (M, N))
    want = A.double() @ B.double().T
    buf = torch.full((M * N + 64,), float("nan"), device="cuda")            # what lies behind the result must stay
    out = buf[:M * N].view(M, N)
    ctx.twist_gemm_raw(0, M, N, K, A, B, out)
    torch.cuda.synchronize()
    # fp32 sums of K exact products: 2^-24 sqrt(K) at most; a dropped or repeated chunk of 8 would show as sqrt(8 / K) >= 0.15
    assert float((out.double() - want).norm() / want.norm()) <= 5e-6
    assert torch.isnan(buf[M * N:]).all()


# Products whose contraction is cut (tile, then shape): parts of uneven length, a last one shorter than a slice, ragged edges; NN and TN
@pytest.mark.parametrize("tile,layout,M,N,K", [((32, 32), 2, 136, 200, 5000), ((32, 32), 2, 33, 40, 16000), ((32, 32), 1, 70, 72, 3000), ((64, 64), 2, 768, 192, 8100),
                                               ((64, 64), 2, 520, 776, 8100), ((64, 64), 1, 264, 776, 12008), ((128, 128), 2, 1536, 776, 4000),
                                               ((128, 128), 1, 1100, 1032, 4000), ((256, 128), 2, 1536, 776, 8200), ((256, 128), 1, 1100, 1032, 9001),
                                               ((256, 256), 2, 2816, 2048, 8200)])
def test_cut_bf16_projection(lib, tile, layout, M, N, K):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG3))
    scratch = torch.full((1 << 24,), float("nan"), device="cuda")
    for f32 in (False, True):
        rows, cols, parts = ctx.twist_gemm_kernel(layout, M, N, K, f32, scratch.numel())
        assert (rows, cols) == tile and parts > 1, (rows, cols, parts)
    up = lambda n: (n + 7) // 8 * 8
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, B = (torch.randn((r, up(c)), generator=gen, device="cuda").bfloat16()[:, :c] for r, c in (((K, M) if layout == 2 else (M, K)), (K, N)))
    want = (A.double().T if layout == 2 else A.double()) @ B.double()
    for dt in (torch.float32, torch.bfloat16):
        buf = torch.full((M * N + 64,), float("nan"), dtype=dt, device="cuda")            # what lies behind the result must stay
        out = buf[:M * N].view(M, N)
        ctx.twist_gemm_raw_cut(layout, M, N, K, A, B, out, scratch, alpha=0.5)
        torch.cuda.synchronize()
        rows = (out.double() - 0.5 * want).norm(dim=1) / (0.5 * want).norm(dim=1)
        # fp32 sums of K exact products: 2^-24 sqrt(K) at most; one left out or counted twice shows as 1 / sqrt(K), the rounding to bf16 as 2e-3
        assert float(rows.max()) <= (2.0 ** -24 * K ** 0.5 if dt == torch.float32 else 5e-3)
        assert torch.isnan(buf[M * N:]).all() and torch.isnan(scratch[parts * M * N:]).all()


# Tiles whose two groups of waves share the contraction: every tile in every layout, ragged rows and columns, contractions that end within a
# slice, on an odd and on an even one; cut; with alpha, and with the activation of the up projection
@pytest.mark.parametrize("tile,layout,M,N,K", [
    ((64, 96), 0, 326, 3333, 856), ((128, 96), 0, 3527, 844, 208), ((128, 128), 0, 787, 3836, 200), ((128, 192), 0, 1619, 3636, 808), ((192, 128), 0, 1309, 3077, 648),
    ((64, 96), 1, 3611, 267, 887), ((128, 96), 1, 1374, 2178, 219), ((128, 128), 1, 1647, 1881, 209), ((128, 192), 1, 1578, 3605, 976), ((192, 128), 1, 1038, 3635, 730),
    ((64, 96), 2, 2729, 323, 943), ((128, 96), 2, 2942, 1040, 210), ((128, 128), 2, 1932, 1571, 203), ((128, 192), 2, 2306, 2462, 890), ((192, 128), 2, 1035, 3598, 637),
    ((128, 128), 2, 1020, 2045, 8190)])
def test_bf16_projection_in_two_groups(lib, tile, layout, M, N, K):
    cut = K > 8000
    ctx = lib.Context(lib.desc_from_cfg(si.ModelCfg(d_model=64, n_heads=1, d_head=8, d_ff=N, act="relu", dtype="bf16")))
    scratch = torch.full((1 << 24,), float("nan"), device="cuda")
    rows, cols, parts = ctx.twist_gemm_kernel(layout, M, N, K, True, scratch.numel() if cut else 0)
    assert (rows, cols) == tile and (parts > 1) == cut, (rows, cols, parts)
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    up = lambda n: (n + 7) // 8 * 8
    def operand(r, c):                                                   # rows padded to whole chunks: with zeros along k, with NaNs otherwise
        x = torch.full((r, up(c)), 0.0 if c == K else float("nan"), device="cuda").bfloat16()
        x[:, :c] = torch.randn((r, c), generator=gen, device="cuda").bfloat16()
        return x[:, :c]
    A = operand(K, M) if layout == 2 else operand(M, K)
    B = operand(N, K) if layout == 0 else operand(K, N)
    want = (A.double().T if layout == 2 else A.double()) @ (B.double().T if layout == 0 else B.double())
    for dt, alpha in ((torch.float32, 0.5), (torch.float32, 1.0), (torch.bfloat16, 1.0)):
        buf = torch.full((M * N + 64,), float("nan"), dtype=dt, device="cuda")             # what lies behind the result must stay
        out = buf[:M * N].view(M, N)
        if dt == torch.float32 and cut: ctx.twist_gemm_raw_cut(layout, M, N, K, A, B, out, scratch, alpha=alpha)
        else: ctx.twist_gemm_raw(layout, M, N, K, A, B, out, alpha=alpha)
        torch.cuda.synchronize()
        err = (out.double() - alpha * want).norm(dim=1) / (alpha * want).norm(dim=1)
        # fp32 sums of K exact products: 2^-24 sqrt(K) at most; one left out or counted twice shows as 1 / sqrt(K), the rounding to bf16 as 2e-3
        assert float(err.max()) <= (2.0 ** -24 * K ** 0.5 if dt == torch.float32 else 5e-3)
        assert torch.isnan(buf[M * N:]).all()
    if layout == 0:
        got, act = ctx.twist_gemm_act_raw(A.contiguous(), B.contiguous(), None, ctx.desc.act)
        torch.cuda.synchronize()
        assert torch.equal(got, out) and torch.equal(act, out.relu())


# Kernels are chosen by time among those whose fp32 sums are no coarser than on tiles of 256 rows, 64x64 and 32x32: errors as measured on the kernel that those
# alone would give the product to, cut where that pays (tiles of 64x96 to 192x128 with a shorter cut leave 1.2 to 2.1 times that; the last two are uncut and
# at 0.7).  (5 % for the norm over 1e5 outputs and more of other normal operands)
@pytest.mark.parametrize("layout,M,N,K,err", [(2, 6728, 136, 7984, 1.80e-7), (1, 1344, 872, 7960, 2.19e-7), (1, 4216, 488, 7448, 2.11e-7), (2, 2456, 1000, 8144, 2.22e-7),
                                              (1, 544, 2544, 4368, 1.95e-7), (1, 496, 6720, 7552, 2.62e-7), (2, 1920, 1144, 3488, 2.01e-7), (1, 728, 5504, 4928, 2.42e-7),
                                              (0, 2880, 328, 7600, 2.63e-7), (2, 3280, 1568, 1024, 1.84e-7), (0, 7224, 728, 568, 1.32e-7)])
def test_bf16_projection_sums_as_finely(lib, layout, M, N, K, err):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG3))
    gen = torch.Generator(device="cuda").manual_seed(K)
    A = torch.randn((K, M) if layout == 2 else (M, K), generator=gen, device="cuda").bfloat16()
    B = torch.randn((N, K) if layout == 0 else (K, N), generator=gen, device="cuda").bfloat16()
    want = (A.double().T if layout == 2 else A.double()) @ (B.double().T if layout == 0 else B.double())
    out, scratch = torch.empty((M, N), device="cuda"), torch.empty(1 << 24, device="cuda")
    ctx.twist_gemm_raw_cut(layout, M, N, K, A, B, out, scratch)
    torch.cuda.synchronize()
    assert float((out.double() - want).norm() / want.norm()) <= 1.05 * err


# ... and as weight gradients in one launch, whole and cut
@pytest.mark.parametrize("tile,cut,K,shapes", [((64, 96), False, 1000, [(264, 1541), (520, 768), (0, 8), (768, 264)]),
                                               ((192, 128), False, 1000, [(2000, 2048), (1032, 520)]), ((128, 128), True, 8190, [(1152, 804), (575, 928)])])
def test_weight_gradients_in_two_groups(lib, tile, cut, K, shapes):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG3))
    gen = torch.Generator(device="cuda").manual_seed(K)
    up = lambda n: (n + 7) // 8 * 8
    rows = lambda n: torch.randn((K, up(n)), generator=gen, device="cuda").bfloat16()[:, :n]
    scratch = torch.full((1 << 24,), float("nan"), device="cuda")
    bufs = [torch.full((M * N + 64,), float("nan"), device="cuda") for M, N in shapes]
    products = [(rows(M), rows(N), buf[:M * N].view(M, N)) for (M, N), buf in zip(shapes, bufs)]
    alphas = (0.5, 1.0, 2.0, 1.0)[:len(shapes)]
    r, c, parts = ctx.twist_weight_grads_raw(K, products, scratch, alphas)
    torch.cuda.synchronize()
    assert (r, c) == tile and (parts > 1) == cut, (r, c, parts)
    for (a, b, out), buf, alpha in zip(products, bufs, alphas):
        want = alpha * (a.double().T @ b.double())
        assert out.numel() == 0 or float(((out.double() - want).norm(dim=1) / want.norm(dim=1)).max()) <= 2.0 ** -24 * K ** 0.5
        assert torch.isnan(buf[out.numel():]).all()


# fp32 weight gradients in one launch, on every tile, whole and cut: odd sizes (partial products that leave the next product's unaligned), an empty one; then
# rows that are not 16-byte aligned, and contractions of a few elements: one by one
@pytest.mark.parametrize("tile,cut,K,shapes", [(32, False, 100, [(33, 41), (70, 36), (131, 40), (8, 33)]), (32, True, 1249, [(88, 345), (344, 87), (88, 833), (0, 8)]),
                                               (64, False, 1100, [(360, 1127), (1128, 360)]), (64, True, 3337, [(176, 351), (353, 176), (176, 320), (961, 176)]),
                                               (128, False, 321, [(752, 2400), (2401, 751)])])
def test_fp32_weight_gradients_in_one_launch(lib, tile, cut, K, shapes):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG1))
    gen = torch.Generator(device="cuda").manual_seed(K)
    rows = lambda n: torch.randn((K, (n + 3) // 4 * 4), generator=gen, device="cuda")[:, :n]
    alphas = (0.5, 1.0, 2.0, 1.0)[:len(shapes)]
    scratch = torch.full((1 << 24,), float("nan"), device="cuda")
    bufs = [torch.full((M * N + 64,), float("nan"), device="cuda") for M, N in shapes]
    products = [(rows(M), rows(N), buf[:M * N].view(M, N)) for (M, N), buf in zip(shapes, bufs)]
    r, _, parts = ctx.twist_weight_grads_raw(K, products, scratch, alphas)
    torch.cuda.synchronize()
    assert r == tile and (parts > 1) == cut, (r, parts)
    for (a, b, out), buf, alpha in zip(products, bufs, alphas):
        want = alpha * (a.double().T @ b.double())
        # fp32 sums of K products, 2^-24 sqrt(K) at most; one left out or counted twice shows as 1 / sqrt(K)
        assert out.numel() == 0 or float(((out.double() - want).norm(dim=1) / want.norm(dim=1)).max()) <= 2.0 ** -24 * K ** 0.5
        assert torch.isnan(buf[out.numel():]).all()
    assert torch.isnan(scratch[parts * sum(M * N for M, N in shapes) if cut else 0:]).all()
    a, b, out = products[0]
    for x, y in ((a[:, 1:], b), (a[:5], b[:5])):
        one = torch.empty((x.shape[1], y.shape[1]), device="cuda"), torch.empty((x.shape[1], y.shape[1]), device="cuda")
        assert ctx.twist_weight_grads_raw(x.shape[0], [(x, y, one[0]), (x, y, one[1])], scratch, (1.0, 0.5)) == (0, 0, 0)
        torch.cuda.synchronize()
        want = x.double().T @ y.double()
        assert torch.equal(one[0] * 0.5, one[1]) and float((one[0].double() - want).norm() / want.norm()) <= 2.0 ** -24 * K ** 0.5


# ... whose sums are no coarser than those of the products one by one on rows that are not aligned: groups that fewer parts of the contraction or four waves to
# a tile instead of eight would give a larger error for (1.15 to 1.6 times).  (3 % for the norm over the 3000 outputs and more of each)
@pytest.mark.parametrize("K,shapes", [(2948, [(1276, 448), (448, 1276), (1276, 508), (1524, 1276)]), (923, [(124, 92), (184, 124), (124, 404), (1212, 124)]),
                                      (850, [(708, 72), (72, 708)]), (5454, [(864, 372), (744, 864)]), (2937, [(448, 604), (1208, 448)]), (256, [(64, 128), (256, 128)])])
def test_fp32_weight_gradients_in_one_launch_sum_as_finely(lib, K, shapes):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG1))
    gen = torch.Generator(device="cuda").manual_seed(K)
    operands = [[torch.randn((K, n), generator=gen, device="cuda") for n in shape] for shape in shapes]
    scratch = torch.empty(1 << 24, device="cuda")
    odd = lambda x: torch.cat((x[:, :1], x), 1)[:, 1:]
    err = []
    for rows, common in ((odd, False), (lambda x: x, True)):
        products = [(rows(a), rows(b), torch.empty((a.shape[1], b.shape[1]), device="cuda")) for a, b in operands]
        assert (ctx.twist_weight_grads_raw(K, products, scratch, (1.0,) * len(shapes)) != (0, 0, 0)) == common
        torch.cuda.synchronize()
        want = [a.double().T @ b.double() for a, b in operands]
        err.append([float((out.double() - w).norm() / w.norm()) for (_, _, out), w in zip(products, want)])
    assert all(b <= 1.03 * a for a, b in zip(*err)), err


# the up projection with its activation: the projection's bits and the activation kernel's of them, on every tile and on the plain kernel, with and without the
# projection itself
@pytest.mark.parametrize("act", ["gelu_tanh", "relu"])
@pytest.mark.parametrize("bf16,M,N,K,tile", [(True, 33, 136, 72, (32, 32)), (True, 999, 1000, 200, (64, 64)), (True, 2100, 1544, 264, (128, 128)),
                                             (True, 8190, 776, 768, (256, 128)), (True, 4000, 3080, 264, (256, 256)), (True, 80, 130, 66, 0),
                                             (False, 80, 136, 72, 0), (False, 1000, 1543, 200, 0)])
def test_projection_with_its_activation(lib, act, bf16, M, N, K, tile):
    cfg = si.ModelCfg(d_model=64, n_heads=1, d_head=8, d_ff=N, act=act, dtype="bf16" if bf16 else "f32")
    ctx = lib.Context(lib.desc_from_cfg(cfg))
    assert not tile or ctx.twist_gemm_kernel(0, M, N, K)[:2] == tile
    gen = torch.Generator(device="cuda").manual_seed(M)
    dt = torch.bfloat16 if bf16 else torch.float32
    A, B = (torch.randn(s, generator=gen, device="cuda").to(dt) * 0.2 for s in ((M, K), (N, K)))
    want = torch.empty((M, N), dtype=dt, device="cuda")
    ctx.twist_gemm_raw(0, M, N, K, A, B, want)
    want_a, _ = ctx.twist_act_raw(want, N)
    kind = ctx.desc.act
    got, a = ctx.twist_gemm_act_raw(A, B, None, kind)
    _, only = ctx.twist_gemm_act_raw(A, B, None, kind, act_only=True)
    torch.cuda.synchronize()
    assert torch.equal(got, want) and torch.equal(a, want_a) and torch.equal(only, want_a)


# Weight gradients that share a launch, on every tile, whole and cut: edges of tiles in both directions, products of odd sizes (whose partial
# products leave the next product's unaligned), an empty one, a last part shorter than the others
@pytest.mark.parametrize("tile,cut,K,shapes", [
    ((32, 32), False, 100, [(33, 41), (70, 36), (131, 40), (8, 33)]), ((32, 32), True, 9000, [(33, 41), (70, 36), (131, 41), (8, 40)]),
    ((64, 64), False, 1100, [(520, 776), (776, 515), (264, 520), (515, 776)]), ((64, 64), True, 8100, [(260, 390), (264, 201), (100, 100)]),
    ((256, 128), False, 2000, [(2100, 1024), (0, 8), (1024, 2100), (3000, 1001)]), ((256, 128), True, 8200, [(768, 768), (768, 769), (576, 768), (768, 192)]),
    ((256, 256), False, 1500, [(2816, 2048), (5000, 2048), (3072, 2048), (2048, 1001)]),
    ((256, 256), True, 8200, [(768, 3072), (3000, 769), (2304, 768), (768, 775)])])
def test_weight_gradients_in_one_launch(lib, tile, cut, K, shapes):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG3))
    gen = torch.Generator(device="cuda").manual_seed(K)
    up = lambda n: (n + 7) // 8 * 8
    rows = lambda n: torch.randn((K, up(n)), generator=gen, device="cuda").bfloat16()[:, :n]
    alphas = (0.5, 1.0, 2.0, 1.0)
    scratch = torch.full((1 << 24,), float("nan"), device="cuda")
    bufs = [torch.full((M * N + 64,), float("nan"), device="cuda") for M, N in shapes]
    products = [(rows(M), rows(N), buf[:M * N].view(M, N)) for (M, N), buf in zip(shapes, bufs)]
    rows, cols, parts = ctx.twist_weight_grads_raw(K, products, scratch, alphas)
    torch.cuda.synchronize()
    assert (rows, cols) == tile and (parts > 1) == cut, (rows, cols, parts)
    for (a, b, out), buf, alpha in zip(products, bufs, alphas):
        want = alpha * (a.double().T @ b.double())
        # fp32 sums of K exact products: 2^-24 sqrt(K) at most; one left out or counted twice shows as 1 / sqrt(K)
        assert out.numel() == 0 or float(((out.double() - want).norm(dim=1) / want.norm(dim=1)).max()) <= 2.0 ** -24 * K ** 0.5
        assert torch.isnan(buf[out.numel():]).all()
    assert torch.isnan(scratch[parts * sum(M * N for M, N in shapes) if cut else 0:]).all()
    a, b, out = products[0]
    one_by_one = [(a[:, 1:], b, torch.empty((a.shape[1] - 1, b.shape[1]), device="cuda")), products[1]]     # rows that are not 16-byte aligned
    assert ctx.twist_weight_grads_raw(K, one_by_one, scratch, alphas) == (0, 0, 0)
    torch.cuda.synchronize()
    assert float((one_by_one[0][2].double() - 0.5 * a[:, 1:].double().T @ b.double()).norm() / out.double().norm()) <= 2.0 ** -24 * K ** 0.5


@pytest.mark.parametrize("tile,layout,M,N,K", [(32, 2, 132, 200, 1100), (32, 1, 131, 72, 2001), (64, 2, 1500, 1500, 2000), (64, 0, 1500, 1500, 1999), (128, 1, 1024, 768, 8003),
                                               (128, 2, 1023, 769, 8003)])
def test_cut_fp32_projection(lib, tile, layout, M, N, K):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG1))
    scratch = torch.full((1 << 24,), float("nan"), device="cuda")
    rows, _, parts = ctx.twist_gemm_kernel(layout, M, N, K, True, scratch.numel())
    assert rows == tile and parts > 1, (rows, parts)
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn((K, M) if layout == 2 else (M, K), generator=gen, device="cuda")
    B = torch.randn((N, K) if layout == 0 else (K, N), generator=gen, device="cuda")
    want = (A.double().T if layout == 2 else A.double()) @ (B.double().T if layout == 0 else B.double())
    buf = torch.full((M * N + 64,), float("nan"), device="cuda")
    out = buf[:M * N].view(M, N)
    ctx.twist_gemm_raw_cut(layout, M, N, K, A, B, out, scratch, alpha=0.5)
    torch.cuda.synchronize()
    rows = (out.double() - 0.5 * want).norm(dim=1) / (0.5 * want).norm(dim=1)
    # K products of one rounding each and K additions; a product left out shows as 1 / sqrt(K) >= 1e-2
    assert float(rows.max()) <= 2.0 ** -24 * (2 * K) ** 0.5
    assert torch.isnan(buf[M * N:]).all() and torch.isnan(scratch[parts * M * N:]).all()


# contractions of a few elements: the plain kernel up to 16 (TN: 8), the matrix instruction from there on
@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("K", [1, 8, 9, 16, 17])
def test_fp32_projection_of_a_short_contraction(lib, layout, K):
    ctx = lib.Context(lib.desc_from_cfg(si.CFG1))
    M, N = 2050, 2101
    assert (ctx.twist_gemm_kernel(layout, M, N, K, True)[0] == 0) == (K <= (8 if layout == 2 else 16))
    gen = torch.Generator(device="cuda").manual_seed(K)
    A = torch.randn((K, M) if layout == 2 else (M, K), generator=gen, device="cuda")
    B = torch.randn((N, K) if layout == 0 else (K, N), generator=gen, device="cuda")
    want = (A.double().T if layout == 2 else A.double()) @ (B.double().T if layout == 0 else B.double())
    out = torch.full((M, N), float("nan"), device="cuda")
    ctx.twist_gemm_raw(layout, M, N, K, A, B, out)
    torch.cuda.synchronize()
    # K products and K additions of one rounding each
    assert float((out.double() - want).norm() / want.norm()) <= 2.0 ** -24 * (2 * K) ** 0.5
