"""Per-kernel parity: every HIP kernel, called through the C boundary, against the CPU oracle on the same
seeded inputs.  Sizes span several tiles and ragged tails.  Bars (relative L2 per tensor): fp32 path 1e-4,
bf16 path 2e-2; where the arithmetic allows a much tighter bound the test uses it."""
import numpy as np
import pytest
import torch

from paper_2203_12533_amd import binding as pwb
from paper_2203_12533_amd import inputs as I
from gpu_util import DT, TOL, assert_close, dev_act, dev_f32, dev_i32, empty_act, host, ptr, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = pwb.Context(0)
    yield c
    c.close()


def _rand(seed, shape, std=1.0):
    return I.normal(seed, 77, int(np.prod(shape)), std).reshape(shape)


# ---- GEMM ---------------------------------------------------------------------------------------------

# (4096, 4096, K): 256 full 256x256 tiles, the ring-buffered kernel, with 1, 2 and 3 k-tiles of 64;
# (1024, 4096, K): 64 full tiles, (2048, 12288, K): 384 - rounds that leave much of the chip idle, on 128 x 128 tiles
GEMM_SHAPES = [(300, 200, 136), (512, 384, 256), (130, 72, 8), (4096, 4096, 128), (4072, 4088, 200), (4096, 4096, 64),
               (4096, 4096, 192), (1024, 4096, 192), (1024, 4096, 64), (2048, 12288, 128)]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("shape", GEMM_SHAPES)
def test_gemm_forward_layout_bias(ctx, orc, shape, bf16):
    """C = x[M,K] . W[K,N] + b: A row-major in k, B stored k-major (the forward projections)."""
    M, N, K = shape
    if not bf16 and M * N * K > 1e9:
        pytest.skip("fp32 ALU path is for the small configuration")
    x, xv = dev_act(_rand(1, (M, K)), bf16)
    w, wv = dev_act(_rand(2, (K, N), 0.05), bf16)
    b = _rand(3, (N,))
    bd = dev_f32(b)
    out = empty_act((M, N), bf16)
    ctx.gemm(dtype=DT[bf16], a_kmajor=0, b_kmajor=1, M=M, N=N, K=K, lda=K, ldb=N, ldc=N, epilogue=pwb.PW_EPI_BIAS,
             out_dtype=DT[bf16], accumulate=0, A=ptr(x), B=ptr(w), bias=ptr(bd), C=ptr(out))
    ctx.synchronize()
    ref = orc.linear_fwd(xv, wv, b.astype(np.float64))
    assert_close(host(out), ref, 4e-3 if bf16 else 2e-6)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("shape", GEMM_SHAPES[:3] + [(4096, 4096, 128), (4096, 4096, 64), (4096, 4096, 192), (1024, 4096, 192),
                                                    (2048, 12288, 64)])
def test_gemm_dgrad_and_wgrad_layouts(ctx, orc, shape, bf16):
    """dx = dy . W^T (B stored [n][k]) and dW = x^T . dy (both operands k-major), fp32 accumulate-into."""
    M, N, K = shape          # M tokens, N = in features, K = out features
    if not bf16 and M * N * K > 1e9:
        pytest.skip("fp32 ALU path is for the small configuration")
    if bf16 and (N % 8 or K % 8 or M % 8):
        pytest.skip("bf16 operands need 16-byte aligned rows")
    dy, dyv = dev_act(_rand(4, (M, K)), bf16)
    w, wv = dev_act(_rand(5, (N, K), 0.05), bf16)
    x, xv = dev_act(_rand(6, (M, N)), bf16)
    dx = empty_act((M, N), bf16)
    ctx.gemm(dtype=DT[bf16], a_kmajor=0, b_kmajor=0, M=M, N=N, K=K, lda=K, ldb=K, ldc=N, epilogue=pwb.PW_EPI_STORE,
             out_dtype=DT[bf16], accumulate=0, A=ptr(dy), B=ptr(w), C=ptr(dx))
    base = _rand(7, (N, K))
    dw = dev_f32(base)
    for acc in (1, 0):
        ctx.gemm(dtype=DT[bf16], a_kmajor=1, b_kmajor=1, M=N, N=K, K=M, lda=N, ldb=K, ldc=K,
                 epilogue=pwb.PW_EPI_STORE, out_dtype=pwb.PW_F32, accumulate=acc, A=ptr(x), B=ptr(dy), C=ptr(dw))
        ctx.synchronize()
        rdx, rdw, _ = orc.linear_bwd(xv, wv, dyv)
        want = rdw + base if acc else rdw
        assert_close(host(dw), want, 2e-6, acc)
    assert_close(host(dx), rdx, 4e-3 if bf16 else 2e-6)


# ragged, 64 full tiles (both on the any-shape kernel), 256 full tiles (ring kernel)
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("shape", [(264, 328, 192), (1024, 4096, 128), (4096, 4096, 128), (2048, 12288, 64)])
def test_gemm_fused_epilogues(ctx, orc, bf16, shape):
    M, N, K = shape
    if not bf16 and M * N * K > 1e8:
        pytest.skip("fp32 ALU path is for the small configuration")
    x, xv = dev_act(_rand(8, (M, K)), bf16)
    w, wv = dev_act(_rand(9, (K, N), 0.08), bf16)
    b = _rand(10, (N,), 0.5)
    bd = dev_f32(b)
    lin = orc.linear_fwd(xv, wv, b.astype(np.float64))
    common = dict(dtype=DT[bf16], a_kmajor=0, b_kmajor=1, M=M, N=N, K=K, lda=K, ldb=N, ldc=N, accumulate=0,
                  A=ptr(x), B=ptr(w))
    # bias + GELU, both the pre-activation and the activation are kept
    u, h = empty_act((M, N), bf16), empty_act((M, N), bf16)
    ctx.gemm(epilogue=pwb.PW_EPI_BIAS_GELU, out_dtype=DT[bf16], bias=ptr(bd), C=ptr(u), C2=ptr(h), **common)
    # bias + residual into the fp32 stream
    res = _rand(11, (M, N))
    resd, xo = dev_f32(res), torch.empty((M, N), dtype=torch.float32, device="cuda")
    ctx.gemm(epilogue=pwb.PW_EPI_BIAS_RESIDUAL, out_dtype=pwb.PW_F32, bias=ptr(bd), aux=ptr(resd), C=ptr(xo), **common)
    # product times gelu'(aux)
    pre, prev = dev_act(_rand(12, (M, N), 1.5), bf16)
    du = empty_act((M, N), bf16)
    ctx.gemm(epilogue=pwb.PW_EPI_GELU_BWD, out_dtype=DT[bf16], aux=ptr(pre), C=ptr(du), **common)
    ctx.synchronize()
    tol = 4e-3 if bf16 else 2e-6
    assert_close(host(u), lin, tol)
    assert_close(host(h), orc.gelu_fwd(lin), tol * 1.5)
    assert_close(host(xo), lin + res, 2e-6 if not bf16 else 1e-5)
    nobias = orc.linear_fwd(xv, wv)
    assert_close(host(du), orc.gelu_bwd(prev, nobias), tol)


# tiles of 32 x 32 (one of them, short k), 16 x 32 (the second shape) and, from 256 tiles of 64 x 64 on, 64 x 64; fewer rows than a
# fragment piece, one past a tile, k not a multiple of the 16-deep step and shorter than the four slices of it; rows of odd length
# (no alignment anywhere)
@pytest.mark.parametrize("a_k,b_k", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(1, 3, 5), (33, 65, 16), (31, 32, 130), (1025, 1021, 67), (3, 20000, 33)])
def test_gemm_fp32_edges_in_every_layout(ctx, M, N, K, a_k, b_k):
    a, b = _rand(21, (K, M + 1) if a_k else (M, K + 3)), _rand(22, (K, N + 1) if b_k else (N, K + 5))
    ad, bd, out = dev_f32(a), dev_f32(b), torch.full((M, N + 3), 7.0, device="cuda")
    ctx.gemm(dtype=pwb.PW_F32, a_kmajor=a_k, b_kmajor=b_k, M=M, N=N, K=K, lda=a.shape[1], ldb=b.shape[1], ldc=N + 3,
             epilogue=pwb.PW_EPI_STORE, out_dtype=pwb.PW_F32, accumulate=0, A=ptr(ad), B=ptr(bd), C=ptr(out))
    ctx.synchronize()
    a, b = a.astype(np.float64), b.astype(np.float64)
    ref = (a[:, :M].T if a_k else a[:, :K]) @ (b[:, :N] if b_k else b[:, :K].T)
    got = host(out)
    # fp32 sums of at most K products: K * 2^-24 relative to the sum of magnitudes bounds any order
    bound = (K + 4) * 2.0 ** -24 * ((np.abs(a[:, :M].T) if a_k else np.abs(a[:, :K])) @ (np.abs(b[:, :N]) if b_k else np.abs(b[:, :K].T)))
    assert (np.abs(got[:, :N] - ref) <= bound).all()
    assert (got[:, N:] == 7.0).all()


# tiles of 16 x 32 up to 128 tiles of 32 x 32 (the third shape: exactly; the fourth: a row of tiles more), edges of the lower tile
@pytest.mark.parametrize("a_k,b_k", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(16, 32, 64), (17, 31, 129), (512, 256, 83), (513, 256, 83), (47, 33, 1000)])
def test_gemm_fp32_low_tiles_in_every_layout(ctx, M, N, K, a_k, b_k):
    test_gemm_fp32_edges_in_every_layout(ctx, M, N, K, a_k, b_k)


# from 129 tiles of 32 x 32 on these: ragged rows and columns, k of less than one step, of one and of four and a bit, one row or column
@pytest.mark.parametrize("a_k,b_k", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(417, 389, 67), (417, 389, 5), (417, 389, 16), (1, 6000, 33), (6000, 1, 33)])
def test_gemm_fp32_square_tiles_in_every_layout(ctx, M, N, K, a_k, b_k):
    test_gemm_fp32_edges_in_every_layout(ctx, M, N, K, a_k, b_k)


# up to four tiles of 32 x 32 and a short k: on those tiles (one k later on 16 x 32), rows and columns that end inside them
@pytest.mark.parametrize("a_k,b_k", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (17, 20, 31), (32, 32, 256), (31, 32, 257), (33, 64, 160), (64, 35, 161), (97, 30, 100), (130, 31, 64)])
def test_gemm_fp32_of_a_few_tiles_in_every_layout(ctx, M, N, K, a_k, b_k):
    test_gemm_fp32_edges_in_every_layout(ctx, M, N, K, a_k, b_k)


# both operands k-major, rows that straddle cache lines, more than 2^20 values of both: tiles of 16 x 32 up to 140000 / (tiles of
# 32 x 32) steps of k (1400 here), from there on 32 x 32; 60000 / tiles past k = 4096
@pytest.mark.parametrize("M,N,K", [(130, 620, 1399), (130, 620, 1401), (41, 151, 5999), (41, 151, 6001)])
def test_gemm_fp32_of_long_kmajor_rows_that_straddle_lines(ctx, M, N, K):
    test_gemm_fp32_edges_in_every_layout(ctx, M, N, K, 1, 1)


# one size per tile shape of the any-shape kernel (64 x 64 and 128 x 64 tiles with k split over waves, 128 x 128 in both
# loop forms), ragged in every dimension, k from one partial step on; what lies behind the last k of a row is no number, and
# the last size has rows too far apart for 32-bit offsets
@pytest.mark.parametrize("a_k,b_k", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K,pad", [(8, 8, 8, 8), (1000, 776, 328, 8), (72, 40, 1288, 8), (1160, 1032, 72, 8), (1672, 1800, 200, 8),
                                       (2312, 2440, 136, 8), (2312, 2440, 2120, 8), (16, 24, 72, 1 << 23)])
def test_gemm_bf16_any_shape_in_every_layout(ctx, M, N, K, pad, a_k, b_k):
    if pad > 8 and (a_k or b_k):
        pytest.skip("72 rows of that length")

    def operand(seed, rows, cols):
        t = torch.full((rows, cols + pad), float("nan"), dtype=torch.bfloat16, device="cuda")
        v = I.round_to_bf16(_rand(seed, (rows, cols)))
        t[:, :cols] = torch.from_numpy(v).cuda().to(torch.bfloat16)
        return t, v.astype(np.float64)

    a, av = operand(23, K, M) if a_k else operand(23, M, K)
    b, bv = operand(24, K, N) if b_k else operand(24, N, K)
    ldc = (N + 7) // 8 * 8 + 8
    out = torch.full((M, ldc), 7.0, device="cuda")
    ctx.gemm(dtype=pwb.PW_BF16, a_kmajor=a_k, b_kmajor=b_k, M=M, N=N, K=K, lda=a.shape[1], ldb=b.shape[1], ldc=ldc,
             epilogue=pwb.PW_EPI_STORE, out_dtype=pwb.PW_F32, accumulate=0, A=ptr(a), B=ptr(b), C=ptr(out))
    ctx.synchronize()
    av, bv = av.T if a_k else av, bv if b_k else bv.T
    got = host(out)
    # the products are exact in fp32; fp32 sums of K of them, in any order
    assert (np.abs(got[:, :N] - av @ bv) <= (K + 4) * 2.0 ** -24 * (np.abs(av) @ np.abs(bv))).all()
    assert (got[:, N:] == 7.0).all()


# 210 ragged tiles of 128 x 128, four waves to each (with row-major operands and a plain output k goes over two groups from 1536 on)
@pytest.mark.parametrize("a_k,b_k", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("K", [248, 256, 264, 328, 448, 832, 904, 1096])
def test_gemm_bf16_two_groups_of_waves_in_every_layout(ctx, K, a_k, b_k):
    test_gemm_bf16_any_shape_in_every_layout(ctx, 1672, 1800, K, 8, a_k, b_k)


# the same tiles with k over two groups of four waves half a tile apart, whole tiles and (both operands row-major) ragged ones: one k tile
# more in the first group than in the second or as many, an even and an odd number of them, a partial last one; one k below the limit
@pytest.mark.parametrize("M,N,K,a_k,b_k", [(1664, 1792, K, a_k, b_k) for K in (2040, 2048, 2056, 2112, 2120, 2176, 2240) for a_k in (0, 1) for b_k in (0, 1)] +
                         [(1672, 1800, K, 0, 0) for K in (1528, 1536, 1544, 1600, 1664, 1672)] +
                         [(1672, 1800, K, a_k, b_k) for K in (4088, 4096, 4104) for a_k, b_k in ((0, 1), (1, 0), (1, 1))])
def test_gemm_bf16_two_groups_of_waves_with_a_long_k(ctx, M, N, K, a_k, b_k):
    test_gemm_bf16_any_shape_in_every_layout(ctx, M, N, K, 8, a_k, b_k)


# 128 x 64 tiles, k over two pairs of waves: in step up to twelve k tiles (the last of them partial or not), half a tile apart from there on
@pytest.mark.parametrize("a_k,b_k", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("K", [8, 64, 136, 712, 768, 776, 832, 896, 904])
def test_gemm_bf16_two_pairs_of_waves_in_every_layout(ctx, K, a_k, b_k):
    test_gemm_bf16_any_shape_in_every_layout(ctx, 1000, 1112, K, 8, a_k, b_k)


# 264 full tiles of 256 x 256, 2048 deep: a round of 256 on the ring kernel, the last columns (two tiles wide) on their own; and
# 160 of them 2056 deep and more (any-shape kernel) or 2112 (ring).  Every operand and output that goes by columns takes part.
@pytest.mark.parametrize("N,K", [(16896, 2048), (10240, 2056), (10240, 2112)])
@pytest.mark.parametrize("b_k", [0, 1])
def test_gemm_whose_last_columns_are_a_problem_of_their_own(ctx, N, K, b_k):
    _bf16_epilogues(ctx, 1024, N, K, b_k)


def _bf16_epilogues(ctx, M, N, K, b_k):
    g = torch.Generator(device="cuda").manual_seed(N + K + b_k)
    rn = lambda *s, std=1.0: torch.randn(*s, generator=g, device="cuda") * std  # noqa: E731
    x, w = rn(M, K).bfloat16(), rn(*((K, N) if b_k else (N, K)), std=0.02).bfloat16()
    bias, res, pre = rn(N), rn(M, N), rn(M, N).bfloat16()
    lin = x.float() @ (w.float() if b_k else w.float().T.contiguous())
    kw = dict(dtype=pwb.PW_BF16, a_kmajor=0, b_kmajor=b_k, M=M, N=N, K=K, lda=K, ldb=N if b_k else K, ldc=N, A=ptr(x), B=ptr(w))
    u, h, du = (torch.empty((M, N), dtype=torch.bfloat16, device="cuda") for _ in range(3))
    y, acc = torch.empty((M, N), device="cuda"), res.clone()
    torch.cuda.synchronize()
    ctx.gemm(epilogue=pwb.PW_EPI_BIAS_GELU, out_dtype=pwb.PW_BF16, accumulate=0, bias=ptr(bias), C=ptr(u), C2=ptr(h), **kw)
    ctx.gemm(epilogue=pwb.PW_EPI_BIAS_RESIDUAL, out_dtype=pwb.PW_F32, accumulate=0, bias=ptr(bias), aux=ptr(res), C=ptr(y), **kw)
    ctx.gemm(epilogue=pwb.PW_EPI_GELU_BWD, out_dtype=pwb.PW_BF16, accumulate=0, aux=ptr(pre), C=ptr(du), **kw)
    ctx.gemm(epilogue=pwb.PW_EPI_STORE, out_dtype=pwb.PW_F32, accumulate=1, C=ptr(acc), **kw)
    dw = torch.empty((K, N), device="cuda")          # both operands k-major: M rows of k, K x N outputs
    ctx.gemm(dtype=pwb.PW_BF16, a_kmajor=1, b_kmajor=1, M=K, N=N, K=M, lda=K, ldb=N, ldc=N, epilogue=pwb.PW_EPI_STORE, out_dtype=pwb.PW_F32,
             accumulate=0, A=ptr(x), B=ptr(pre), C=ptr(dw))
    ctx.synchronize()
    # (GELU and its slope in 64 bits: 1 + tanh cancels in 32, which is 1.7e-3 of a column of arguments around -4.6, 1.2e-2 around -5)
    leaf = pre.double().requires_grad_(True)
    slope = torch.autograd.grad(torch.nn.functional.gelu(leaf, approximate="tanh").sum(), leaf)[0].float()
    z = lin + bias
    gelu = torch.nn.functional.gelu(z.double(), approximate="tanh").float()
    # column by column, so that no part of the product can hide behind the rest: bf16 storage 2^-9, fp32 sums of K products
    for got, ref, tol in ((u, z, 4e-3), (h, gelu, 6e-3), (y, z + res, 1e-5), (du, lin * slope, 4e-3),
                          (acc, lin + res, 1e-5), (dw, x.float().T.contiguous() @ pre.float(), 1e-5)):
        err = (got.float() - ref).norm(dim=0) / ref.norm(dim=0)
        assert err.max().item() < tol


# every epilogue of the any-shape kernel, by tile shape (64 x 64, 128 x 64, 128 x 128), whole tiles and ragged rows and columns: a bias
# held over a tile's steps, old values and aux rows fetched ahead, a last vector of columns, fewer rows than a step covers
# (128 x 128 row-major ones of k over two groups from k = 256 on, ragged, and 1024, whole: one k on either side of both)
@pytest.mark.parametrize("M,N,K", [(256, 512, 128), (200, 264, 520), (1024, 1536, 264), (1000, 1112, 776), (1024, 3072, 1016), (1024, 3072, 1024),
                                   (1000, 3080, 248), (1000, 3080, 256), (1000, 3080, 264), (1672, 1800, 328), (1664, 2048, 2048),
                                   (2304, 2432, 128), (2312, 2440, 136)])
@pytest.mark.parametrize("b_k", [0, 1])
def test_gemm_bf16_epilogues_of_every_tile_shape(ctx, M, N, K, b_k):
    _bf16_epilogues(ctx, M, N, K, b_k)


@pytest.mark.parametrize("bf16", [False, True])
def test_gemm_pair_small_problems_and_rejection(ctx, orc, bf16):
    """Two problems that do not qualify for a shared launch still give both results; one bad argument set
    means neither runs."""
    (M0, N0, K0), (M1, N1, K1) = (136, 72, 64), (40, 264, 200)
    x0, x0v = dev_act(_rand(20, (M0, K0)), bf16)
    w0, w0v = dev_act(_rand(21, (K0, N0), 0.1), bf16)
    x1, x1v = dev_act(_rand(22, (M1, K1)), bf16)
    w1, w1v = dev_act(_rand(23, (K1, N1), 0.1), bf16)
    c0 = torch.full((M0, N0), 7.0, device="cuda")
    c1 = torch.full((M1, N1), 7.0, device="cuda")
    def args(x, w, c, M, N, K):
        return dict(dtype=DT[bf16], a_kmajor=0, b_kmajor=1, M=M, N=N, K=K, lda=K, ldb=N, ldc=N,
                    epilogue=pwb.PW_EPI_STORE, out_dtype=pwb.PW_F32, accumulate=0, A=ptr(x), B=ptr(w), C=ptr(c))
    with pytest.raises(pwb.PwError):
        ctx.gemm_pair(args(x0, w0, c0, M0, N0, K0), {**args(x1, w1, c1, M1, N1, K1), "ldb": 8})
    ctx.synchronize()
    assert (host(c0) == 7.0).all() and (host(c1) == 7.0).all()
    ctx.gemm_pair(args(x0, w0, c0, M0, N0, K0), args(x1, w1, c1, M1, N1, K1))
    ctx.synchronize()
    assert_close(host(c0), orc.linear_fwd(x0v, w0v), 2e-6)
    assert_close(host(c1), orc.linear_fwd(x1v, w1v), 2e-6)


# ---- fused epilogues of the step's two largest non-GEMM passes -------------------------------------------

def _adam_case(seed, n_in, n_out, ntok):
    x, xv = dev_act(_rand(seed, (ntok, n_in)), True)
    dy, dyv = dev_act(_rand(seed + 1, (ntok, n_out), 0.3), True)
    w = _rand(seed + 2, (n_in, n_out), 0.02).astype(np.float32)
    m = _rand(seed + 3, (n_in, n_out), 0.05).astype(np.float32)
    # second moments bounded away from zero: where v and g are both tiny the update is a quotient of two roundings
    v = ((0.05 + np.abs(_rand(seed + 4, (n_in, n_out), 0.05))) ** 2).astype(np.float32)
    return dict(x=x, xv=xv, dy=dy, dyv=dyv, w=w, m=m, v=v, wd=dev_f32(w), md=dev_f32(m), vd=dev_f32(v),
                wlp=torch.zeros((n_in, n_out), dtype=torch.bfloat16, device="cuda"),
                g=torch.full((n_in, n_out), float("nan"), device="cuda"), n_in=n_in, n_out=n_out, ntok=ntok)


def _adam_gemm_kw(c, hp, t, store_g):
    ep = pwb.AdamEpilogue(ptr(c["wd"]), ptr(c["md"]), ptr(c["vd"]), ptr(c["wlp"]), *hp, t)
    return dict(dtype=pwb.PW_BF16, a_kmajor=1, b_kmajor=1, M=c["n_in"], N=c["n_out"], K=c["ntok"], lda=c["n_in"],
                ldb=c["n_out"], ldc=c["n_out"], epilogue=pwb.PW_EPI_ADAM, out_dtype=pwb.PW_F32, accumulate=0,
                A=ptr(c["x"]), B=ptr(c["dy"]), C=ptr(c["g"]) if store_g else None, adam=ep)


def _check_adam_case(orc, c, hp, t, store_g):
    _, g, _ = orc.linear_bwd(c["xv"], np.zeros((c["n_in"], c["n_out"])), c["dyv"])
    rw, rm, rv = orc.adam(c["w"], c["m"], c["v"], g, *[np.float32(h) for h in hp], t)
    if store_g:
        assert_close(host(c["g"]), g, 2e-6, "g")
    assert_close(host(c["md"]), rm, 1e-5, "m")
    assert_close(host(c["vd"]), rv, 1e-5, "v")
    w64 = c["w"].astype(np.float64)
    # the update is small against w: compare it, and allow the fp32 storage of w on top
    assert_close(host(c["wd"]) - w64, rw - w64, 1e-4, "dw", norm_slack=1e-3, extra=np.abs(w64) * 1.2e-7)
    assert np.array_equal(c["wlp"].float().cpu().numpy(), I.round_to_bf16(c["wd"].cpu().numpy()))   # bf16 copy = RNE(w)


@pytest.mark.parametrize("t", [1, 3])
def test_gemm_with_adam_epilogue(ctx, orc, t):
    """dW = x^T . dy with the Adam update of W in the GEMM's epilogue (26 bytes of optimizer traffic per parameter,
    the gradient stored only on request): against the oracle's linear backward followed by the oracle's Adam."""
    hp = (1e-3, 0.9, 0.95, 1e-8)
    c = _adam_case(80, 2048, 5120, 192)                   # 160 tiles of 256 x 256: one launch of the ring kernel
    if t == 1:
        c["md"].zero_(), c["vd"].zero_()
        c["m"][:], c["v"][:] = 0, 0
    ctx.gemm(**_adam_gemm_kw(c, hp, t, store_g=True))
    ctx.synchronize()
    _check_adam_case(orc, c, hp, t, store_g=True)
    # without the gradient output, from the same state: same update
    c2 = _adam_case(80, 2048, 5120, 192)
    if t == 1:
        c2["md"].zero_(), c2["vd"].zero_()
        c2["m"][:], c2["v"][:] = 0, 0
    ctx.gemm(**_adam_gemm_kw(c2, hp, t, store_g=False))
    ctx.synchronize()
    for k in ("wd", "md", "vd", "wlp"):
        assert torch.equal(c[k], c2[k]), k
    assert torch.isnan(c2["g"]).all()


def test_gemm_group_with_adam_epilogues_and_bias_gradient(ctx, orc):
    """Two weight gradients sharing one launch (128 + 32 tiles), both with the Adam epilogue, one with the bias
    gradient riding along - the QKV / out-projection pair of a layer."""
    hp = (1e-3, 0.9, 0.95, 1e-8)
    a, b = _adam_case(90, 2048, 4096, 128), _adam_case(95, 2048, 1024, 128)
    dbias = torch.full((4096,), float("nan"), device="cuda")
    ctx.gemm_group([{**_adam_gemm_kw(a, hp, 2, True), "b_colsum": ptr(dbias)}, _adam_gemm_kw(b, hp, 2, False)])
    ctx.synchronize()
    _check_adam_case(orc, a, hp, 2, True)
    _check_adam_case(orc, b, hp, 2, False)
    assert_close(host(dbias), a["dyv"].sum(axis=0), 1e-5)
    # what the kernel cannot take is refused before anything runs: ragged shape, row-major operand, accumulate
    w0 = a["wd"].clone()
    for bad in (dict(M=2040, lda=2040), dict(a_kmajor=0), dict(accumulate=1)):
        with pytest.raises(pwb.PwError):
            ctx.gemm(**{**_adam_gemm_kw(a, hp, 2, True), **bad})
    ctx.synchronize()
    assert torch.equal(w0, a["wd"])


def test_profile_reports_the_launches_by_shape(ctx):
    """The measurement aid's per-shape table: three launches of one shape and one of another, bracketed by events."""
    x = torch.zeros(512 * 512, dtype=torch.bfloat16, device="cuda")
    c = torch.empty(512 * 512, dtype=torch.bfloat16, device="cuda")

    def run(K):
        ctx.gemm(dtype=pwb.PW_BF16, a_kmajor=0, b_kmajor=1, M=512, N=512, K=K, lda=K, ldb=512, ldc=512, accumulate=0,
                 epilogue=pwb.PW_EPI_STORE, out_dtype=pwb.PW_BF16, A=ptr(x), B=ptr(x), C=ptr(c))
    ctx.profile_begin()
    for K in (256, 512, 512, 512):
        run(K)
    n, ms, fl = ctx.profile_end()
    rows = ctx.profile_gemm_shapes()
    assert n == 4 and ms > 0 and fl == 2.0 * 512 * 512 * (256 + 3 * 512)
    assert sorted((r["K"], r["launches"]) for r in rows) == [(256, 1), (512, 3)]
    assert all(r["M"] == 512 and r["N"] == 512 and r["members"] == 1 and r["a_kmajor"] == 0 and r["b_kmajor"] == 1
               and r["epilogue"] == pwb.PW_EPI_STORE for r in rows)
    assert abs(sum(r["total_ms"] for r in rows) - ms) < 1e-6 * max(ms, 1.0) + 1e-9
    assert sum(r["total_flops"] for r in rows) == fl


def test_lm_head_fused_with_the_loss(ctx, orc):
    """The LM-head GEMM with the loss in its epilogue: a first pass over y . Wh leaves only softmax statistics per
    64-column group and the targets' logits, a second pass writes (softmax - onehot) / N in bf16 - the logits
    themselves are never stored.  Against the oracle's linear forward + softmax cross-entropy."""
    B, T, d, V = 4, 512, 256, 8192                        # 8 x 32 tiles
    N = B * T
    y, yv = dev_act(_rand(100, (N, d)), True)
    wh, whv = dev_act(_rand(101, (d, V), 0.08), True)
    tok = I.tokens(102, 1, (B, T + 1), V)
    tok[1, 5], tok[2, 7] = -3, V + 11                      # out-of-range ids are clamped, as everywhere
    tokd = dev_i32(tok)
    part = torch.full((N, V // 64, 2), float("nan"), device="cuda")
    zt, lse, rows, loss = (torch.full((n,), float("nan"), device="cuda") for n in (N, N, N, 1))
    dz = torch.full((N, V), float("nan"), dtype=torch.bfloat16, device="cuda")
    common = dict(dtype=pwb.PW_BF16, a_kmajor=0, b_kmajor=1, M=N, N=V, K=d, lda=d, ldb=V, ldc=V, accumulate=0,
                  A=ptr(y), B=ptr(wh))
    xe = pwb.XentEpilogue(ptr(tokd), T, ptr(part), ptr(zt), ptr(lse), 1.0 / N)
    ctx.gemm(epilogue=pwb.PW_EPI_XENT_STATS, out_dtype=pwb.PW_BF16, C=None, xent=xe, **common)
    ctx.op("xent_from_stats", ptr(part), ptr(zt), ptr(lse), ptr(rows), ptr(loss), N, V // 64)
    ctx.gemm(epilogue=pwb.PW_EPI_XENT_GRAD, out_dtype=pwb.PW_BF16, C=ptr(dz), xent=xe, **common)
    ctx.synchronize()
    z = orc.linear_fwd(yv, whv)
    tgt = np.clip(tok[:, 1:].reshape(-1), 0, V - 1)
    rl, rdz = orc.softmax_xent(z, tgt)
    zmax = z.max(axis=1)
    rlse = np.log(np.exp(z - zmax[:, None]).sum(axis=1)) + zmax
    assert abs(host(loss)[0] - rl) / rl < 1e-5
    assert_close(host(lse), rlse, 1e-5, "lse")
    assert_close(host(zt), z[np.arange(N), tgt], 1e-5, "target logits")
    assert_close(host(rows), rlse - z[np.arange(N), tgt], 1e-5, "row losses")
    assert_close(host(dz), rdz, 6e-3, "dz")
    with pytest.raises(pwb.PwError):                       # ragged vocabulary: refused, nothing runs
        ctx.gemm(epilogue=pwb.PW_EPI_XENT_STATS, out_dtype=pwb.PW_BF16, C=None, xent=xe, **{**common, "N": V - 8})


def test_gemm_rejects_what_the_kernel_cannot_take(ctx):
    a = torch.zeros(64 * 64, dtype=torch.bfloat16, device="cuda")
    c = torch.zeros(64 * 64, dtype=torch.float32, device="cuda")
    base = dict(dtype=pwb.PW_BF16, a_kmajor=0, b_kmajor=0, M=16, N=16, K=20, lda=20, ldb=20, ldc=16,
                epilogue=pwb.PW_EPI_STORE, out_dtype=pwb.PW_F32, accumulate=0, A=ptr(a), B=ptr(a), C=ptr(c))
    with pytest.raises(pwb.PwError):
        ctx.gemm(**base)                                   # K not a multiple of 8
    with pytest.raises(pwb.PwError):
        ctx.gemm(**{**base, "K": 16, "lda": 8, "ldb": 16})  # lda < K
    with pytest.raises(pwb.PwError):
        ctx.gemm(**{**base, "K": 16, "lda": 16, "ldb": 16, "A": ptr(a) + 2})   # misaligned
    with pytest.raises(pwb.PwError):
        ctx.gemm(**{**base, "K": 16, "lda": 16, "ldb": 16, "epilogue": pwb.PW_EPI_BIAS_RESIDUAL})   # no aux
    ctx.gemm(**{**base, "K": 16, "lda": 16, "ldb": 16, "M": 0})    # empty problem: accepted, nothing launched
    ctx.synchronize()


# ---- LayerNorm ----------------------------------------------------------------------------------------

@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("N,d", [(37, 256), (5, 1000), (600, 2048), (3, 8192), (2100, 2048), (1030, 512), (70, 4096)])
def test_layernorm_forward_backward(ctx, orc, N, d, bf16):
    x = _rand(20, (N, d), 2.0) + 0.5
    g, b = 1 + _rand(21, (d,), 0.1), _rand(22, (d,), 0.1)
    xd, gd, bd = dev_f32(x), dev_f32(g), dev_f32(b)
    y = empty_act((N, d), bf16)
    mean, rstd = torch.empty(N, device="cuda"), torch.empty(N, device="cuda")
    ctx.op("layernorm_fwd", DT[bf16], ptr(xd), ptr(gd), ptr(bd), ptr(y), ptr(mean), ptr(rstd), N, d)
    ry, rmean, rrstd = orc.layernorm_fwd(x, g, b)
    dy, dyv = dev_act(_rand(23, (N, d)), bf16)
    dres = _rand(24, (N, d))
    dresd = dev_f32(dres)
    dx = torch.empty((N, d), device="cuda")
    dxlp = empty_act((N, d), bf16) if bf16 else None
    dg, db, dsum = dev_f32(np.ones(d)), dev_f32(np.ones(d)), dev_f32(np.ones(d))
    ws = torch.empty(pwb.lib().pw_layernorm_bwd_ws_floats(N, d), device="cuda")
    ctx.op("layernorm_bwd", DT[bf16], ptr(dy), ptr(xd), ptr(gd), ptr(mean), ptr(rstd), ptr(dresd), ptr(dx), ptr(dxlp),
           ptr(dg), ptr(db), ptr(dsum), ptr(ws), N, d, 1)
    # without the residual input and the optional outputs, overwrite mode
    dx0, dg0, db0 = torch.empty((N, d), device="cuda"), dev_f32(np.ones(d)), dev_f32(np.ones(d))
    ctx.op("layernorm_bwd", DT[bf16], ptr(dy), ptr(xd), ptr(gd), ptr(mean), ptr(rstd), None, ptr(dx0), None,
           ptr(dg0), ptr(db0), None, ptr(ws), N, d, 0)
    ctx.synchronize()
    assert_close(host(y), ry, 4e-3 if bf16 else 2e-6)
    assert_close(host(mean), rmean, 1e-5)
    assert_close(host(rstd), rrstd, 1e-5)
    rdx, rdg, rdb = orc.layernorm_bwd(dyv, x, g)
    assert_close(host(dx), rdx + dres, 1e-5)
    assert_close(host(dg), rdg + 1.0, 1e-5)                                            # accumulate = 1 adds
    assert_close(host(db), rdb + 1.0, 1e-5)
    assert_close(host(dsum), (rdx + dres).sum(axis=0) + 1.0, 1e-5)                     # column sums of dx
    assert_close(host(dx0), rdx, 1e-5)
    assert_close(host(dg0), rdg, 1e-5)
    assert_close(host(db0), rdb, 1e-5)
    if bf16:
        assert_close(host(dxlp), rdx + dres, 4e-3)


# the block kernel's widths (256, 512 and 1024 threads, one and two pieces each), one column group past each, and row counts
# that make a block go round twice and end inside its last group of rows; every optional argument left out as well
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("N,d", [(1, 516), (2051, 1024), (2050, 1028), (6, 2052), (1031, 4096), (300, 4100), (2, 8188)])
def test_layernorm_backward_in_blocks_of_rows(ctx, bf16, N, d):
    x, g = _rand(81, (N, d)) + 0.3, 1.0 + _rand(82, (d,), 0.2)
    (dy, dyv), dres = dev_act(_rand(83, (N, d)), bf16), _rand(84, (N, d))
    xd, gd, rd = dev_f32(x), dev_f32(g), dev_f32(dres)
    mu = x.astype(np.float64).mean(1)
    rs = 1.0 / np.sqrt(x.astype(np.float64).var(1) + 1e-5)
    md, sd = dev_f32(mu), dev_f32(rs)
    ws = torch.empty(pwb.lib().pw_layernorm_bwd_ws_floats(N, d), device="cuda")
    xh = (x - mu[:, None]) * rs[:, None]
    gg = dyv * g
    base = rs[:, None] * (gg - gg.mean(1, keepdims=True) - xh * (gg * xh).mean(1, keepdims=True))
    for full in (True, False):
        dx, lp = torch.empty((N, d), device="cuda"), empty_act((N, d), bf16)
        dg, db, ds = (torch.full((d,), 2.0, device="cuda") for _ in range(3))
        ctx.op("layernorm_bwd", DT[bf16], ptr(dy), ptr(xd), ptr(gd), ptr(md), ptr(sd), ptr(rd) if full else None, ptr(dx),
               ptr(lp) if full else None, ptr(dg), ptr(db), ptr(ds) if full else None, ptr(ws), N, d, int(full))
        ctx.synchronize()
        want = base + dres if full else base
        assert_close(host(dx), want, 2e-6 * (1 + np.sqrt(d) / 64))
        assert_close(host(dg), (dyv * xh).sum(0) + 2.0 * full, 1e-5)
        assert_close(host(db), dyv.sum(0) + 2.0 * full, 1e-5)
        if full:
            assert_close(host(lp), want, 4e-3 if bf16 else 1e-5)
            assert_close(host(ds), want.sum(0) + 2.0, 1e-5)


# ---- attention ----------------------------------------------------------------------------------------

@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("B,T,H,hd", [(2, 200, 2, 64), (1, 130, 3, 128), (2, 1, 1, 64), (1, 384, 2, 128)])
def test_attention_forward_backward(ctx, orc, B, T, H, hd, bf16):
    d = H * hd
    qkv, qkvv = dev_act(_rand(30, (B * T, 3 * d), 1.0), bf16)
    o = empty_act((B * T, d), bf16)
    lse = torch.empty((B, H, T), device="cuda")
    ctx.op("attention_fwd", DT[bf16], ptr(qkv), ptr(o), ptr(lse), B, T, H, hd)
    ctx.synchronize()
    ro = orc.attention_fwd(qkvv, B, T, H, hd)
    assert_close(host(o), ro, 6e-3 if bf16 else 1e-5)
    # log-sum-exp of the scaled causal scores, brute force for a few rows
    r = qkvv.reshape(B, T, 3, H, hd)
    for (b, h, i) in [(0, 0, 0), (B - 1, H - 1, T - 1), (0, H - 1, T // 2)]:
        s = r[b, : i + 1, 1, h] @ r[b, i, 0, h] / np.sqrt(hd)
        want = np.log(np.exp(s - s.max()).sum()) + s.max()
        assert abs(host(lse)[b, h, i] - want) < (2e-2 if bf16 else 1e-4)
    dout, doutv = dev_act(_rand(31, (B * T, d)), bf16)
    dqkv = empty_act((B * T, 3 * d), bf16)
    delta = torch.empty((B, H, T), device="cuda")
    ctx.op("attention_bwd", DT[bf16], ptr(qkv), ptr(o), ptr(dout), ptr(lse), ptr(delta), ptr(dqkv), B, T, H, hd)
    ctx.synchronize()
    rd = orc.attention_bwd(qkvv, doutv, B, T, H, hd)
    got = host(dqkv)
    for name, sl in (("dq", slice(0, d)), ("dk", slice(d, 2 * d)), ("dv", slice(2 * d, 3 * d))):
        assert_close(got[:, sl], rd[:, sl], 1.5e-2 if bf16 else 1e-5, name)


def _mha_case(ctx, orc, bf16, B, Tq, Tk, H, hd, causal, packed_kv):
    """General attention against the oracle: q from its own array, k and v either packed [K|V] rows or separate."""
    d = H * hd
    es = 2 if bf16 else 4
    q, qv = dev_act(_rand(32, (B * Tq, d), 1.0), bf16)
    if packed_kv:
        kv, kvv = dev_act(_rand(33, (B * Tk, 2 * d), 1.0), bf16)
        kp, vp, ldkv, kh, vh = ptr(kv), ptr(kv) + d * es, 2 * d, kvv[:, :d], kvv[:, d:]
    else:
        k, kh = dev_act(_rand(33, (B * Tk, d), 1.0), bf16)
        v, vh = dev_act(_rand(34, (B * Tk, d), 1.0), bf16)
        kp, vp, ldkv = ptr(k), ptr(v), d
    a = pwb.MhaArgs(DT[bf16], ptr(q), kp, vp, d, ldkv, B, Tq, Tk, H, hd, int(causal))
    o, o_lo = empty_act((B * Tq, d), bf16), empty_act((B * Tq, d), bf16)
    lse = torch.empty((B, H, Tq), device="cuda")
    ctx.mha_fwd(a, ptr(o), ptr(lse), o_lo=ptr(o_lo))
    ctx.synchronize()
    ro = orc.mha_fwd(qv, kh, vh, B, Tq, Tk, H, hd, causal=causal)
    # o_lo holds what rounding O left over (nothing in fp32); the sum is the kernel's fp32 result, itself exact only
    # as far as the bf16 probabilities of the second product allow
    assert_close(host(o) + host(o_lo), ro, 4e-3 if bf16 else 1e-5)
    assert np.abs(host(o_lo)).max() <= (np.abs(host(o)).max() * 2.0 ** -8 if bf16 else 0.0)
    assert_close(host(o), ro, 6e-3 if bf16 else 1e-5)
    qr, kr = qv.reshape(B, Tq, H, hd), np.ascontiguousarray(kh).reshape(B, Tk, H, hd)
    for (b, h, i) in [(0, 0, 0), (B - 1, H - 1, Tq - 1), (0, H - 1, Tq // 2)]:
        s = kr[b, : (i + 1 if causal else Tk), h] @ qr[b, i, h] / np.sqrt(hd)
        want = np.log(np.exp(s - s.max()).sum()) + s.max()
        assert abs(host(lse)[b, h, i] - want) < (2e-2 if bf16 else 1e-4)
    dout, doutv = dev_act(_rand(35, (B * Tq, d)), bf16)
    dq = empty_act((B * Tq, d), bf16)
    dkv = empty_act((B * Tk, 2 * d), bf16)             # gradients always packed [dK|dV] here
    delta = torch.empty((B, H, Tq), device="cuda")
    ctx.mha_bwd(a, ptr(o), ptr(dout), ptr(lse), ptr(delta), ptr(dq), d, ptr(dkv), ptr(dkv) + d * es, 2 * d, o_lo=ptr(o_lo))
    ctx.synchronize()
    rdq, rdk, rdv = orc.mha_bwd(qv, kh, vh, doutv, B, Tq, Tk, H, hd, causal=causal)
    tol = 1.5e-2 if bf16 else 1e-5
    assert_close(host(dq), rdq, tol)
    assert_close(host(dkv)[:, :d], rdk, tol)
    assert_close(host(dkv)[:, d:], rdv, tol)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("B,Tq,Tk,H,hd", [(2, 70, 200, 2, 64), (1, 130, 97, 3, 128), (2, 5, 1, 1, 64), (1, 300, 384, 2, 128),
                                          (2, 129, 64, 2, 128)])
def test_unmasked_attention_with_separate_lengths(ctx, orc, B, Tq, Tk, H, hd, bf16):
    _mha_case(ctx, orc, bf16, B, Tq, Tk, H, hd, causal=False, packed_kv=True)


def test_causal_attention_block_order_with_partial_problem_groups(ctx, orc):
    """Under the causal mask the workgroups of several problems are interleaved, longest blocks first: 9 problems of 5 blocks of 128
    rows, the last of them ragged, one more than there are XCDs (which orders there are: ..._block_orders)."""
    _mha_case(ctx, orc, True, 3, 520, 520, 3, 128, causal=True, packed_kv=False)


@pytest.mark.parametrize("bf16", [False, True])
def test_general_attention_entry_point_other_layouts(ctx, orc, bf16):
    _mha_case(ctx, orc, bf16, 2, 150, 150, 2, 128, causal=True, packed_kv=False)    # causal, k and v separate
    _mha_case(ctx, orc, bf16, 1, 96, 96, 2, 64, causal=False, packed_kv=False)      # encoder self-attention shape


def test_attention_output_remainder_keeps_query_gradient_accurate(ctx, orc):
    """Near-uniform attention over keys and values that share a large common component (what an encoder's output
    looks like at initialisation): delta = rowsum(dO * O) from the bf16-rounded O alone puts several per cent of
    error into dq and dk; with the rounding remainder kept by the forward call they meet the bf16 bar."""
    B, Tq, Tk, H, hd = 1, 256, 1024, 2, 128
    d = H * hd
    common = _rand(50, (1, 2 * d), 2.0)
    q, qv = dev_act(_rand(51, (B * Tq, d), 0.05), True)
    kv, kvv = dev_act(_rand(52, (B * Tk, 2 * d), 1.0) + common, True)
    dout, doutv = dev_act(_rand(53, (B * Tq, d)), True)
    a = pwb.MhaArgs(pwb.PW_BF16, ptr(q), ptr(kv), ptr(kv) + d * 2, d, 2 * d, B, Tq, Tk, H, hd, 0)
    rdq, rdk, rdv = orc.mha_bwd(qv, kvv[:, :d], kvv[:, d:], doutv, B, Tq, Tk, H, hd)
    errs = {}
    for keep in (False, True):
        o, o_lo = empty_act((B * Tq, d), True), empty_act((B * Tq, d), True)
        lse, delta = torch.empty((B, H, Tq), device="cuda"), torch.empty((B, H, Tq), device="cuda")
        dq, dkv = empty_act((B * Tq, d), True), empty_act((B * Tk, 2 * d), True)
        lo = ptr(o_lo) if keep else 0
        ctx.mha_fwd(a, ptr(o), ptr(lse), o_lo=lo)
        ctx.mha_bwd(a, ptr(o), ptr(dout), ptr(lse), ptr(delta), ptr(dq), d, ptr(dkv), ptr(dkv) + d * 2, 2 * d, o_lo=lo)
        ctx.synchronize()
        errs[keep] = (rel_l2(host(dq), rdq), rel_l2(host(dkv)[:, :d], rdk), rel_l2(host(dkv)[:, d:], rdv))
        if keep:   # with 1024 keys of similar weight the bf16 probabilities average out: o + o_lo is O to many more bits
            ro = orc.mha_fwd(qv, kvv[:, :d], kvv[:, d:], B, Tq, Tk, H, hd)
            assert rel_l2(host(o) + host(o_lo), ro) < 0.2 * rel_l2(host(o), ro)
    print("dq, dk, dv errors without / with the remainder:", errs[False], errs[True])
    assert max(errs[True]) < 1.5e-2
    for got, want, name in ((host(dq), rdq, "dq"), (host(dkv)[:, :d], rdk, "dk"), (host(dkv)[:, d:], rdv, "dv")):
        assert_close(got, want, 1.5e-2, name)          # the last pass of the loop kept the remainder
    assert errs[False][0] > 3 * errs[True][0]          # what the remainder is for


def test_general_attention_rejects_bad_arguments(ctx):
    q = torch.zeros((64, 128), device="cuda")
    lse = torch.zeros((1, 1, 64), device="cuda")
    ok = dict(dtype=pwb.PW_F32, q=ptr(q), k=ptr(q), v=ptr(q), ldq=128, ldkv=128, B=1, Tq=64, Tk=64, H=1, hd=128, causal=0)
    for bad in (dict(hd=96), dict(Tk=0), dict(ldkv=64), dict(causal=1, Tk=32), dict(k=0), dict(dtype=7)):
        a = pwb.MhaArgs(**{**ok, **bad})
        with pytest.raises(pwb.PwError):
            ctx.mha_fwd(a, ptr(q), ptr(lse))
    ctx.mha_fwd(pwb.MhaArgs(**ok), ptr(q), ptr(lse))
    ctx.synchronize()


@pytest.mark.parametrize("hd", [64, 128])
def test_packed_causal_bf16_attention_rejects_misaligned_arrays(ctx, hd):
    B, T, H = 1, 40, 2
    d = H * hd
    t = lambda n: torch.zeros(n + 8, dtype=torch.bfloat16, device="cuda")  # noqa: E731
    qkv, o, g, dqkv = t(B * T * 3 * d), t(B * T * d), t(B * T * d), t(B * T * 3 * d)
    lse, delta = torch.zeros((B, H, T), device="cuda"), torch.zeros((B, H, T), device="cuda")

    def fwd(i=0, j=0):
        ctx.op("attention_fwd", pwb.PW_BF16, ptr(qkv) + i, ptr(o) + j, ptr(lse), B, T, H, hd)

    def bwd(i=0, j=0, k=0, m=0):
        ctx.op("attention_bwd", pwb.PW_BF16, ptr(qkv) + i, ptr(o) + j, ptr(g) + k, ptr(lse), ptr(delta), ptr(dqkv) + m, B, T, H, hd)
    for off in (2, 8):
        for bad in (dict(i=off), dict(j=off)):
            with pytest.raises(pwb.PwError):
                fwd(**bad)
        for bad in (dict(i=off), dict(j=off), dict(k=off)):
            with pytest.raises(pwb.PwError):
                bwd(**bad)
    with pytest.raises(pwb.PwError):
        bwd(m=2)
    if hd == 64:
        with pytest.raises(pwb.PwError):
            bwd(m=8)
    else:
        bwd(m=8)                              # taken at this head width
    fwd()
    bwd()
    ctx.synchronize()


# query blocks of 128, key tiles of 64, 32-row MFMA blocks and one to either side of each; what the split of the
# probabilities leaves out at this head width (nothing forward, 2^-17 backward) is far below the rounding of the stored results
# (2^-9, uniform: 1.7e-3 in the norm)
@pytest.mark.parametrize("Tq,Tk,causal", [(1, 1, 0), (31, 65, 0), (32, 64, 0), (33, 63, 0), (129, 127, 0), (128, 257, 0), (96, 96, 1),
                                          (161, 161, 1)])
def test_bf16_attention_at_head_width_64_is_exact_up_to_its_storage(ctx, Tq, Tk, causal):
    B, H, hd = 2, 3, 64
    d = H * hd
    (q, qv), (kv, kvv), (go, gov) = (dev_act(_rand(s, shp), True) for s, shp in
                                     ((71, (B * Tq, d)), (72, (B * Tk, 2 * d)), (73, (B * Tq, d))))
    o, o_lo, dq, dkv = (empty_act(shp, True) for shp in ((B * Tq, d), (B * Tq, d), (B * Tq, d), (B * Tk, 2 * d)))
    lse, delta = torch.empty((B, H, Tq), device="cuda"), torch.empty((B, H, Tq), device="cuda")
    a = pwb.MhaArgs(pwb.PW_BF16, ptr(q), ptr(kv), ptr(kv) + 2 * d, d, 2 * d, B, Tq, Tk, H, hd, causal)
    ctx.mha_fwd(a, ptr(o), ptr(lse), ptr(o_lo))
    ctx.mha_bwd(a, ptr(o), ptr(go), ptr(lse), ptr(delta), ptr(dq), d, ptr(dkv), ptr(dkv) + 2 * d, 2 * d, ptr(o_lo))
    ctx.synchronize()
    heads = lambda t, T: np.moveaxis(t.reshape(B, T, H, hd), 2, 1)  # noqa: E731
    q_, k_, v_, g_ = heads(qv, Tq), heads(kvv[:, :d], Tk), heads(kvv[:, d:], Tk), heads(gov, Tq)
    s = q_ @ k_.swapaxes(2, 3) / 8.0
    if causal:
        s = np.where(np.tril(np.ones((Tq, Tk), bool)), s, -np.inf)
    m = s.max(-1, keepdims=True)
    p = np.exp(s - m)
    l = p.sum(-1, keepdims=True)
    p /= l
    ro = p @ v_
    ds = p * (g_ @ v_.swapaxes(2, 3) - (g_ * ro).sum(-1, keepdims=True)) / 8.0
    flat = lambda t: np.moveaxis(t, 1, 2).reshape(-1, d)  # noqa: E731
    assert np.abs(host(lse) - (m + np.log(l))[..., 0]).max() < 1e-5
    rk = flat(ds.swapaxes(2, 3) @ q_)
    for got, ref in ((host(o), flat(ro)), (host(dq), flat(ds @ k_)), (host(dkv)[:, :d], rk), (host(dkv)[:, d:], flat(p.swapaxes(2, 3) @ g_))):
        if Tk == 1 and ref is not None and not np.abs(ref).max() > 1e-12:
            assert np.abs(got).max() == 0.0      # one key: the score gradients are zero, exactly
        else:
            assert rel_l2(got, ref) < 2e-3
    assert rel_l2(host(o) + host(o_lo), flat(ro)) < 2e-5


# O and its remainder together hold 2^-18 of O; the sums behind them are fp32 ones, so nothing but that storage may show: the
# error of the pair is that of the exact O stored as such a pair (2.4e-6 in the norm), a tenth more for the sums' own 5e-7 or so.
@pytest.mark.parametrize("B,Tq,Tk,H,causal", [(2, 200, 300, 3, 0), (1, 64, 1000, 2, 0), (70, 33, 65, 4, 0), (2, 300, 300, 2, 1)])
def test_bf16_attention_at_head_width_64_keeps_fp32_sums_in_its_remainder(ctx, B, Tq, Tk, H, causal):
    hd = 64
    d = H * hd
    (q, qv), (kv, kvv) = (dev_act(_rand(s, shp), True) for s, shp in ((98, (B * Tq, d)), (99, (B * Tk, 2 * d))))
    o, o_lo, lse = empty_act((B * Tq, d), True), empty_act((B * Tq, d), True), torch.empty((B, H, Tq), device="cuda")
    ctx.mha_fwd(pwb.MhaArgs(pwb.PW_BF16, ptr(q), ptr(kv), ptr(kv) + 2 * d, d, 2 * d, B, Tq, Tk, H, hd, causal), ptr(o), ptr(lse), ptr(o_lo))
    ctx.synchronize()
    heads = lambda t, T: np.moveaxis(t.reshape(B, T, H, hd), 2, 1)  # noqa: E731
    s = heads(qv, Tq) @ heads(kvv[:, :d], Tk).swapaxes(2, 3) / 8.0
    if causal:
        s = np.where(np.tril(np.ones((Tq, Tk), bool)), s, -np.inf)
    p = np.exp(s - s.max(-1, keepdims=True))
    ro = np.moveaxis(p / p.sum(-1, keepdims=True) @ heads(kvv[:, d:], Tk), 1, 2).reshape(-1, d)
    hi = I.round_to_bf16(ro.astype(np.float32)).astype(np.float64)
    pair = hi + I.round_to_bf16((ro - hi).astype(np.float32)).astype(np.float64)
    assert rel_l2(host(o) + host(o_lo), ro) < 1.1 * rel_l2(pair, ro)


# bf16 blocks of 64 rows whose tiles two waves share (few blocks), and of 128 (many): one row to either side of a block, a
# tile and a wave's part of it; a second wave with nothing to do
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("B,Tq,Tk,H,causal", [(1, 64, 32, 1, 0), (1, 63, 65, 2, 0), (1, 65, 128, 2, 0), (2, 129, 193, 1, 0), (1, 33, 33, 1, 1),
                                              (1, 65, 65, 2, 1), (2, 128, 128, 1, 1), (1, 193, 193, 2, 1), (3, 400, 400, 8, 1),
                                              (40, 70, 100, 4, 0), (17, 130, 130, 8, 1), (33, 70, 130, 8, 0), (33, 65, 65, 8, 1)])
def test_bf16_attention_blocks_of_64_and_of_128_rows(ctx, orc, B, Tq, Tk, H, hd, causal):
    _mha_case(ctx, orc, True, B, Tq, Tk, H, hd, causal, packed_kv=True)


@pytest.mark.parametrize("B,Tq,Tk,H,causal", [(13, 65, 129, 5, 0), (13, 128, 130, 5, 0), (26, 97, 33, 5, 0), (13, 129, 129, 5, 1), (11, 300, 300, 4, 1),
                                              (26, 66, 66, 5, 1), (13, 192, 192, 5, 1)])
def test_bf16_attention_at_head_width_128_with_a_chip_full_of_key_blocks(ctx, orc, B, Tq, Tk, H, causal):
    """More than 128 blocks of 128 keys and more than one tile of 64 queries: two waves share 32 keys in dK/dV, each with its own
    half of every tile - whole and ragged tiles, a last tile with nothing in its second half, keys that fill no block."""
    _mha_case(ctx, orc, True, B, Tq, Tk, H, 128, causal=bool(causal), packed_kv=True)


# the order of a causal launch's blocks: by rank over all problems, with eight of them and one to either side, and numbers that eight does
# not divide; problem groups where fewer than eight are (7 of 16 blocks: groups of 4 and 3, in dK/dV of 2 and a last one of 1), or more than
# an L2 holds (at width 128 from 65536 rows of keys on, which 1008 problems of 65 stay below; 254 of 3 blocks: groups of 22 and a last one
# of 12, in dK/dV of 11 and a last one of 1)
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("B,T,H", [(1, 260, 7), (2, 200, 4), (3, 200, 3), (11, 140, 3), (1, 513, 13), (63, 65, 16), (64, 65, 16), (1, 1000, 7),
                                   (127, 260, 2)])
def test_bf16_causal_attention_block_orders(ctx, orc, B, T, H, hd):
    _mha_case(ctx, orc, True, B, T, T, H, hd, causal=True, packed_kv=True)


# dK/dV at head width 64, by blocks of 128 keys: unmasked two waves share 32 keys up to 128 of them, from 129 on in workgroups of eight
# waves; causal, with blocks of 64 that two waves share, a block per compute unit at most (208) and more (260), and one wave to 32 keys
@pytest.mark.parametrize("B,Tq,Tk,H,causal", [(32, 70, 40, 4, 0), (43, 200, 40, 3, 0), (64, 70, 40, 4, 0), (65, 200, 40, 4, 0),
                                              (65, 130, 130, 2, 1), (8, 775, 775, 2, 1), (10, 770, 770, 2, 1)])
def test_bf16_attention_gradients_at_head_width_64_around_a_block_per_unit(ctx, orc, B, Tq, Tk, H, causal):
    _mha_case(ctx, orc, True, B, Tq, Tk, H, 64, causal=bool(causal), packed_kv=True)


# the same for packed causal calls, whose probabilities and dS are rounded: two parts on 208 and 260 blocks, one wave to 32 keys on 136 and 260
@pytest.mark.parametrize("B,T,H", [(8, 775, 2), (10, 770, 2), (34, 130, 2), (65, 130, 2)])
def test_bf16_packed_causal_attention_at_head_width_64_around_a_block_per_unit(ctx, orc, B, T, H):
    test_attention_forward_backward(ctx, orc, B, T, H, 64, True)


# more than 128 blocks of 128 keys and a single tile of queries: four waves to 128 keys in dK/dV, at both ends of that tile (at head width
# 64 from 257 blocks on, one block to either side; up to there eight waves, half of them without queries up to 32)
@pytest.mark.parametrize("B,Tq,Tk,H,causal", [(40, 60, 100, 4, 0), (33, 64, 130, 8, 0), (33, 64, 64, 8, 1), (140, 1, 20, 1, 0)])
def test_bf16_attention_at_head_width_128_with_one_tile_of_queries(ctx, orc, B, Tq, Tk, H, causal):
    _mha_case(ctx, orc, True, B, Tq, Tk, H, 128, causal=bool(causal), packed_kv=True)


@pytest.mark.parametrize("B,Tq,Tk,H", [(40, 60, 100, 4), (140, 1, 20, 1), (43, 32, 130, 2), (43, 33, 130, 2), (64, 64, 100, 4), (257, 64, 100, 1),
                                       (257, 1, 30, 1), (70, 33, 130, 2), (257, 65, 100, 1)])
def test_bf16_attention_at_head_width_64_with_one_tile_of_queries(ctx, orc, B, Tq, Tk, H):
    _mha_case(ctx, orc, True, B, Tq, Tk, H, 64, causal=False, packed_kv=True)


# dK/dV where two waves share 32 keys, with keys that no query attends to (an infinite key): all of a wave's, some of it, all but one
# of a block's.  The gradients of the finite keys are what these alone give.
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("off", [range(32), range(40, 50), range(127), range(100, 150), range(1, 150)])
def test_bf16_attention_gradients_beside_keys_at_minus_infinity(ctx, orc, off, hd):
    B, Tq, Tk = 70, 70, 150
    q, k, v, g = (_rand(s, (B * t, hd)) for s, t in ((81, Tq), (82, Tk), (83, Tk), (84, Tq)))
    q[:, 0], gone = 1.0, np.zeros(Tk, bool)
    gone[list(off)] = True
    gone = np.tile(gone, B)
    (qt, qv), (kt, kv), (vt, vv), (gt, gv) = (dev_act(x, True) for x in (q, k, v, g))
    kt[torch.as_tensor(gone, device="cuda")] = 0.0
    kt[torch.as_tensor(gone, device="cuda"), 0] = -torch.inf
    o, dq, dk, dv = (empty_act(x.shape, True) for x in (q, q, k, v))
    lse, delta = torch.empty((B, 1, Tq), device="cuda"), torch.empty((B, 1, Tq), device="cuda")
    torch.cuda.synchronize()
    a = pwb.MhaArgs(pwb.PW_BF16, ptr(qt), ptr(kt), ptr(vt), hd, hd, B, Tq, Tk, 1, hd, 0)
    ctx.mha_fwd(a, ptr(o), ptr(lse))
    ctx.mha_bwd(a, ptr(o), ptr(gt), ptr(lse), ptr(delta), ptr(dq), hd, ptr(dk), ptr(dv), hd)
    ctx.synchronize()
    kept, n = (np.ascontiguousarray(x[~gone]) for x in (kv, vv)), int((~gone).sum()) // B
    _, rk, rv = orc.mha_bwd(qv, *kept, gv, B, Tq, n, 1, hd, causal=False)
    if n > 1:                                 # (one key: its score gradients are zero in exact arithmetic)
        assert_close(host(dk)[~gone], rk, 1.5e-2)
    assert_close(host(dv)[~gone], rv, 1.5e-2)


# keys that no query attends to (scores of -inf) in every tile of one wave's part, and all but the first of the other's
@pytest.mark.parametrize("hd", [64, 128])
def test_bf16_attention_with_scores_of_minus_infinity(ctx, orc, hd):
    B, Tq, Tk, H = 1, 50, 160, 1
    q, k, v = _rand(81, (Tq, hd), 1.0), _rand(82, (Tk, hd), 1.0), _rand(83, (Tk, hd), 1.0)
    q[:, 0], off = 1.0, np.arange(Tk) // 32 % 4 != 0
    (qt, qv), (kt, kv), (vt, vv) = (dev_act(x, True) for x in (q, k, v))
    kt[torch.as_tensor(off, device="cuda")] = 0.0
    kt[torch.as_tensor(off, device="cuda"), 0] = -torch.inf
    o, lse = empty_act((Tq, hd), True), torch.empty((B, H, Tq), device="cuda")
    torch.cuda.synchronize()
    ctx.mha_fwd(pwb.MhaArgs(pwb.PW_BF16, ptr(qt), ptr(kt), ptr(vt), hd, hd, B, Tq, Tk, H, hd, 0), ptr(o), ptr(lse))
    ctx.synchronize()
    ro = orc.mha_fwd(qv, np.ascontiguousarray(kv[~off]), np.ascontiguousarray(vv[~off]), B, Tq, int((~off).sum()), H, hd, causal=False)
    assert_close(host(o), ro, 6e-3)


# Keys that score -inf (an infinite key) and the finite ones between them, by the tiles and waves of each kernel.  Some key
# of every query is finite: its output is what the finite keys alone give.
def _minus_inf_case(ctx, orc, bf16, B, Tq, Tk, hd, off, lead=0):
    """lead: elements in front of every array, so that rows of bf16 start off the 16-byte grid."""
    q, k, v = _rand(81, (B * Tq, hd), 1.0), _rand(82, (B * Tk, hd), 1.0), _rand(83, (B * Tk, hd), 1.0)
    q[:, 0] = 1.0
    dt = torch.bfloat16 if bf16 else torch.float32

    def place(x):
        t = torch.zeros(lead + x.size, dtype=dt, device="cuda")
        t[lead:] = torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda().reshape(-1).to(dt)
        return t, t[lead:].float().cpu().numpy().reshape(x.shape).astype(np.float64)

    (qt, qv), (kt, kv), (vt, vv) = place(q), place(k), place(v)
    gone = torch.as_tensor(np.tile(off, B), device="cuda")
    kt[lead:].view(B * Tk, hd)[gone] = 0.0
    kt[lead:].view(B * Tk, hd)[gone, 0] = -torch.inf
    o, lse = torch.full((lead + B * Tq * hd,), 7.0, dtype=dt, device="cuda"), torch.empty((B, 1, Tq), device="cuda")
    at = lambda t: ptr(t) + lead * t.element_size()  # noqa: E731
    ctx.mha_fwd(pwb.MhaArgs(DT[bf16], at(qt), at(kt), at(vt), hd, hd, B, Tq, Tk, 1, hd, 0), at(o), ptr(lse))
    ctx.synchronize()
    keep = ~np.tile(off, B)
    ro = orc.mha_fwd(qv, np.ascontiguousarray(kv[keep]), np.ascontiguousarray(vv[keep]), B, Tq, int((~off).sum()), 1, hd, causal=False)
    assert_close(host(o[lead:]).reshape(B * Tq, hd), ro, 6e-3 if bf16 else 1e-5)
    s = np.einsum("bqd,bkd->bqk", qv.reshape(B, Tq, hd), kv.reshape(B, Tk, hd)[:, ~off]) / np.sqrt(hd)
    assert np.abs(host(lse)[:, 0] - np.log(np.exp(s).sum(-1))).max() < 1e-4


# the fp32 kernel's waves take every fourth tile of 16 keys: one wave's first tile, all of its tiles, all but one key; and the
# same kernel for bf16 rows that are not 16-byte aligned
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("off", [range(16, 32), range(16, 20), [j for j in range(150) if j // 16 % 4 == 2], range(1, 150), range(149)])
def test_fp32_attention_with_scores_of_minus_infinity(ctx, orc, off, hd, bf16):
    mask = np.zeros(150, bool)
    mask[list(off)] = True
    _minus_inf_case(ctx, orc, bf16, 2, 35, 150, hd, mask, lead=4 if bf16 else 0)


# the bf16 kernel of 128-row blocks (enough of them for it), tiles of 64 keys: the first tile, a later one, all but one key
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("off", [range(64), range(64, 128), range(100), range(149), range(1, 150)])
def test_bf16_attention_of_many_blocks_with_scores_of_minus_infinity(ctx, orc, off, hd):
    mask = np.zeros(150, bool)
    mask[list(off)] = True
    _minus_inf_case(ctx, orc, True, 260, 20, 150, hd, mask)


# one tile of 16 positions and one to either side, several tiles per wave; what a query may not see (or a key is not
# seen by) must not matter even where it is not a number
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("T", [2, 15, 16, 17, 83])
def test_fp32_causal_attention_ignores_what_is_masked(ctx, T, hd):
    B, H, d = 2, 2, 2 * hd
    qkv, dout = _rand(41, (B, T, 3 * d)), _rand(42, (B, T, d))

    def run(qkv, dout):
        qd, gd = dev_f32(qkv), dev_f32(dout)
        o, g, lse, delta = torch.empty_like(gd), torch.empty_like(qd), torch.empty((B, H, T), device="cuda"), torch.empty((B, H, T), device="cuda")
        ctx.op("attention_fwd", pwb.PW_F32, ptr(qd), ptr(o), ptr(lse), B, T, H, hd)
        ctx.op("attention_bwd", pwb.PW_F32, ptr(qd), ptr(o), ptr(gd), ptr(lse), ptr(delta), ptr(g), B, T, H, hd)
        ctx.synchronize()
        return host(o), host(g)

    q, k, v = (np.moveaxis(t.reshape(B, T, H, hd), 2, 1).astype(np.float64) for t in np.split(qkv, 3, axis=2))
    go = np.moveaxis(dout.reshape(B, T, H, hd), 2, 1).astype(np.float64)
    s = np.where(np.tril(np.ones((T, T), bool)), q @ k.swapaxes(2, 3) / np.sqrt(hd), -np.inf)
    p = np.exp(s - s.max(-1, keepdims=True))
    p /= p.sum(-1, keepdims=True)
    ro = p @ v
    ds = p * (go @ v.swapaxes(2, 3) - (go * ro).sum(-1, keepdims=True)) / np.sqrt(hd)
    flat = lambda t: np.moveaxis(t, 1, 2).reshape(B, T, d)  # noqa: E731
    ro, rq, rk, rv = flat(ro), flat(ds @ k), flat(ds.swapaxes(2, 3) @ q), flat(p.swapaxes(2, 3) @ go)
    o, g = run(qkv, dout)
    for got, ref in ((o, ro), (g[..., :d], rq), (g[..., d:2 * d], rk), (g[..., 2 * d:], rv)):
        assert_close(got, ref, 1e-5)
    bad = qkv.copy()
    bad[:, -1, d:] = np.nan                     # the last key and value: no earlier query sees them
    bad[:, -1, 2 * d:] = np.inf
    o, g = run(bad, dout)
    assert_close(o[:, :-1], ro[:, :-1], 1e-5)
    if T > 2:
        assert_close(g[:, 1:-1, :d], rq[:, 1:-1], 1e-5)
    bad, bad_g = qkv.copy(), dout.copy()
    bad[:, 0, :d] = np.nan                      # the first query and its output gradient: no later key is seen by it
    bad_g[:, 0] = np.inf
    o, g = run(bad, bad_g)
    assert_close(g[:, 1:, d:2 * d], rk[:, 1:], 1e-5)
    assert_close(g[:, 1:, 2 * d:], rv[:, 1:], 1e-5)


# The same for the bf16 kernels at head width 64: 32-row blocks on the diagonal and one position to either side, in workgroups
# of 64 rows (few) and of 128 (many), the hidden rows one and a third of all.  Packed calls, whose probabilities are rounded to
# bf16, hide such rows from other tiles (64 keys; in the dK/dV kernel 32 queries) only.
@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("B,T,H", [(2, 2, 2), (2, 31, 2), (2, 33, 2), (1, 64, 2), (1, 97, 2), (2, 200, 2), (33, 33, 4), (33, 100, 4), (17, 161, 4),
                                   (33, 161, 4), (10, 770, 2)])
def test_bf16_causal_attention_at_head_width_64_ignores_what_is_masked(ctx, B, T, H, packed):
    hd = 64
    d = H * hd
    qkv, dout = I.round_to_bf16(_rand(41, (B, T, 3 * d))), I.round_to_bf16(_rand(42, (B, T, d)))

    def run(qkv, dout):
        dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda().to(torch.bfloat16)  # noqa: E731
        qd, gd = dev(qkv), dev(dout)
        o, g, lse, delta = torch.empty_like(gd), torch.empty_like(qd), torch.empty((B, H, T), device="cuda"), torch.empty((B, H, T), device="cuda")
        if packed:
            ctx.op("attention_fwd", pwb.PW_BF16, ptr(qd), ptr(o), ptr(lse), B, T, H, hd)
            ctx.op("attention_bwd", pwb.PW_BF16, ptr(qd), ptr(o), ptr(gd), ptr(lse), ptr(delta), ptr(g), B, T, H, hd)
        else:
            q, kv, o_lo = qd[..., :d].contiguous(), qd[..., d:].contiguous(), torch.empty_like(gd)
            dq, dkv = torch.empty_like(q), torch.empty_like(kv)
            a = pwb.MhaArgs(pwb.PW_BF16, ptr(q), ptr(kv), ptr(kv) + 2 * d, d, 2 * d, B, T, T, H, hd, 1)
            ctx.mha_fwd(a, ptr(o), ptr(lse), ptr(o_lo))
            ctx.mha_bwd(a, ptr(o), ptr(gd), ptr(lse), ptr(delta), ptr(dq), d, ptr(dkv), ptr(dkv) + 2 * d, 2 * d, ptr(o_lo))
            ctx.synchronize()
            g = torch.cat([dq, dkv], 2)
        ctx.synchronize()
        return host(o), host(g)

    q, k, v = (np.moveaxis(t.reshape(B, T, H, hd), 2, 1).astype(np.float64) for t in np.split(qkv, 3, axis=2))
    go = np.moveaxis(dout.reshape(B, T, H, hd), 2, 1).astype(np.float64)
    s = np.where(np.tril(np.ones((T, T), bool)), q @ k.swapaxes(2, 3) / np.sqrt(hd), -np.inf)
    p = np.exp(s - s.max(-1, keepdims=True))
    p /= p.sum(-1, keepdims=True)
    ro = p @ v
    ds = p * (go @ v.swapaxes(2, 3) - (go * ro).sum(-1, keepdims=True)) / np.sqrt(hd)
    flat = lambda t: np.moveaxis(t, 1, 2).reshape(B, T, d)  # noqa: E731
    ro, rq, rk, rv = flat(ro), flat(ds @ k), flat(ds.swapaxes(2, 3) @ q), flat(p.swapaxes(2, 3) @ go)
    for n in sorted({1, T // 3} - {0}):
        bad = qkv.copy()
        bad[:, T - n:, d:2 * d] = np.nan            # the last keys and values: no earlier query sees them
        bad[:, T - n:, 2 * d:] = -np.inf
        o, g = run(bad, dout)
        end = (T - n) // 64 * 64 if packed else T - n
        if end > 0:
            assert_close(o[:, :end], ro[:, :end], 6e-3)
        if end > 1:
            assert_close(g[:, 1:end, :d], rq[:, 1:end], 1.5e-2)
        bad, bad_g = qkv.copy(), dout.copy()
        bad[:, :n, :d] = np.nan                     # the first queries and their output gradients: no later key is seen by them
        bad_g[:, :n] = np.inf
        o, g = run(bad, bad_g)
        assert_close(o[:, n:], ro[:, n:], 6e-3)
        first = (n + 31) // 32 * 32 if packed else n
        if first < T:
            assert_close(g[:, first:, d:2 * d], rk[:, first:], 1.5e-2)
            assert_close(g[:, first:, 2 * d:], rv[:, first:], 1.5e-2)


# infinities that are seen: they arrive as infinities, and once - not again for the rows behind the end of a sequence that ends
# inside a tile, nor as the difference of two parts of a probability
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("T", [5, 33, 70])
@pytest.mark.parametrize("packed", [True, False])
def test_bf16_attention_passes_infinite_values_on(ctx, T, hd, packed):
    q, k, v, g = (_rand(s, (T, hd)) for s in (91, 92, 93, 94))
    v[T - 1, 3], g[T - 1, 5] = np.inf, -np.inf
    qkv, qkvv = dev_act(np.concatenate([q, k, v], 1), True)
    gt, gv = dev_act(g, True)
    o, o_lo, dqkv = empty_act((T, hd), True), empty_act((T, hd), True), empty_act((T, 3 * hd), True)
    lse, delta = torch.empty((1, 1, T), device="cuda"), torch.empty((1, 1, T), device="cuda")
    at = lambda t, i: ptr(t) + 2 * hd * i  # noqa: E731
    a = pwb.MhaArgs(pwb.PW_BF16, at(qkv, 0), at(qkv, 1), at(qkv, 2), 3 * hd, 3 * hd, 1, T, T, 1, hd, int(packed))
    ctx.mha_fwd(a, ptr(o), ptr(lse), ptr(o_lo))
    ctx.mha_bwd(a, ptr(o), ptr(gt), ptr(lse), ptr(delta), at(dqkv, 0), 3 * hd, at(dqkv, 1), at(dqkv, 2), 3 * hd, ptr(o_lo))
    ctx.synchronize()
    qv, kv, vv = np.split(qkvv, 3, axis=1)
    s = qv @ kv.T / np.sqrt(hd)
    p = np.exp(np.where(np.tril(np.ones((T, T), bool)), s, -np.inf) if packed else s)
    p /= p.sum(1, keepdims=True)
    sees = slice(T - 1, T) if packed else slice(0, T)          # queries that see the last key; every key is seen by the last query
    for got, ref, col, inf in ((host(o)[sees], (p @ np.where(np.isfinite(vv), vv, 0.0))[sees], 3, np.inf),
                               (host(dqkv)[:, 2 * hd:], p.T @ np.where(np.isfinite(gv), gv, 0.0), 5, -np.inf)):
        assert (got[:, col] == inf).all()
        rest = np.arange(hd) != col
        assert_close(got[:, rest], ref[:, rest], 1.5e-2)


# the same on more than 128 blocks of keys (where two waves of eight share 32 keys in dK/dV: all but causal calls of width 64): queries that
# end inside a tile, in its first half and in its second
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("T", [70, 100])
@pytest.mark.parametrize("packed", [True, False])
def test_bf16_attention_of_many_blocks_passes_infinite_values_on(ctx, T, packed, hd):
    B = 130
    q, k, v, g = (_rand(s, (T, hd)) for s in (91, 92, 93, 94))
    v[T - 1, 3], g[T - 1, 5] = np.inf, -np.inf
    qkv, qkvv = dev_act(np.tile(np.concatenate([q, k, v], 1), (B, 1)), True)
    gt, gv = dev_act(np.tile(g, (B, 1)), True)
    o, o_lo, dqkv = empty_act((B * T, hd), True), empty_act((B * T, hd), True), empty_act((B * T, 3 * hd), True)
    lse, delta = torch.empty((B, 1, T), device="cuda"), torch.empty((B, 1, T), device="cuda")
    at = lambda t, i: ptr(t) + 2 * hd * i  # noqa: E731
    a = pwb.MhaArgs(pwb.PW_BF16, at(qkv, 0), at(qkv, 1), at(qkv, 2), 3 * hd, 3 * hd, B, T, T, 1, hd, int(packed))
    ctx.mha_fwd(a, ptr(o), ptr(lse), ptr(o_lo))
    ctx.mha_bwd(a, ptr(o), ptr(gt), ptr(lse), ptr(delta), at(dqkv, 0), 3 * hd, at(dqkv, 1), at(dqkv, 2), 3 * hd, ptr(o_lo))
    ctx.synchronize()
    qv, kv, _ = np.split(qkvv[:T], 3, axis=1)
    s = qv @ kv.T / np.sqrt(hd)
    p = np.exp(np.where(np.tril(np.ones((T, T), bool)), s, -np.inf) if packed else s)
    p /= p.sum(1, keepdims=True)
    got, ref = host(dqkv)[:, 2 * hd:], np.tile(p.T @ np.where(np.isfinite(gv[:T]), gv[:T], 0.0), (B, 1))
    assert (got[:, 5] == -np.inf).all()
    rest = np.arange(hd) != 5
    assert_close(got[:, rest], ref[:, rest], 1.5e-2)


# the widest rows that 32-bit offsets into tiles of 128 keys take, with a chip full of key blocks
@pytest.mark.parametrize("hd", [64, 128])
def test_bf16_attention_with_the_widest_rows_of_many_key_blocks(ctx, orc, hd):
    Tq, Tk, H, ld = 66, 130, 65, 1 << 24
    d = H * hd

    def far(x):
        t = torch.empty(((x.shape[0] - 1) * ld + x.shape[1],), dtype=torch.bfloat16, device="cuda")
        t.as_strided(x.shape, (ld, 1)).copy_(torch.from_numpy(x).cuda().to(torch.bfloat16))
        return t

    q, kv, g = (I.round_to_bf16(_rand(s, shp)) for s, shp in ((95, (Tq, d)), (96, (Tk, 2 * d)), (97, (Tq, d))))
    qt, kvt, (gt, _) = far(q), far(kv), dev_act(g, True)
    o, o_lo, dq, dkv = (empty_act(shp, True) for shp in ((Tq, d), (Tq, d), (Tq, d), (Tk, 2 * d)))
    lse, delta = torch.empty((1, H, Tq), device="cuda"), torch.empty((1, H, Tq), device="cuda")
    a = pwb.MhaArgs(pwb.PW_BF16, ptr(qt), ptr(kvt), ptr(kvt) + 2 * d, ld, ld, 1, Tq, Tk, H, hd, 0)
    torch.cuda.synchronize()
    ctx.mha_fwd(a, ptr(o), ptr(lse), ptr(o_lo))
    ctx.mha_bwd(a, ptr(o), ptr(gt), ptr(lse), ptr(delta), ptr(dq), d, ptr(dkv), ptr(dkv) + 2 * d, 2 * d, ptr(o_lo))
    ctx.synchronize()
    qv, kv_, gv = (np.ascontiguousarray(x, np.float64) for x in (q, kv, g))
    k, v = np.ascontiguousarray(kv_[:, :d]), np.ascontiguousarray(kv_[:, d:])
    assert_close(host(o), orc.mha_fwd(qv, k, v, 1, Tq, Tk, H, hd), 6e-3)
    for got, ref in zip((host(dq), host(dkv)[:, :d], host(dkv)[:, d:]), orc.mha_bwd(qv, k, v, gv, 1, Tq, Tk, H, hd)):
        assert_close(got, ref, 1.5e-2)
    del qt, kvt
    torch.cuda.empty_cache()                  # 6.6 GB


# rows too far apart for 32-bit byte offsets into a tile: keys and values from 2^32 / (2 * 127) elements on (tiles of up to 128
# rows), queries from 2^32 / (2 * 63) on (tiles of 64)
@pytest.mark.parametrize("hd", [64, 128])
def test_bf16_attention_with_rows_far_apart(ctx, orc, hd):
    Tq, Tk, ldq, ldkv = 66, 130, (1 << 25) + (1 << 20), (1 << 24) + (1 << 18)
    assert 63 * ldq * 2 >= 1 << 32 and 127 * ldkv * 2 >= 1 << 32

    def far(x, ld):
        t = torch.empty(((x.shape[0] - 1) * ld + x.shape[1],), dtype=torch.bfloat16, device="cuda")
        rows = t.as_strided(x.shape, (ld, 1))
        rows.copy_(torch.from_numpy(np.ascontiguousarray(x)).cuda().to(torch.bfloat16))
        return t, rows

    q, kv, g = (I.round_to_bf16(_rand(s, shp)) for s, shp in ((95, (Tq, hd)), (96, (Tk, 2 * hd)), (97, (Tq, hd))))
    (qt, _), (kvt, _), (gt, _) = far(q, ldq), far(kv, ldkv), dev_act(g, True)
    o, o_lo, dq, dkv = (empty_act(shp, True) for shp in ((Tq, hd), (Tq, hd), (Tq, hd), (Tk, 2 * hd)))
    lse, delta = torch.empty((1, 1, Tq), device="cuda"), torch.empty((1, 1, Tq), device="cuda")
    a = pwb.MhaArgs(pwb.PW_BF16, ptr(qt), ptr(kvt), ptr(kvt) + 2 * hd, ldq, ldkv, 1, Tq, Tk, 1, hd, 0)
    ctx.mha_fwd(a, ptr(o), ptr(lse), ptr(o_lo))
    ctx.mha_bwd(a, ptr(o), ptr(gt), ptr(lse), ptr(delta), ptr(dq), hd, ptr(dkv), ptr(dkv) + 2 * hd, 2 * hd, ptr(o_lo))
    ctx.synchronize()
    qv, kv_, gv = (np.ascontiguousarray(x, np.float64) for x in (q, kv, g))
    k, v = np.ascontiguousarray(kv_[:, :hd]), np.ascontiguousarray(kv_[:, hd:])
    assert_close(host(o), orc.mha_fwd(qv, k, v, 1, Tq, Tk, 1, hd), 6e-3)
    for got, ref in zip((host(dq), host(dkv)[:, :hd], host(dkv)[:, hd:]), orc.mha_bwd(qv, k, v, gv, 1, Tq, Tk, 1, hd)):
        assert_close(got, ref, 1.5e-2)
    del qt, kvt
    torch.cuda.empty_cache()                  # 13 GB


# ---- softmax cross-entropy ----------------------------------------------------------------------------

@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("B,T,V", [(3, 5, 1024), (2, 7, 4096), (1, 3, 32768), (2, 2, 8)])
def test_softmax_xent(ctx, orc, B, T, V, bf16):
    N = B * T
    z, zv = dev_act(_rand(40, (N, V), 2.0), bf16)
    tok = I.tokens(41, 1, (B, T + 1), V)
    tokd = dev_i32(tok)
    loss, rows = torch.empty(1, device="cuda"), torch.empty(N, device="cuda")
    ctx.op("softmax_xent", DT[bf16], ptr(z), ptr(tokd), ptr(loss), ptr(rows), B, T, V)
    ctx.synchronize()
    rl, rdz = orc.softmax_xent(zv, tok[:, 1:].reshape(-1))
    assert abs(host(loss)[0] - rl) / rl < 1e-5
    assert_close(host(z), rdz, 6e-3 if bf16 else 1e-5)
    if not bf16:
        assert np.abs(host(z).sum(axis=1)).max() < 1e-6     # rows of dlogits sum to 0


# rows held in registers in 1, 2, 4 and 8 pieces per thread, one column past each, and rows read twice
@pytest.mark.parametrize("bf16,V", [(True, 4096), (True, 4104), (True, 8200), (True, 16392), (True, 32776), (False, 2052),
                                    (False, 4100), (False, 8196), (False, 16388)])
def test_softmax_xent_at_every_row_length(ctx, orc, bf16, V):
    B, T = 2, 3
    z, zv = dev_act(_rand(61, (B * T, V), 2.0), bf16)
    tok = I.tokens(8, 6, (B, T + 1), V)
    tok[0, 1], tok[1, 3] = V - 1, 0
    td, loss, rows = dev_i32(tok), torch.empty(1, device="cuda"), torch.empty(B * T, device="cuda")
    ctx.op("softmax_xent", DT[bf16], ptr(z), ptr(td), ptr(loss), ptr(rows), B, T, V)
    ctx.synchronize()
    tgt = tok[:, 1:].reshape(-1)
    lse = np.log(np.exp(zv - zv.max(1, keepdims=True)).sum(1)) + zv.max(1)
    want = lse - zv[np.arange(B * T), tgt]
    dz = np.exp(zv - lse[:, None])
    dz[np.arange(B * T), tgt] -= 1.0
    assert np.abs(host(rows) - want).max() < 1e-5 * np.abs(want).max()
    assert abs(host(loss)[0] - want.mean()) < 1e-5 * want.mean()
    assert_close(host(z), dz / (B * T), 4e-3 if bf16 else 1e-5)


# ---- embedding ----------------------------------------------------------------------------------------

def test_embedding_forward_is_bit_exact_and_backward_is_deterministic(ctx, orc):
    B, T, d, V = 4, 129, 256, 97          # V small: many repeated ids
    tok = I.tokens(50, 1, (B, T + 1), V)
    tok[0, :40] = 5                        # one id repeated many times, in a row and across rows
    tok[1, 10:30] = 5
    wte, wpe = _rand(51, (V, d), 0.02), _rand(52, (T, d), 0.02)
    tokd, wted, wped = dev_i32(tok), dev_f32(wte), dev_f32(wpe)
    x = torch.empty((B * T, d), device="cuda")
    ctx.op("embedding_fwd", ptr(tokd), ptr(wted), ptr(wped), ptr(x), B, T, d, V)
    ctx.synchronize()
    inp = tok[:, :T]
    want = (wte[inp.reshape(-1)] + np.tile(wpe, (B, 1))).astype(np.float32)      # one fp32 add per element
    assert np.array_equal(x.cpu().numpy(), want)
    # the oracle adds in double, where the sum of two fp32 values is exact; rounded once it must give the same bits
    assert np.array_equal(x.cpu().numpy(), orc.embedding_fwd(inp, wte, wpe).astype(np.float32))
    dx = _rand(53, (B * T, d))
    dxd = dev_f32(dx)
    outs = []
    for _ in range(2):
        dwte = torch.full((V, d), 7.0, device="cuda")        # stale contents must be overwritten
        dwpe = torch.full((T, d), 7.0, device="cuda")
        ctx.op("embedding_bwd", ptr(tokd), ptr(dxd), ptr(dwte), ptr(dwpe), B, T, d, V)
        ctx.synchronize()
        outs.append((dwte.cpu().numpy(), dwpe.cpu().numpy()))
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
    rwte, rwpe = orc.embedding_bwd(inp, dx, V)
    assert_close(outs[0][0], rwte, 1e-6)
    assert_close(outs[0][1], rwpe, 1e-6)
    unused = sorted(set(range(V)) - set(inp.reshape(-1).tolist()))
    for u in unused:
        assert (outs[0][0][u] == 0).all()


def test_embedding_backward_handles_one_id_everywhere(ctx, orc):
    """Degenerate case: every position holds the same id (the list of matches exceeds one LDS batch)."""
    B, T, d, V = 3, 1000, 64, 11
    tok = np.full((B, T + 1), 4, dtype=np.int32)
    dx = _rand(54, (B * T, d))
    tokd, dxd = dev_i32(tok), dev_f32(dx)
    dwte, dwpe = torch.empty((V, d), device="cuda"), torch.empty((T, d), device="cuda")
    ctx.op("embedding_bwd", ptr(tokd), ptr(dxd), ptr(dwte), ptr(dwpe), B, T, d, V)
    ctx.synchronize()
    rwte, _ = orc.embedding_bwd(tok[:, :T], dx, V)
    assert_close(host(dwte), rwte, 1e-5)


# positions that fit an id's row of dwte and that do not (4 columns hold three), more of them than the list of one pass
# (2048), rows of one to eight pieces per thread, the smallest and a large table
@pytest.mark.parametrize("B,T,d,V", [(1, 1, 4, 1), (4, 1024, 4, 1), (2, 700, 8, 3), (3, 50, 1028, 40), (2, 300, 2048, 60),
                                     (1, 40, 4100, 7), (2, 33, 8192, 9), (2, 600, 64, 9000), (1, 1500, 260, 100)])
def test_embedding_backward_adds_rows_in_order_of_position(ctx, B, T, d, V):
    tok = I.tokens(7, 5, (B, T + 1), V)
    dx = _rand(51, (B, T, d))
    td, xd = dev_i32(tok), dev_f32(dx)
    dwte, dwpe = torch.full((V, d), 3.0, device="cuda"), torch.full((T, d), 3.0, device="cuda")
    ctx.op("embedding_bwd", ptr(td), ptr(xd), ptr(dwte), ptr(dwpe), B, T, d, V)
    ctx.synchronize()
    want, wpe = np.zeros((V, d), np.float32), np.zeros((T, d), np.float32)
    for b in range(B):
        for t in range(T):                     # fp32 additions one after the other: the same bits
            want[tok[b, t]] += dx[b, t]
        wpe += dx[b]
    assert np.array_equal(dwte.cpu().numpy(), want)
    assert np.array_equal(dwpe.cpu().numpy(), wpe)


# rows of every width of a group of threads; few ids, so that every block has several long rows: as many positions as are
# sorted side by side, row by row and looked up in order (by scan: 256 of a block and one more; gathered: what fits the row,
# a part of the list, n^2 against 128 N), one block for all ids, the last position that is scanned for and one more
@pytest.mark.parametrize("B,T,d,V", [(1, 256, 64, 5), (1, 257, 64, 5), (1, 300, 60, 1), (3, 600, 128, 40), (3, 701, 64, 33), (3, 701, 128, 9),
                                     (3, 701, 512, 9), (3, 701, 516, 6), (3, 701, 1024, 3), (2, 1500, 1024, 5), (1, 2048, 256, 700), (1, 2049, 256, 700),
                                     (2, 1100, 2052, 11), (1, 2300, 4, 3)])
def test_embedding_backward_of_few_ids_adds_rows_in_order_of_position(ctx, B, T, d, V):
    tok = I.tokens(9, 7, (B, T + 1), V)
    tok[:, ::3] = V // 2                           # one of them a third of all
    dx = _rand(55, (B, T, d))
    td, xd = dev_i32(tok), dev_f32(dx)
    dwte, dwpe = torch.full((V, d), 3.0, device="cuda"), torch.full((T, d), 3.0, device="cuda")
    ctx.op("embedding_bwd", ptr(td), ptr(xd), ptr(dwte), ptr(dwpe), B, T, d, V)
    ctx.synchronize()
    want, wpe = np.zeros((V, d), np.float32), np.zeros((T, d), np.float32)
    for b in range(B):
        for t in range(T):                         # fp32 additions one after the other: the same bits
            want[tok[b, t]] += dx[b, t]
        wpe += dx[b]
    assert np.array_equal(dwte.cpu().numpy(), want)
    assert np.array_equal(dwpe.cpu().numpy(), wpe)


# ---- column sums and optimisers -----------------------------------------------------------------------

@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("rows,cols", [(513, 768), (8, 64), (2048, 8192), (1, 12)])
def test_colsum(ctx, rows, cols, bf16):
    a, av = dev_act(_rand(60, (rows, cols)), bf16)
    out = dev_f32(np.full(cols, 3.0))
    ws = torch.empty(pwb.lib().pw_colsum_ws_floats(rows, cols), device="cuda")
    ctx.op("colsum", DT[bf16], ptr(a), ptr(out), ptr(ws), rows, cols, 1)
    ctx.synchronize()
    assert_close(host(out), av.sum(axis=0) + 3.0, 1e-5)
    ctx.op("colsum", DT[bf16], ptr(a), ptr(out), ptr(ws), rows, cols, 0)
    ctx.synchronize()
    assert_close(host(out), av.sum(axis=0), 1e-5)


@pytest.mark.parametrize("n", [1, 1023, 1 << 20])
def test_sgd_and_adam_kernels(ctx, orc, n):
    w, g = _rand(70, (n,)), _rand(71, (n,), 0.1)
    g[: n // 3] = 0.0
    wd, gd = dev_f32(w), dev_f32(g)
    ctx.op("sgd", ptr(wd), ptr(gd), n, 0.01)
    ctx.synchronize()
    assert_close(host(wd), orc.sgd(w.astype(np.float64), g.astype(np.float64), np.float32(0.01)), 1e-7)
    wd, md, vd = dev_f32(w), dev_f32(np.zeros(n)), dev_f32(np.zeros(n))
    wlp = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    rw, rm, rv = w.astype(np.float64), np.zeros(n), np.zeros(n)
    lr, b1, b2, eps = 1e-3, 0.9, 0.95, 1e-8
    for t in (1, 2, 3):
        ctx.op("adam", ptr(wd), ptr(md), ptr(vd), ptr(gd), ptr(wlp), n, lr, b1, b2, eps, t)
        rw, rm, rv = orc.adam(rw, rm, rv, g.astype(np.float64), np.float32(lr), np.float32(b1), np.float32(b2),
                              np.float32(eps), t)
    ctx.synchronize()
    assert np.abs(host(wd) - rw).max() < 1e-6            # identical gradient: the kernel itself is held to 1e-6
    assert_close(host(md), rm, 1e-6)
    assert_close(host(vd), rv, 1e-6)
    assert np.array_equal(wlp.float().cpu().numpy(), I.round_to_bf16(wd.cpu().numpy()))   # bf16 copy is RNE of w
