"""The GEMM for launches of few tiles: every tile shape and epilogue, ragged
rows, columns and K, against the fp64 formula, and the LayerNorm fold through
its producer and consumer forms."""
import numpy as np
import pytest

import oracle
from paper_2609_10018_amd import ffi, inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
BF16 = inputs.BF16
NAN = float("nan")


def _operands(M, N, K, lda, ldw, seed):
    """Rows of lda / ldw elements with NaN past K; exactly K (rounded up to 8)
    elements in the last row of the buffer."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    k8 = (K + 7) // 8 * 8
    out = []
    for rows, ld, std in ((M, lda, 1.0), (N, ldw, 0.1)):
        v = (torch.randn(rows, K, generator=g, device="cuda") * std).bfloat16()
        buf = torch.full(((rows - 1) * ld + k8,), NAN, device="cuda", dtype=torch.bfloat16)
        torch.as_strided(buf, (rows, K), (ld, 1)).copy_(v)
        out += [buf, v.double()]
    return out + [torch.randn(N, generator=g, device="cuda") * 0.1, g]


# 256 workgroups at most in one round: 16x32, 32x32, 32x64 and 64x64 tiles.
SHAPES = [(1, 8, 8, 8, 8), (1, 1000, 768, 768, 768), (17, 40, 64, 72, 64), (33, 72, 65, 72, 80),
          (197, 1152, 200, 200, 256), (197, 1536, 1030, 1032, 1032), (250, 2000, 96, 96, 96),
          (788, 1150, 391, 392, 392), (197, 768, 3072, 3072, 3072)]


@pytest.mark.parametrize("M,N,K,lda,ldw", SHAPES)
@pytest.mark.parametrize("epi", [ffi.EPI_BIAS, ffi.EPI_BIAS_GELU, ffi.EPI_BIAS_RESID,
                                 ffi.EPI_BIAS_F32OUT])
def test_small_linear(epi, M, N, K, lda, ldw):
    a, a64, w, w64, bias, g = _operands(M, N, K, lda, ldw, M + N + K)
    ldc = (N + 7) // 8 * 8 + 8
    dt = torch.float32 if epi == ffi.EPI_BIAS_F32OUT else torch.bfloat16
    c0 = torch.randn(M, ldc, generator=g, device="cuda").to(dt)
    c = c0.clone()
    ffi.op_linear(BF16, epi, a, lda, w, ldw, c, ldc, bias, M, N, K)
    z = a64 @ w64.t() + bias.double()
    if epi == ffi.EPI_BIAS_GELU:
        z = torch.from_numpy(oracle.gelu(z.cpu().numpy())).cuda()
    elif epi == ffi.EPI_BIAS_RESID:
        z = z + c0[:, :N].double()
    # fp32 sums of K products (bounded like a random walk by 2^-20 of their
    # size) and, for bf16 results, one rounding (2^-9) and GELU's 1e-4.
    scale = float(z.abs().max()) + K ** 0.5 * 0.1
    tol = scale * 2.0 ** -20 * 4 if dt == torch.float32 else scale * 2.0 ** -8 + 2e-4
    assert float((c[:, :N].double() - z).abs().max()) < tol
    assert torch.equal(c[:, N:], c0[:, N:])


def test_a_row_does_not_depend_on_the_tile_shape():
    """The same rows in launches of 1, 64, 200 and 394 rows: the same bits."""
    N, K = 1152, 773
    a, _, w, _, bias, _ = _operands(394, N, K, 776, 776, 3)
    outs = []
    for M in (1, 64, 200, 394):
        c = torch.empty(M, N, device="cuda", dtype=torch.bfloat16)
        ffi.op_linear(BF16, ffi.EPI_BIAS, a, 776, w, 776, c, N, bias, M, N, K)
        outs.append(c)
    for c in outs[:-1]:
        assert torch.equal(c, outs[-1][:c.shape[0]])


@pytest.mark.parametrize("M,d,N,K,tokens", [(5, 64, 24, 40, 0), (197, 192, 100, 192, 197),
                                            (40, 200, 300, 72, 5), (197, 768, 1152, 384, 197),
                                            (700, 768, 512, 100, 7)])
def test_small_folded_layernorm(M, d, N, K, tokens):
    """x += A W^T + b with row statistics, then LN(x) V^T + c from x and them."""
    a, a64, w, w64, bias, g = _operands(M, d, K, (K + 7) // 8 * 8, (K + 7) // 8 * 8, M + d)
    x = torch.randn(M, d, generator=g, device="cuda").bfloat16()
    x64 = x.double()
    cls, c64 = None, None
    if tokens:
        cls = torch.randn((M + tokens - 1) // tokens, d, generator=g, device="cuda")
        c64 = cls.double()
        x64[::tokens] = c64
    ld = ((d + 63) // 64 + 1) // 2 * 2
    st = torch.full((M, ld, 2), NAN, device="cuda")
    k8 = (K + 7) // 8 * 8
    ffi.op_linear_ln(ffi.EPI_BIAS_RESID, a, k8, w, k8, x, d, bias, M, d, K, ld, stats_out=st,
                     C_cls=cls, tokens=max(tokens, 1))
    x64 = x64 + a64 @ w64.t() + bias.double()
    got = x.double()
    if tokens:
        assert float((cls.double() - x64[::tokens]).abs().max()) < 1e-4
    assert float((got - x64).abs().max()) < 2.0 ** -8 * float(x64.abs().max()) + 1e-4
    for j in range((d + 63) // 64):
        seg = x64[:, 64 * j:min(d, 64 * j + 64)]
        s = st[:, j].double()
        assert float((s[:, 0] - seg.sum(1)).abs().max()) < 1e-3
        m2 = ((seg - seg.mean(1, keepdim=True)) ** 2).sum(1)
        assert float(((s[:, 1] - m2) / m2.clamp(min=1e-3)).abs().max()) < 1e-3
    v = (torch.randn(N, d, generator=g, device="cuda") * 0.1).bfloat16()
    cb, col = torch.randn(N, generator=g, device="cuda"), v.double().sum(1).float()
    y = torch.empty(M, (N + 7) // 8 * 8, device="cuda", dtype=torch.bfloat16)
    ffi.op_linear_ln(ffi.EPI_BIAS, x, d, v, d, y, y.shape[1], cb, M, N, d, ld, stats_in=st,
                     colsum=col)
    mean = x64.mean(1, keepdim=True)
    u = (got - mean) / torch.sqrt(((x64 - mean) ** 2).mean(1, keepdim=True) + 1e-6)
    z = u @ v.double().t() + cb.double()
    assert float((y[:, :N].double() - z).abs().max()) < 2.0 ** -7 * float(z.abs().max())


@pytest.mark.parametrize("M,N,K,lda", [(1, 1, 1, 4), (16, 16, 32, 32), (17, 33, 70, 72),
                                       (40, 200, 131, 132), (197, 520, 384, 384)])
@pytest.mark.parametrize("epi", [ffi.EPI_BIAS, ffi.EPI_BIAS_GELU, ffi.EPI_BIAS_RESID])
def test_small_linear_f32(epi, M, N, K, lda):
    g = torch.Generator(device="cuda").manual_seed(M + N)
    A, W = (torch.randn(n, K, generator=g, device="cuda") for n in (M, N))
    bufs = []
    for v in (A, W):  # the last row ends with its K-th value
        b = torch.full(((v.shape[0] - 1) * lda + K,), NAN, device="cuda")
        torch.as_strided(b, v.shape, (lda, 1)).copy_(v)
        bufs.append(b)
    bias, c0 = torch.randn(N, generator=g, device="cuda"), torch.randn(M, N + 1, device="cuda")
    c = c0.clone()
    ffi.op_linear(inputs.FP32, epi, bufs[0], lda, bufs[1], lda, c, N + 1, bias, M, N, K)
    z = A.double() @ W.double().t() + bias.double()
    if epi == ffi.EPI_BIAS_GELU:
        z = torch.from_numpy(np.asarray(oracle.gelu(z.cpu().numpy()))).cuda()
    elif epi == ffi.EPI_BIAS_RESID:
        z = z + c0[:, :N].double()
    scale = float(z.abs().max()) + K ** 0.5
    assert float((c[:, :N].double() - z).abs().max()) < scale * 2.0 ** -20
    assert torch.equal(c[:, N], c0[:, N])


@pytest.mark.parametrize("M,N,K,ld", [(3000, 700, 40, 40), (3000, 700, 64, 64), (2500, 1000, 130, 136),
                                      (2050, 1030, 333, 336), (7289, 384, 691, 1536),
                                      (1576, 768, 1536, 1536)])
@pytest.mark.parametrize("epi", [ffi.EPI_BIAS, ffi.EPI_BIAS_GELU, ffi.EPI_BIAS_RESID,
                                 ffi.EPI_BIAS_F32OUT])
def test_linear_in_less_than_a_round_of_128_tiles(epi, M, N, K, ld):
    """Too large for 64x64 tiles in one round, fewer 128x128 tiles than CUs."""
    test_small_linear(epi, M, N, K, ld, ld)


@pytest.mark.parametrize("M,N,K,ld", [(4000, 2200, 200, 200), (3901, 2301, 72, 72), (4033, 2176, 1088, 1088)])
@pytest.mark.parametrize("epi", [ffi.EPI_BIAS, ffi.EPI_BIAS_GELU, ffi.EPI_BIAS_RESID])
def test_linear_in_192_row_tiles(epi, M, N, K, ld):
    """More 192x256 tiles than 256x256 ones in the same round."""
    test_small_linear(epi, M, N, K, ld, ld)


@pytest.mark.parametrize("M,d,N,K,tokens", [(4200, 2112, 2200, 1100, 197), (4001, 2240, 2184, 1090, 0)])
def test_folded_layernorm_in_192_row_tiles(M, d, N, K, tokens):
    test_small_folded_layernorm(M, d, N, K, tokens)


@pytest.mark.parametrize("M,N,K,ld", [(16500, 64, 64, 64), (16449, 40, 128, 136), (16500, 23, 100, 104),
                                      (20001, 64, 328, 328)])
@pytest.mark.parametrize("epi", [ffi.EPI_BIAS, ffi.EPI_BIAS_GELU, ffi.EPI_BIAS_RESID,
                                 ffi.EPI_BIAS_F32OUT])
def test_linear_of_few_columns(epi, M, N, K, ld):
    """At most 64 columns over more rows than one round of 64x64 tiles."""
    test_small_linear(epi, M, N, K, ld, ld)


@pytest.mark.parametrize("K", [64, 72])
def test_folded_layernorm_of_few_columns(K):
    test_small_folded_layernorm(16500, 64, 56, K, 197)
