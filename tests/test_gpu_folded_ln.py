"""Kernel-level parity of the LayerNorm folded into the bf16 GEMMs (the
pre-norm LayerNorm of every block, Section 4.1), through
elasto_op_linear_ln:

* producer: the residual GEMM's per-row, per-64-column-segment statistics
  (sum, sum of squared deviations from the segment mean) against fp64 sums of
  the fp64 result, on rows whose mean is 0, 10, 100 and 1000 times their
  spread (trained ViTs carry large-mean channels in the residual stream);
* consumer: rstd * (A W'^T) - rstd * mean * colsum + bias' with W' = gamma (.)
  W, from exact statistics of the bf16 input, against the oracle's LayerNorm
  followed by the linear layer (and GELU), on rows whose mean is 0, 10 and
  100 times their spread.  The folded form subtracts rstd * mean * colsum
  from an fp32 product that carries the mean, so its error grows like
  2^-24 sqrt(K / 16) |mean| / spread (about 1e-3 at 100; at 1000, with the
  spread below the bf16 spacing of the mean, an fp32 emulation of the form
  is off by 17%): the range covered here is the range the form is for;
* both kernels' tile paths: launches large enough for the persistent kernel
  and its tail launch, and small ones.
"""
import numpy as np
import pytest

import oracle
from paper_2609_10018_amd import ffi, inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import dev, rel_err  # noqa: E402

# Consumer bar: the bf16 rounding of the output (2^-9 relative) and of the
# folded weights gamma (.) W (2^-9 relative each, summed over K at random
# signs) stay well below it.
CONSUMER_TOL = 1e-2
# Producer statistics are formed from the fp32 values of the result (each
# within ~1e-6 relative of the fp64 value): the sums to 1e-5 of the sum of
# magnitudes, the deviation sums to 1e-3 relative.
SUM_TOL = 1e-5
M2_TOL = 1e-3


def host(t):
    return t.float().cpu().numpy().astype(np.float64)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ffi.load_library()


def segment_stats(x, width):
    """fp64 (sum, sum of squared deviations) of each row's 64-column segments."""
    nseg = (width + 63) // 64
    out = np.zeros((x.shape[0], nseg, 2))
    for j in range(nseg):
        seg = x[:, 64 * j:min(64 * (j + 1), width)]
        m = seg.mean(axis=1, keepdims=True)
        out[:, j, 0] = seg.sum(axis=1)
        out[:, j, 1] = ((seg - m) ** 2).sum(axis=1)
    return out


def row_offsets(rng, M, ratio, spread):
    return (ratio * spread * rng.choice([-1.0, 1.0], size=(M, 1))
            * (1 + 0.1 * rng.standard_normal((M, 1))))


@pytest.mark.parametrize("M,N,K,tokens", [(24000, 768, 768, 197), (300, 768, 768, 0),
                                          (197, 576, 384, 197), (64, 136, 256, 0)])
@pytest.mark.parametrize("ratio", [0.0, 10.0, 100.0, 1000.0])
def test_producer_statistics(M, N, K, tokens, ratio):
    rng = np.random.default_rng(int(M + N + ratio))
    A = rng.standard_normal((M, K)).astype(np.float32)
    W = (rng.standard_normal((N, K)) * 0.05).astype(np.float32)
    bias = (0.1 * rng.standard_normal(N)).astype(np.float32)
    spread = 0.05 * np.sqrt(K)
    res = (row_offsets(rng, M, ratio, spread) + 0.5 * rng.standard_normal((M, N))).astype(np.float32)
    Ad, Wd, Cd = dev(A, torch.bfloat16), dev(W, torch.bfloat16), dev(res, torch.bfloat16)
    res_bf = host(Cd)
    ccls = None
    if tokens:
        ccls = dev(res[::tokens], torch.float32)   # class rows: fp32 residual
        res_bf[::tokens] = res[::tokens].astype(np.float64)
    ld = ((N + 63) // 64 + 1) // 2 * 2
    stats = torch.full((M, ld, 2), float("nan"), dtype=torch.float32, device="cuda")
    ffi.op_linear_ln(ffi.EPI_BIAS_RESID, Ad, K, Wd, K, Cd, N, dev(bias, torch.float32), M, N, K,
                     ld, stats_out=stats, C_cls=ccls, tokens=max(tokens, 1))
    torch.cuda.synchronize()
    z = res_bf + host(Ad) @ host(Wd).T + bias.astype(np.float64)
    exp = segment_stats(z, N)
    got = stats.cpu().numpy().astype(np.float64)[:, :exp.shape[1]]
    assert np.isfinite(got).all()
    mag = segment_stats(np.abs(z), N)[:, :, 0]
    sum_err = float(np.max(np.abs(got[:, :, 0] - exp[:, :, 0]) / mag))
    m2_err = float(np.max(np.abs(got[:, :, 1] - exp[:, :, 1]) / exp[:, :, 1]))
    print(f"M {M} N {N} ratio {ratio:g}: sum err {sum_err:.2e}, deviation-sum err {m2_err:.2e}")
    assert sum_err < SUM_TOL
    assert m2_err < M2_TOL
    # The output itself: residual + product (class rows in C_cls, fp32).
    out = host(Cd)
    if tokens:
        out[::tokens] = host(ccls)
    assert rel_err(out, z) < 2e-2


@pytest.mark.parametrize("M,N,K", [(24000, 2304, 768), (300, 768, 768), (197, 1152, 576),
                                   (100, 200, 144)])
@pytest.mark.parametrize("ratio", [0.0, 10.0, 100.0])
@pytest.mark.parametrize("epi", [ffi.EPI_BIAS, ffi.EPI_BIAS_GELU])
def test_consumer_matches_layernorm_then_linear(M, N, K, ratio, epi):
    rng = np.random.default_rng(int(M + N + K + ratio + epi))
    x = (row_offsets(rng, M, ratio, 1.0) + rng.standard_normal((M, K))).astype(np.float32)
    xb = inputs.bf16_round(x).astype(np.float64)
    g = 1 + 0.1 * rng.standard_normal(K)
    b = 0.1 * rng.standard_normal(K)
    W = inputs.bf16_round((rng.standard_normal((N, K)) * 0.05).astype(np.float32)).astype(np.float64)
    b1 = 0.1 * rng.standard_normal(N)
    Wf = inputs.bf16_round((W * g[None, :]).astype(np.float32)).astype(np.float64)
    colsum = Wf.sum(axis=1)
    biasf = b1 + W @ b
    ld = ((K + 63) // 64 + 1) // 2 * 2
    st = np.zeros((M, ld, 2))
    st[:, :(K + 63) // 64] = segment_stats(xb, K)
    C = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    ffi.op_linear_ln(epi, dev(xb, torch.bfloat16), K, dev(Wf, torch.bfloat16), K, C, N,
                     dev(biasf, torch.float32), M, N, K, ld, stats_in=dev(st, torch.float32),
                     colsum=dev(colsum, torch.float32), eps=1e-6)
    torch.cuda.synchronize()
    ref = oracle.layer_norm(xb, g, b, 1e-6) @ W.T + b1
    if epi == ffi.EPI_BIAS_GELU:
        ref = oracle.gelu(ref)
    err = rel_err(host(C), ref)
    print(f"M {M} N {N} K {K} ratio {ratio:g} epi {epi}: rel err {err:.2e}")
    assert err < CONSUMER_TOL


def test_linear_ln_argument_checks():
    A = torch.zeros((8, 64), dtype=torch.bfloat16, device="cuda")
    W = torch.zeros((8, 64), dtype=torch.bfloat16, device="cuda")
    C = torch.zeros((8, 8), dtype=torch.bfloat16, device="cuda")
    b = torch.zeros(8, dtype=torch.float32, device="cuda")
    st = torch.zeros((8, 2, 2), dtype=torch.float32, device="cuda")
    with pytest.raises(ffi.ElastoError):        # neither statistics pointer
        ffi.op_linear_ln(ffi.EPI_BIAS, A, 64, W, 64, C, 8, b, 8, 8, 64, 2)
    with pytest.raises(ffi.ElastoError):        # both
        ffi.op_linear_ln(ffi.EPI_BIAS, A, 64, W, 64, C, 8, b, 8, 8, 64, 2, stats_out=st,
                         stats_in=st, colsum=b)
    with pytest.raises(ffi.ElastoError):        # producer with a non-residual epilogue
        ffi.op_linear_ln(ffi.EPI_BIAS, A, 64, W, 64, C, 8, b, 8, 8, 64, 2, stats_out=st)
    with pytest.raises(ffi.ElastoError):        # consumer without column sums
        ffi.op_linear_ln(ffi.EPI_BIAS, A, 64, W, 64, C, 8, b, 8, 8, 64, 2, stats_in=st)
    with pytest.raises(ffi.ElastoError):        # odd stats_ld
        ffi.op_linear_ln(ffi.EPI_BIAS, A, 64, W, 64, C, 8, b, 8, 8, 64, 1, stats_in=st,
                         colsum=b)


def test_unwritten_statistics_slots_do_not_matter():
    """An odd number of segments leaves the last slot of a row unwritten: what
    memory happens to hold there (a NaN) is no part of the row's statistics."""
    M, d, N = 300, 192, 64
    g = torch.Generator(device="cuda").manual_seed(0)
    x = torch.randn(M, d, generator=g, device="cuda").bfloat16()
    v = (torch.randn(N, d, generator=g, device="cuda") * 0.1).bfloat16()
    seg = x.double().reshape(M, 3, 64)
    st = torch.full((M, 4, 2), float("nan"), device="cuda")
    st[:, :3, 0] = seg.sum(2).float()
    st[:, :3, 1] = ((seg - seg.mean(2, keepdim=True)) ** 2).sum(2).float()
    bias, col = torch.zeros(N, device="cuda"), v.double().sum(1).float()
    y = torch.empty(M, N, device="cuda", dtype=torch.bfloat16)
    ffi.op_linear_ln(ffi.EPI_BIAS, x, d, v, d, y, N, bias, M, N, d, 4, stats_in=st, colsum=col)
    u = torch.nn.functional.layer_norm(x.double(), (d,), eps=1e-6)
    z = u @ v.double().t()
    # bf16 rounding of the result and a folded product of 192 terms.
    assert float((y.double() - z).abs().max()) < 2.0 ** -7 * float(z.abs().max())
