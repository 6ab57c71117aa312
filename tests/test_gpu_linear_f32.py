"""fp32 linear layers at the sizes where their tiles and loaders change, against
the fp64 formula."""
import numpy as np
import pytest

import oracle
from paper_2609_10018_amd import ffi, inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
FP32 = inputs.FP32


@pytest.mark.parametrize("epi", [ffi.EPI_BIAS, ffi.EPI_BIAS_GELU, ffi.EPI_BIAS_RESID,
                                 ffi.EPI_BIAS_F32OUT])
@pytest.mark.parametrize("M,N,K,lda,ldw,ldc,off", [
    (1, 1, 1, 1, 1, 1, 0),
    (64, 64, 32, 32, 32, 64, 0),
    (65, 66, 33, 33, 34, 67, 0),             # odd strides: element loads
    (129, 63, 100, 100, 104, 64, 0),         # ragged last step after whole ones
    (130, 70, 96, 96, 96, 72, 1),            # unaligned A
    (8200, 1030, 40, 40, 40, 1030, 0),       # 128x128 tiles, ragged in every way
    (8200, 1030, 37, 39, 37, 1031, 0),
])
def test_linear_f32(epi, M, N, K, lda, ldw, ldc, off):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    nan = float("nan")
    # Exactly the rows' active prefixes lie in the buffers' last rows.
    a = torch.full((off + (M - 1) * lda + K,), nan, device="cuda")
    w = torch.full(((N - 1) * ldw + K,), nan, device="cuda")
    A, W = rnd(M, K), rnd(N, K) * 0.1
    torch.as_strided(a[off:], (M, K), (lda, 1)).copy_(A)
    torch.as_strided(w, (N, K), (ldw, 1)).copy_(W)
    bias, c0 = rnd(N), rnd(M, ldc)
    c = c0.clone()
    ffi.op_linear(FP32, epi, a[off:], lda, w, ldw, c, ldc, bias, M, N, K)
    z = A.double() @ W.double().t() + bias.double()
    if epi == ffi.EPI_BIAS_GELU:
        z = torch.from_numpy(oracle.gelu(z.cpu().numpy())).cuda()
    elif epi == ffi.EPI_BIAS_RESID:
        z = z + c0[:, :N].double()
    # A sum of K products of at most 5 x 0.5 and a bias, each rounded to 2^-24.
    assert float((c[:, :N].double() - z).abs().max()) < (2.5 * K + 10) * (K + 4) * 2.0 ** -24
    assert torch.equal(c[:, N:], c0[:, N:])


def test_patch_f32_forward_with_an_odd_patch():
    """The patch loader's element path: a patch of 6 pixels (no 16-byte runs)."""
    import dataclasses
    cfg = dataclasses.replace(inputs.CONFIGS["tiny"], img=30, patch=6)
    w = inputs.make_weights(cfg)
    t = inputs.make_dn_table(cfg, w)
    x = inputs.make_images(cfg, 3)
    vit = ffi.ElasticViT(cfg, w, t, 3)
    out = torch.empty(3, cfg.num_classes, device="cuda")
    for k in range(t.num_modes):
        vit.set_mode(k)
        vit.forward(torch.from_numpy(x).cuda(), out)
        ref = oracle.elastic_forward(w, cfg, t, k, x)
        assert np.max(np.abs(out.cpu().numpy() - ref)) < 1e-4 * np.max(np.abs(ref))
    vit.close()
