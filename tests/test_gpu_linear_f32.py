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
    (8200, 1030, 40, 40, 40, 1030, 0),       # 64x64 tiles, several rounds, ragged in every way
    (8200, 1030, 37, 39, 37, 1031, 0),
    (3100, 1030, 133, 136, 136, 1030, 0),    # 64x64 tiles, both LDS stages, a ragged last step
    (2000, 2010, 133, 136, 136, 2010, 0),    # 128x128 tiles (256 of them: the load of 1024 64x64)
    (2048, 2048, 160, 160, 160, 2048, 0),    # whole tiles and steps
    (1999, 2047, 101, 103, 101, 2049, 0),    # element loads
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
    # K roundings of 2^-24 of sums of at most about `scale`, in random directions
    # (sqrt(K) of them, and four times that for the largest of many), and the
    # epilogue's.
    scale = float(z.abs().max()) + K ** 0.5 * 0.1 + 1.0
    assert float((c[:, :N].double() - z).abs().max()) < (4 * K ** 0.5 + 4) * scale * 2.0 ** -24
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
