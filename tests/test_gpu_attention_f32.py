"""fp32 attention at the sizes where its key groups and loaders change, against
the fp64 formula."""
import math

import numpy as np
import pytest

from paper_2609_10018_amd import ffi, inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
FP32 = inputs.FP32


def _attend(qkv, B, T, h, hd, scale):
    x = qkv.astype(np.float64).reshape(B, T, -1)[..., :3 * h * hd].reshape(B, T, h, 3, hd)
    q, k, v = (x[:, :, :, i].transpose(0, 2, 1, 3) for i in range(3))
    s = q @ k.transpose(0, 1, 3, 2) * scale
    p = np.exp(s - s.max(axis=-1, keepdims=True))
    return ((p / p.sum(-1, keepdims=True)) @ v).transpose(0, 2, 1, 3).reshape(B * T, h * hd)


# A fp32 sum of n terms is off by at most n 2^-24 of the sum of their absolute
# values: (hd + T) 2^-24 <= 2.4e-5 of the largest output over these cases.
@pytest.mark.parametrize("B,T,h,hd,stride,off", [
    (2, 1, 1, 1, 3, 0),          # one key; one feature
    (1, 16, 2, 16, 96, 0),       # whole tiles, one wave with keys
    (2, 65, 3, 64, 576, 0),      # a key tile for a fifth wave turn
    (1, 257, 2, 64, 400, 0),     # a second group of keys: rescaled sums
    (1, 129, 2, 128, 768, 0),    # two key tiles a group (wide heads)
    (1, 140, 1, 100, 301, 1),    # odd rows from an unaligned pointer
    (3, 50, 2, 47, 290, 0),
    (2, 33, 2, 32, 193, 3),
    (1, 40, 1, 112, 336, 0),
])
def test_attention_f32(B, T, h, hd, stride, off):
    rng = np.random.default_rng(T + hd)
    qkv = rng.standard_normal((B * T, stride)).astype(np.float32)
    buf = torch.zeros(off + B * T * stride, device="cuda")
    buf[off:] = torch.from_numpy(qkv).cuda().reshape(-1)
    os_ = h * hd + 3
    out = torch.full((off + B * T * os_,), 7.0, device="cuda")
    ffi.op_attention(FP32, buf[off:], stride, out[off:], os_, B, T, h, hd, 1 / math.sqrt(hd))
    got = out[off:].reshape(B * T, os_).cpu().numpy()
    ref = _attend(qkv, B, T, h, hd, 1 / math.sqrt(hd))
    assert np.max(np.abs(got[:, :h * hd] - ref)) < 2.4e-5 * max(1.0, np.max(np.abs(ref)))
    assert (got[:, h * hd:] == 7.0).all()


def test_attention_f32_masked_and_missing_keys():
    """Keys with a score of -inf take no part, also where they are all of a
    wave's first group; a last token that holds infinities is not read for the
    missing keys of the tile's rest."""
    T, hd = 300, 64
    rng = np.random.default_rng(0)
    qkv = rng.standard_normal((T, 3 * hd)).astype(np.float32)
    qkv[:, 0] = 1.0
    ref_in = qkv.copy()
    qkv[:256, hd] = -np.inf                    # keys 0-255: score -inf
    keep = np.arange(256, T)
    q, k, v = ref_in[:, :hd], ref_in[keep, hd:2 * hd], ref_in[keep, 2 * hd:]
    s = q.astype(np.float64) @ k.T.astype(np.float64) / 8.0
    p = np.exp(s - s.max(1, keepdims=True))
    ref = p / p.sum(1, keepdims=True) @ v
    out = torch.empty(T, hd, device="cuda")
    ffi.op_attention(FP32, torch.from_numpy(qkv).cuda(), 3 * hd, out, hd, 1, T, 1, hd, 0.125)
    assert np.max(np.abs(out.cpu().numpy() - ref)) < 1e-5 * np.max(np.abs(ref))
    qkv = ref_in[:17].copy()
    qkv[16, 2 * hd:] = np.inf
    ffi.op_attention(FP32, torch.from_numpy(qkv).cuda(), 3 * hd, out, hd, 1, 17, 1, hd, 0.125)
    assert torch.isinf(out[:17]).all()
    qkv[:, hd] = -np.inf                       # no key left: 0 / 0
    ffi.op_attention(FP32, torch.from_numpy(qkv).cuda(), 3 * hd, out, hd, 1, 17, 1, hd, 0.125)
    assert torch.isnan(out[:17]).all()
