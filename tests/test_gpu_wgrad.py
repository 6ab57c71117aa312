"""The growth step's weight and bias gradients against the fp64 product, at the row
counts and column offsets where the kernel's splits, tiles and masks change.  The
step calls the launcher from C++ only, so it is called here by its symbol."""
import ctypes

import pytest

from paper_2609_10018_amd import ffi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
SYMBOL = "_ZN6elasto17launch_wgrad_bf16EPKNS_9WgradArgsEilPflS3_iP12ihipStream_t"
MAX, SLOTS, MAX_SPLIT = 4, 512, 32       # kWgradMax, kWgradSlots, kWgradMaxSplit
NAN, CANARY = float("nan"), 12345.0


class WgradArgs(ctypes.Structure):
    _fields_ = [("P", ctypes.c_void_p), ("Q", ctypes.c_void_p)] + \
        [(n, ctypes.c_int32) for n in ("ldp", "ldq", "pc", "qc", "ra", "rb")] + \
        [("out", ctypes.c_void_p), ("bias", ctypes.c_void_p)]


def _rows(M, ld, first, count, g):
    """M rows of ld bf16 values, NaN outside columns [first, first + count)."""
    x = torch.full((M, ld), NAN, device="cuda", dtype=torch.bfloat16)
    x[:, first:first + count] = torch.randn(M, count, generator=g, device="cuda").bfloat16()
    return x


# ldp, ldq, pc, qc, ra, rb, with bias: a layer's four problems.
ALIGNED = [(192, 768, 0, 576, 192, 192, False), (768, 192, 576, 0, 192, 192, True),
           (192, 192, 0, 128, 192, 64, False), (576, 192, 384, 0, 192, 192, True)]
UNALIGNED = [(128, 456, 0, 230, 128, 147, False), (456, 128, 230, 0, 147, 128, True),
             (264, 136, 135, 5, 129, 131, True), (16, 8, 7, 3, 1, 1, True)]
ONE = [(40, 1032, 3, 1, 33, 1030, True)]
EMPTY = [(192, 192, 0, 0, 0, 64, True), (64, 64, 1, 2, 60, 61, True), (192, 192, 0, 64, 192, 0, False)]


@pytest.mark.parametrize("M", [1, 63, 64, 197, 591, 1024, 3157, 6305, 12608])
@pytest.mark.parametrize("probs", [ALIGNED, UNALIGNED, ONE, EMPTY],
                         ids=["aligned", "unaligned", "one", "empty"])
def test_wgrad(M, probs):
    fn = getattr(ffi.load_library(), SYMBOL)
    P, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
    fn.argtypes, fn.restype = [P, i32, i64, P, i64, P, i32, P], i32
    g = torch.Generator(device="cuda").manual_seed(M)
    stride = max(p[4] for p in probs) + 3
    part = torch.full((SLOTS * 128 * 128,), NAN, device="cuda")
    bpart = torch.full((MAX_SPLIT * MAX * stride,), NAN, device="cuda")
    args, data = (WgradArgs * len(probs))(), []
    for a, (ldp, ldq, pc, qc, ra, rb, bias) in zip(args, probs):
        p, q = _rows(M, ldp, pc, ra, g), _rows(M, ldq, qc, rb, g)
        out = torch.full((ra * rb + 8,), CANARY, device="cuda")
        b = torch.full((ra + 8,), CANARY, device="cuda")
        (a.P, a.Q, a.ldp, a.ldq, a.pc, a.qc, a.ra, a.rb) = (p.data_ptr(), q.data_ptr(), ldp, ldq, pc,
                                                            qc, ra, rb)
        a.out, a.bias = out.data_ptr(), b.data_ptr() if bias else None
        data.append((p[:, pc:pc + ra].double(), q[:, qc:qc + rb].double(), out, b, p, q))
    stream = torch.cuda.current_stream().cuda_stream
    assert fn(args, len(probs), M, part.data_ptr(), part.numel(), bpart.data_ptr(), stride, stream) == 0
    torch.cuda.synchronize()
    # M products (exact in fp32) of N(0, 1) values: a sum of about sqrt(M), up to five
    # times that, rounded to 2^-24 M times in random directions.  A row of the M left
    # out or counted twice changes the sums by about 1.
    tol = 20.0 * (M + 16) * 2.0 ** -24
    assert tol < 0.05
    for (ldp, ldq, pc, qc, ra, rb, bias), (p, q, out, b, _, _) in zip(probs, data):
        if ra and rb:
            got = out[:ra * rb].reshape(ra, rb).double()
            assert float((got - p.t().contiguous() @ q).abs().max()) < tol
        if bias and ra and rb:
            assert float((b[:ra].double() - p.sum(0)).abs().max()) < tol
            assert bool((b[ra:] == CANARY).all())
        else:
            assert bool((b == CANARY).all())
        assert bool((out[ra * rb:] == CANARY).all())
