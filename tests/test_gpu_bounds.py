"""The bounds that the signature kernels decide by, against the hardware: the fp32
functions of the plane entries over every Philox word, and the sums of the
matrix instructions."""
import ctypes as C
import os

import numpy as np
import pytest
import torch

from gpu_util import down, up

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "libbounds.so")
    L = C.CDLL(path)   # (built with the library)
    L.entry_bound.restype = L.entry_unit.restype = C.c_float
    return L


def p(t):
    return C.c_void_p(t.data_ptr())


def test_approximate_entries(lib):
    """|g' - g| <= kFastErr, from the largest errors of its parts: the radius times the
    trigonometric part's, the radius's own, their product, and two roundings to fp32
    (of g' and of g) of values below 8."""
    out = torch.zeros(4, dtype=torch.float64, device="cuda")
    assert lib.entry_errors(p(out)) == 0
    radius, most, cosine, sine = out.tolist()
    trig = max(cosine, sine)
    bound = lib.entry_bound()
    print("radius off by %.3g (at most %.4f), cosine %.3g, sine %.3g; an entry by %.3g of %.3g"
          % (radius, most, cosine, sine, most * trig + radius + radius * trig + 2.0 ** -21, bound), flush=True)
    assert 0 < radius and 0 < cosine and 0 < sine
    assert (most + radius) * trig + radius + radius * trig + 2 * 2.0 ** -22 <= bound
    assert (most + radius) * lib.entry_unit() + 1 < 32768     # codes of 16 bits


def cases(rng, n, k):
    """Factors and addends: of one size, of sizes 2^-40 .. 1, sums that cancel, an addend
    far larger or smaller than the products."""
    a, b, c = rng.normal(size=(n, 32, k)), rng.normal(size=(n, k, 32)), rng.normal(size=(n, 32, 32))
    kind = np.arange(n) % 6
    spread = np.isin(kind, (1, 4))
    a[spread] *= 2.0 ** rng.integers(-20, 1, a[spread].shape)
    b[spread] *= 2.0 ** rng.integers(-20, 1, b[spread].shape)
    c[kind == 2] = 0
    c[kind == 3] *= 2.0 ** 12
    c[kind == 4] *= 2.0 ** -24
    return a, b, c, kind


def check(got, a, b, c, steps):
    exact = c + a @ b
    size = np.abs(c) + np.abs(a) @ np.abs(b)
    worst = (np.abs(got - exact) / np.where(size > 0, size, 1)).max()
    print("off by %.3g of the terms' sizes, allowed %.3g" % (worst, steps * 2.0 ** -23), flush=True)
    assert worst <= steps * 2.0 ** -23


def bf16(v):
    """(bits, values) of v rounded to bf16."""
    t = torch.from_numpy(v.astype(np.float32)).to(torch.bfloat16)
    return t.view(torch.int16).numpy().view(np.uint16), t.double().numpy()


def test_bf16_product_sums(lib):
    """k_srp_dense_filter's assumption: each of an instruction's 16 additions is off by
    at most 2^-23 of a partial sum, which the sizes of all terms bound."""
    rng, n = np.random.default_rng(1), 600
    a, b, c, kind = cases(rng, n, 16)
    (ab, a), (bb, b) = bf16(a), bf16(b)
    c[kind == 5] = -(a @ b)[kind == 5]
    c = c.astype(np.float32)
    D = torch.empty(n * 1024, device="cuda")
    da, db, dc = up(ab), up(bb), up(c)
    assert lib.product_bf16(p(da), p(db), p(dc), p(D), n) == 0
    check(down(D).reshape(n, 32, 32).astype(np.float64), a, b, c.astype(np.float64), 16)


def test_fp32_product_sums(lib):
    """The same of the chain's instruction and its 2 additions."""
    rng, n = np.random.default_rng(2), 600
    a, b, c, kind = cases(rng, n, 2)
    a, b = a.astype(np.float32), b.astype(np.float32)
    c[kind == 5] = -(a.astype(np.float64) @ b.astype(np.float64))[kind == 5]
    c = c.astype(np.float32)
    D = torch.empty(n * 1024, device="cuda")
    da, db, dc = up(a), up(b), up(c)
    assert lib.product_f32(p(da), p(db), p(dc), p(D), n) == 0
    check(down(D).reshape(n, 32, 32).astype(np.float64), a.astype(np.float64), b.astype(np.float64), c.astype(np.float64), 2)
