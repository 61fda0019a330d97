"""Dense sign random projections: the filtered product (bf16 terms, error
bound, open signs settled in FP32) gives the plain FP32 product's bits."""
import numpy as np
import pytest
import torch

import paper_1110_1328_amd as P

from gpu_util import down

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def contexts():
    """A context that may use a workspace (filtered product) and one whose
    workspace is fixed too small for it (plain product)."""
    a, b = P.bayeslsh_create(0), P.bayeslsh_create(0)
    P.bayeslsh_reserve_workspace(b, 256, fixed=True)
    yield a, b
    a.close()
    b.close()


def bits_of(ctx, x, planes, n_bits, layout):
    out = torch.full((x.shape[0] * (n_bits // 32),), -1, dtype=torch.int32, device="cuda").view(torch.uint32)
    P.bayeslsh_srp_sigs(ctx, P.dense_vectors(x), planes, n_bits, 0, layout, out)
    P.bayeslsh_sync(ctx)
    w = down(out)
    w = w.reshape(x.shape[0], -1) if layout == P.OBJECT_MAJOR else w.reshape(-1, x.shape[0]).T
    return np.unpackbits(np.ascontiguousarray(w).view(np.uint8), axis=1, bitorder="little")


@pytest.mark.parametrize("dim,n_bits", [(32, 1024), (64, 576), (128, 512), (256, 512), (256, 2048)])
@pytest.mark.parametrize("rows", [1, 33, 129, 3000])
def test_filtered_bits_are_the_plain_bits(contexts, dim, n_bits, rows):
    """One row up to more blocks than the chip holds, every dim; rows and
    planes of zeros, infinities, NaN, near the ends of the float range, and a
    block of rows whose every sign is open (the overflowing list)."""
    print("dense SRP filter dim=%d n_bits=%d rows=%d" % (dim, n_bits, rows), flush=True)
    g = torch.Generator(device="cuda").manual_seed(dim * 7 + n_bits + rows)
    x = torch.randn(rows, dim, generator=g, device="cuda")
    planes = torch.randn(dim, n_bits, generator=g, device="cuda")
    if rows >= 33:
        x[0] = 0
        x[1, 3] = float("nan")
        x[2, 1], x[3, 5] = float("inf"), -float("inf")
        x[4] *= 1e-42      # denormal
        x[5] *= 1e-30
        x[6] *= 1e37
        x[7] = -x[8]
        x[9, 1:] *= 1e-12  # one element rules the norm
    if rows == 3000:
        x[64:96] = 0
        planes[:, 0] = 0
        planes[2, 1] = float("nan")
        planes[:, 2] *= 1e-25
        planes[:, 3] *= 1e30
        planes[:, 4] = planes[:, 5]
        planes[:, 40] = -planes[:, 41]
    for layout in (P.OBJECT_MAJOR, P.WORD_MAJOR):
        got = bits_of(contexts[0], x, planes, n_bits, layout)
        want = bits_of(contexts[1], x, planes, n_bits, layout)
        np.testing.assert_array_equal(got, want)
    assert P.bayeslsh_workspace_bytes(contexts[0]) > 256 == P.bayeslsh_workspace_bytes(contexts[1])
    # against 64 bits: a sign may differ only where the projection is within the
    # plain chain's own error, dim 2^-23 ||x|| ||r||
    proj = (x.double() @ planes.double()).cpu().numpy()
    scale = (x.double().norm(dim=1)[:, None] * planes.double().norm(dim=0)[None, :]).cpu().numpy()
    fine = np.isfinite(proj) & np.isfinite(scale) & (scale < 1e38) & (scale > 1e-30)
    wrong = (got != (proj >= 0)) & fine
    assert (np.abs(proj[wrong]) <= dim * 2.0 ** -23 * scale[wrong]).all()


def test_signs_near_zero(contexts):
    """Rows made nearly orthogonal to the first planes: projections within a
    few roundings of zero, where only the chain itself decides."""
    dim, n_bits, rows = 256, 512, 2048
    g = torch.Generator(device="cuda").manual_seed(11)
    planes = torch.randn(dim, n_bits, generator=g, device="cuda")
    x = torch.randn(rows, dim, generator=g, device="cuda")
    q, _ = torch.linalg.qr(planes[:, :64].double().cpu())
    q = q.cuda()
    x[: rows // 2] -= ((x[: rows // 2].double() @ q) @ q.T).float()
    got = bits_of(contexts[0], x, planes, n_bits, P.OBJECT_MAJOR)
    want = bits_of(contexts[1], x, planes, n_bits, P.OBJECT_MAJOR)
    np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("dim,n_bits", [(32, 1024), (64, 1024), (128, 512), (256, 512)])
def test_rows_and_planes_outside_the_filter(contexts, dim, n_bits):
    """Blocks with every wave, one wave or no wave past its list; rows of zeros
    against ordinary planes, planes of zeros, an infinite plane; norms at both ends of
    the range the bound covers; rows and planes whose products are mostly zeros."""
    print("dense SRP outside the filter dim=%d n_bits=%d" % (dim, n_bits), flush=True)
    rows = 128 * 9 + 37
    g = torch.Generator(device="cuda").manual_seed(dim + n_bits)
    x = torch.randn(rows, dim, generator=g, device="cuda")
    planes = torch.randn(dim, n_bits, generator=g, device="cuda")
    x[0:128] *= 1e-30                  # a block of such rows
    x[128 + 40] *= 1e-30               # one wave of a block
    x[256 + 3], x[256 + 70] = 0, float("inf")
    x[384:512] = 0
    x[512:640:2] = 0
    x[640:768] *= 2.0 ** torch.linspace(-78, -60, 128, device="cuda")[:, None]
    x[768:896] *= 2.0 ** torch.linspace(60, 78, 128, device="cuda")[:, None]
    x[896:1024] *= (torch.rand(128, dim, generator=g, device="cuda") < 0.03)
    x[-1] *= 1e-30                     # the last row of a short block
    planes[:, 7] = 0
    planes[3, 9] = float("inf")
    planes[:, 64:96] *= 2.0 ** torch.linspace(-30, -20, 32, device="cuda")
    planes[:, 96:128] *= 2.0 ** torch.linspace(40, 56, 32, device="cuda")
    planes[:, 128:256] *= (torch.rand(dim, 128, generator=g, device="cuda") < 0.1)
    for layout in (P.OBJECT_MAJOR, P.WORD_MAJOR):
        got = bits_of(contexts[0], x, planes, n_bits, layout)
        want = bits_of(contexts[1], x, planes, n_bits, layout)
        np.testing.assert_array_equal(got, want)
    assert (got[384:512, :7] == 1).all() and (got[1030:, 7] == 1).all()


def test_rows_outside_the_filter_cost_little_more_than_the_plain_product(contexts):
    """A row of zeros in every 32, rows of norms near the least float: no more than
    1.6 times the plain product, which a call of such rows takes after a look at them
    (settled sign by sign over 3 times)."""
    rows, dim, n_bits = 100_000, 256, 1024
    planes = torch.randn(dim, n_bits, device="cuda")
    base = torch.randn(rows, dim, device="cuda")
    zeros, tiny = base.clone(), base.clone()
    zeros[::32] = 0
    tiny[::32] *= 1e-30
    out = torch.empty(rows * n_bits // 32, dtype=torch.int32, device="cuda").view(torch.uint32)
    us = {}
    for name, ctx, x in (("plain", contexts[1], base), ("filtered", contexts[0], base), ("zeros", contexts[0], zeros),
                         ("tiny", contexts[0], tiny)):
        v = P.dense_vectors(x)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        runs = []
        for _ in range(6):
            a.record()
            P.bayeslsh_srp_sigs(ctx, v, planes, n_bits, 0, P.OBJECT_MAJOR, out)
            b.record()
            torch.cuda.synchronize()
            runs.append(a.elapsed_time(b) * 1e3)
        us[name] = min(runs)
    print("dense SRP: %s us" % us, flush=True)
    assert us["zeros"] < 1.6 * us["filtered"]
    assert us["tiny"] < 1.6 * us["plain"]
