"""Sparse sign random projections: the bits are those of the FP64 sums whatever
decides most of them -- a table of codes, entries drawn per nonzero, masks in
one launch or several, or (no workspace) the sums alone."""
import numpy as np
import pytest
import torch

import paper_1110_1328_amd as P

from gpu_util import down, up

pytestmark = pytest.mark.gpu


def corpus(rng, n_rows, dim, odd):
    lens = rng.integers(1, 90, n_rows)
    if odd:
        lens[:8] = [0, 1, 2, 31, 32, 33, 64, 500]
    rows = [np.sort(rng.choice(dim, size=int(n), replace=False)) for n in lens]
    vals = [rng.normal(size=len(r)).astype(np.float32) for r in rows]
    if odd:
        rows[9][-1] = dim + 3          # past the dimension: drawn, never read from the table
        rows[10][:] = dim + np.arange(len(rows[10]))
        vals[11][:] = 0
        vals[12][0] = np.nan
        vals[13][0] = np.inf
        vals[14] *= np.float32(1e-42)
        vals[15] *= np.float32(1e35)
        rows[16], vals[16] = rows[16][:1], vals[16][:1]
        rows[17] = rows[7].copy()      # the same row twice, one negated, and a row that nearly cancels
        vals[17] = -vals[7]
        vals[18] = np.where(np.arange(len(vals[18])) % 2, 1, -1).astype(np.float32)
    off = np.zeros(n_rows + 1, np.int64)
    np.cumsum([len(r) for r in rows], out=off[1:])
    return off, np.concatenate(rows).astype(np.uint32), np.concatenate(vals).astype(np.float32)


def bits_of(ctx, vecs, n_rows, n_bits, layout, flags):
    out = torch.full((n_rows * (n_bits // 32),), -1, dtype=torch.int32, device="cuda").view(torch.uint32)
    P.bayeslsh_srp_sigs(ctx, vecs, None, n_bits, 0x1234_5678_9ABC, layout, out, flags=flags)
    P.bayeslsh_sync(ctx)
    w = down(out)
    return w.reshape(n_rows, -1) if layout == P.OBJECT_MAJOR else np.ascontiguousarray(w.reshape(-1, n_rows).T)


@pytest.mark.parametrize("n_bits", [32, 96, 256, 288, 544, 2048])
@pytest.mark.parametrize("flags", [0, P.SRP_PLANES_Q16])
def test_every_route_gives_the_same_bits(n_bits, flags):
    print("sparse SRP routes: %d bits flags %d" % (n_bits, flags), flush=True)
    rng = np.random.default_rng(n_bits + flags)
    n_rows, dim = 2100, 1500
    off, idx, val = corpus(rng, n_rows, dim, True)
    assert off[-1] > 2 * dim
    vecs = P.csr_vectors(up(off), up(idx), up(val), dim)
    got = {}
    mask_row = n_bits // 32 * 4
    # no workspace; masks of 1000 rows and no room for the table; everything
    for name, room in (("sums", 0), ("pieces", 1000 * mask_row), ("table", None)):
        ctx = P.bayeslsh_create(0)
        try:
            if room is not None:
                P.bayeslsh_reserve_workspace(ctx, room, fixed=True)
            for layout in (P.OBJECT_MAJOR, P.WORD_MAJOR):
                got[name, layout] = bits_of(ctx, vecs, n_rows, n_bits, layout, flags)
            if room is None:
                assert P.bayeslsh_workspace_bytes(ctx) >= dim * n_bits * 2
        finally:
            ctx.close()
    want = got["sums", P.OBJECT_MAJOR]
    for key, w in got.items():
        np.testing.assert_array_equal(w, want, err_msg=str(key))
    # an empty row and a row of zeros: every sum is 0, every bit 1
    assert (want[0] == 0xFFFFFFFF).all() and (want[11] == 0xFFFFFFFF).all()
    # a NaN in the row: no bit
    assert (want[12] == 0).all()


@pytest.mark.parametrize("n_rows", [1, 3, 4, 5, 33])
def test_few_rows(n_rows):
    """Blocks that are not full, against the sums alone."""
    rng = np.random.default_rng(n_rows)
    off, idx, val = corpus(rng, n_rows, 1 << 20, False)
    vecs = P.csr_vectors(up(off), up(idx), up(val), 1 << 20)
    a, b = P.bayeslsh_create(0), P.bayeslsh_create(0)
    try:
        P.bayeslsh_reserve_workspace(b, 0, fixed=True)
        for n_bits in (128, 160, 2048):
            np.testing.assert_array_equal(bits_of(a, vecs, n_rows, n_bits, P.OBJECT_MAJOR, 0),
                                          bits_of(b, vecs, n_rows, n_bits, P.OBJECT_MAJOR, 0))
    finally:
        a.close()
        b.close()


@pytest.mark.parametrize("flags", [0, P.SRP_PLANES_Q16])
@pytest.mark.parametrize("dim", [1 << 20, 512])     # entries drawn as they occur, the table
@pytest.mark.parametrize("nnz", [5, 10, 32])
def test_values_at_the_bottom_of_the_float_range(nnz, dim, flags):
    """Rows of +-2^e from the least denormal up: there a rounding is no longer a
    share of what is rounded, and the fp32 sums may decide only what is far
    above it."""
    n_rows, n_bits = 4096, 2048
    print("sparse SRP denormals: %d nonzeros dim %d flags %d" % (nnz, dim, flags), flush=True)
    rng = np.random.default_rng(nnz + flags)
    e = np.full(n_rows, -149)
    e[n_rows // 2:] = rng.integers(-149, -90, n_rows - n_rows // 2)
    val = (np.ldexp(1.0, e)[:, None] * rng.choice([-1.0, 1.0], (n_rows, nnz))).astype(np.float32)
    assert (val != 0).all()
    idx = np.argsort(rng.random((n_rows, 512)), axis=1)[:, :nnz] * (dim // 512)
    off = np.arange(n_rows + 1, dtype=np.int64) * nnz
    vecs = P.csr_vectors(up(off), up(np.sort(idx, axis=1).astype(np.uint32).reshape(-1)), up(val.reshape(-1)), dim)
    a, b = P.bayeslsh_create(0), P.bayeslsh_create(0)
    try:
        P.bayeslsh_reserve_workspace(b, 0, fixed=True)   # the sums alone
        got, want = (bits_of(c, vecs, n_rows, n_bits, P.OBJECT_MAJOR, flags) for c in (a, b))
        assert np.unpackbits((got ^ want).view(np.uint8)).sum() == 0
    finally:
        a.close()
        b.close()


def long_rows(rng, sizes, dim):
    """Rows of `sizes` sorted terms, weights of one size and of many."""
    rows = [np.sort(rng.permutation(dim)[:n]) for n in sizes]
    vals = [np.where(rng.random(n) < 0.5, 1, rng.normal(size=n)).astype(np.float32) for n in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    return off, np.concatenate(rows).astype(np.uint32), np.concatenate(vals)


@pytest.mark.parametrize("n_bits", [160, 1024])
@pytest.mark.parametrize("flags", [0, P.SRP_PLANES_Q16])
def test_rows_longer_than_a_stretch(n_bits, flags):
    """Rows about a multiple of 1024 nonzeros long and far longer: the same bits
    from the table, from drawn entries and from the sums alone."""
    rng = np.random.default_rng(n_bits + flags)
    sizes = [1023, 1024, 1025, 1055, 1056, 1057, 2047, 2048, 2049, 3072, 5000, 9999, 30_000, 7, 1024]
    off, idx, val = long_rows(rng, sizes, 30_000)
    got = {}
    for name, room, dim in (("sums", 0, 30_000), ("drawn", None, 1 << 20), ("table", None, 30_000)):
        ctx = P.bayeslsh_create(0)
        try:
            if room is not None:
                P.bayeslsh_reserve_workspace(ctx, room, fixed=True)
            got[name] = bits_of(ctx, P.csr_vectors(up(off), up(idx), up(val), dim), len(sizes), n_bits, P.OBJECT_MAJOR, flags)
        finally:
            ctx.close()
    for name, w in got.items():
        np.testing.assert_array_equal(w, got["sums"], err_msg=name)


def test_long_rows_keep_their_pace():
    """The same nonzeros in 200 rows of 30,000 as in 60,000 of 100: 800 waves, a
    quarter of what the chip holds, and a few times the open bits, so within 16
    times (with every open bit's entries drawn in FP64 it was over 100)."""
    rng = np.random.default_rng(8)
    ctx, dim = P.bayeslsh_create(0), 1 << 20
    us = {}
    try:
        for n_rows, n in ((60_000, 100), (200, 30_000)):
            step = dim // n
            idx = (np.arange(n) * step + rng.integers(0, step, (n_rows, n))).astype(np.uint32)
            off = np.arange(n_rows + 1, dtype=np.int64) * n
            vecs = P.csr_vectors(up(off), up(idx.reshape(-1)), up(rng.normal(size=idx.size).astype(np.float32)), dim)
            out = torch.empty(n_rows * 64, dtype=torch.int32, device="cuda").view(torch.uint32)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            runs = []
            for _ in range(3):
                a.record()
                P.bayeslsh_srp_sigs(ctx, vecs, None, 2048, 5, P.OBJECT_MAJOR, out)
                b.record()
                torch.cuda.synchronize()
                runs.append(a.elapsed_time(b) * 1e3)
            us[n] = min(runs)
        print("sparse SRP, 6M nonzeros: %s us" % us, flush=True)
        assert us[30_000] < 16 * us[100]
    finally:
        ctx.close()


def srp_us(ctx, vecs, n_rows, n_bits):
    out = torch.empty(n_rows * (n_bits // 32), dtype=torch.int32, device="cuda").view(torch.uint32)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    runs = []
    for _ in range(4):
        a.record()
        P.bayeslsh_srp_sigs(ctx, vecs, None, n_bits, 5, P.OBJECT_MAJOR, out)
        b.record()
        torch.cuda.synchronize()
        runs.append(a.elapsed_time(b) * 1e3)
    return min(runs), down(out)


@pytest.mark.parametrize("n_rows,nnz,n_bits", [(500, 100, 2048), (4000, 30, 128)])
def test_no_workspace_costs_the_entries_only(n_rows, nnz, n_bits):
    """Without room for masks every entry is drawn in FP64, four hashes together:
    about 4 times the filtered call (one hash at a time: over 100 times)."""
    rng = np.random.default_rng(n_rows)
    dim = 1 << 20
    idx = (np.arange(nnz) * (dim // nnz) + rng.integers(0, dim // nnz, (n_rows, nnz))).astype(np.uint32)
    vecs = P.csr_vectors(up(np.arange(n_rows + 1, dtype=np.int64) * nnz), up(idx.reshape(-1)),
                         up(rng.normal(size=idx.size).astype(np.float32)), dim)
    a, b = P.bayeslsh_create(0), P.bayeslsh_create(0)
    try:
        P.bayeslsh_reserve_workspace(b, 0, fixed=True)
        (t, x), (u, y) = srp_us(a, vecs, n_rows, n_bits), srp_us(b, vecs, n_rows, n_bits)
        print("sparse SRP %d rows: with a workspace %.0f us, without %.0f us" % (n_rows, t, u), flush=True)
        np.testing.assert_array_equal(x, y)
        assert u < 16 * t
    finally:
        a.close()
        b.close()


def test_a_table_that_cannot_be_allocated():
    """With 5 GiB of device memory free, a table of 8 GiB is not to be had, the
    masks are: entries are drawn as they occur, as in a workspace of the masks' size."""
    n_rows, nnz, dim, n_bits = 45_000, 100, 1 << 21, 2048
    rng = np.random.default_rng(2)
    idx = (np.arange(nnz) * (dim // nnz) + rng.integers(0, dim // nnz, (n_rows, nnz))).astype(np.uint32)
    vecs = P.csr_vectors(up(np.arange(n_rows + 1, dtype=np.int64) * nnz), up(idx.reshape(-1)),
                         up(rng.normal(size=idx.size).astype(np.float32)), dim)
    assert n_rows * nnz > 2 * dim
    a, b = P.bayeslsh_create(0), P.bayeslsh_create(0)
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    taken = torch.empty(free - (5 << 30), dtype=torch.uint8, device="cuda")
    try:
        P.bayeslsh_reserve_workspace(b, n_rows * n_bits // 8, fixed=True)
        (t, x), (u, y) = srp_us(a, vecs, n_rows, n_bits), srp_us(b, vecs, n_rows, n_bits)
        print("sparse SRP, no table to be had: %.0f us, drawn %.0f us" % (t, u), flush=True)
        assert n_rows * n_bits // 8 <= P.bayeslsh_workspace_bytes(a) < dim * n_bits * 2
        np.testing.assert_array_equal(x, y)
        assert t < 3 * u
    finally:
        del taken
        torch.cuda.empty_cache()
        a.close()
        b.close()


@pytest.mark.parametrize("n_bits", [32, 160, 512, 544])
@pytest.mark.parametrize("flags", [0, P.SRP_PLANES_Q16])
def test_short_rows_taken_at_once(n_bits, flags):
    """1024 rows of 4 terms and fewer, 1025 of them and 1024 with one more term: settled
    without masks or with them, a row's bits are the same."""
    print("sparse SRP short rows: %d bits flags %d" % (n_bits, flags), flush=True)
    rng = np.random.default_rng(n_bits + flags)
    n, dim = 1025, 1 << 20
    idx = np.sort(rng.integers(0, dim // 8, (n, 5)) * 8 + np.arange(5), axis=1).astype(np.uint32)
    val = rng.normal(size=(n, 5)).astype(np.float32)
    val[::7, 1] = -val[::7, 0]
    val[5], val[6, 0], val[7, 0] = 0, np.nan, np.inf
    ctx = P.bayeslsh_create(0)
    try:
        def bits(lens):
            off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
            keep = np.arange(5)[None, :] < np.asarray(lens)[:, None]
            m = len(lens)
            vecs = P.csr_vectors(up(off), up(np.append(idx[:m][keep], idx[0, :1])), up(np.append(val[:m][keep], val[0, :1])), dim)   # (no null arrays)
            return bits_of(ctx, vecs, m, n_bits, P.OBJECT_MAJOR, flags)
        for short in (0, 1, 4):
            more = np.full(n, short)
            longer = np.full(n - 1, short)
            longer[-1] = 5
            got, want = bits(np.full(n - 1, short)), bits(more)
            np.testing.assert_array_equal(got, want[:-1])
            np.testing.assert_array_equal(got[:-1], bits(longer)[:-1])
    finally:
        ctx.close()
