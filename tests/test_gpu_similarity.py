"""Exact similarities over every shape of the kernels: runs of one x (lists, all
pairs) and lone pairs, rows around the table's and the loads' sizes, empty
rows, the largest term number, dense rows with and without 16-byte loads."""
import numpy as np
import pytest
import torch

import paper_1110_1328_amd as P

from gpu_util import down, up

pytestmark = pytest.mark.gpu

TOP = (1 << 32) - 1


@pytest.fixture(scope="module")
def ctx():
    c = P.bayeslsh_create(0)
    yield c
    c.close()


def rows(rng, spread):
    """Sorted unique rows from `spread` terms; some with the top term, some empty."""
    sizes = [0, 1, 3, 4, 5, 15, 16, 63, 64, 65, 100, 127, 128, 129, 255, 256, 257, 383, 384, 385, 511, 512, 513, 700]
    sizes += [int(v) for v in rng.integers(1, 150, 40)]
    out = []
    for i, n in enumerate(sizes):
        r = np.sort(rng.choice(spread, size=n, replace=False)).astype(np.int64)
        if i % 3 == 0 and n:
            r[-1] = TOP
        out.append(r)
    return out


def reference(rs, vs, x, y):
    got = np.zeros(len(x))
    for i, (p, q) in enumerate(zip(x, y)):
        common, a, b = np.intersect1d(rs[p], rs[q], assume_unique=True, return_indices=True)
        if vs is None:
            union = len(rs[p]) + len(rs[q]) - len(common)
            got[i] = len(common) / union if union else 0.0
        else:
            u, v = vs[p].astype(np.float64), vs[q].astype(np.float64)
            norm = np.sqrt((u * u).sum()) * np.sqrt((v * v).sum())
            got[i] = (u[a] * v[b]).sum() / norm if norm > 0 else 0.0
    return got


@pytest.mark.parametrize("kind", ["csr", "sets"])
@pytest.mark.parametrize("spread", [900, 100_000])
def test_sparse_similarity_shapes(ctx, kind, spread):
    print("similarity shapes %s spread %d" % (kind, spread), flush=True)
    rng = np.random.default_rng(spread)
    rs = rows(rng, spread)
    n = len(rs)
    vs = [rng.normal(size=len(r)).astype(np.float32) for r in rs] if kind == "csr" else None
    off = np.zeros(n + 1, np.int64)
    np.cumsum([len(r) for r in rs], out=off[1:])
    idx = np.concatenate(rs).astype(np.uint32)
    vecs = (P.csr_vectors(up(off), up(idx), up(np.concatenate(vs)), 1 << 32) if kind == "csr"
            else P.set_vectors(up(off), up(idx), 1 << 32))
    # lone pairs, all pairs (runs that cross waves), lists of 1, 2, 5 and 70 ids
    x, y = rng.integers(0, n, 1001), rng.integers(0, n, 1001)
    y[0], x[1] = n, n + 5                                    # bad ids
    got = down(P.bayeslsh_exact_similarity(ctx, P.pairs(up(x.astype(np.uint32)), up(y.astype(np.uint32))), vecs))
    with pytest.raises(P.BayesLSHError):
        P.bayeslsh_sync(ctx)
    assert np.isnan(got[:2]).all()
    np.testing.assert_allclose(got[2:], reference(rs, vs, x[2:], y[2:]), rtol=0, atol=1e-12)
    ax, ay = np.triu_indices(n, 1)
    got = down(P.bayeslsh_exact_similarity(ctx, P.all_pairs(n), vecs))[:len(ax)]
    P.bayeslsh_sync(ctx)
    np.testing.assert_allclose(got, reference(rs, vs, ax, ay), rtol=0, atol=1e-12)
    lens = np.array([1, 2, 5, 70, 3])
    q, o = rng.integers(0, n, len(lens)), np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    c = rng.integers(0, n, int(o[-1]))
    got = down(P.bayeslsh_exact_similarity(ctx, P.query_lists(up(q.astype(np.uint32)), up(o), up(c.astype(np.uint32)),
                                                              int(o[-1])), vecs))[:int(o[-1])]
    P.bayeslsh_sync(ctx)
    np.testing.assert_allclose(got, reference(rs, vs, np.repeat(q, lens), c), rtol=0, atol=1e-12)


@pytest.mark.parametrize("dim", [1, 5, 64, 100, 130, 256])
def test_dense_similarity_dims(ctx, dim):
    print("dense similarity dim %d" % dim, flush=True)
    rng = np.random.default_rng(dim)
    v = rng.normal(size=(300, dim)).astype(np.float32)
    v[7] = 0
    x, y = rng.integers(0, 300, 777), rng.integers(0, 300, 777)
    x[5], y[9] = 7, 300
    d = v.astype(np.float64)
    for shift in (0, 1):   # rows from an address that 16-byte loads may start at, and one they may not
        buf = torch.zeros(v.size + 4, device="cuda")
        buf[shift:shift + v.size] = torch.from_numpy(v.reshape(-1)).cuda()
        vecs = P.dense_vectors(buf[shift:shift + v.size].view(300, dim))
        got = down(P.bayeslsh_exact_similarity(ctx, P.pairs(up(x.astype(np.uint32)), up(y.astype(np.uint32))), vecs))
        with pytest.raises(P.BayesLSHError):
            P.bayeslsh_sync(ctx)
        assert np.isnan(got[9])
        ok = np.arange(777) != 9
        a, b = d[x[ok]], d[y[ok]]
        norm = np.sqrt((a * a).sum(1)) * np.sqrt((b * b).sum(1))
        want = np.where(norm > 0, (a * b).sum(1) / np.where(norm > 0, norm, 1), 0)
        np.testing.assert_allclose(got[ok], want, rtol=0, atol=1e-12)


def csr_rows(rng, n, nnz, dim):
    """n rows of nnz sorted unique terms."""
    step = dim // nnz
    idx = np.arange(nnz) * step + rng.integers(0, step, (n, nnz))
    return np.arange(n + 1, dtype=np.int64) * nnz, idx.astype(np.uint32)


def passes_us(f, n=20):
    """Microseconds a call among others, the least of five runs."""
    for _ in range(3):
        f()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    got = []
    for _ in range(5):
        torch.cuda.synchronize()
        a.record()
        for _ in range(n):
            f()
        b.record()
        torch.cuda.synchronize()
        got.append(a.elapsed_time(b) / n * 1e3)
    return min(got)


@pytest.mark.parametrize("kind", ["csr", "sets"])
def test_a_small_sample_is_spread_over_the_chip(ctx, kind):
    """The sample of a prior, a thousand pairs of distinct x: as many waves as the
    chip holds side by side, so about the time of one pair (4 times would be
    four pairs one after another in a wave; a wave of 64 takes 16 times)."""
    rng = np.random.default_rng(3)
    off, idx = csr_rows(rng, 5000, 100, 1 << 20)
    vecs = (P.csr_vectors(up(off), up(idx.reshape(-1)), up(rng.normal(size=idx.size).astype(np.float32)), 1 << 20)
            if kind == "csr" else P.set_vectors(up(off), up(idx.reshape(-1)), 1 << 20))
    us = {}
    for m in (1, 1000):
        x, y = (up(rng.integers(0, 5000, m).astype(np.uint32)) for _ in range(2))
        out, c = torch.empty(m, dtype=torch.float64, device="cuda"), P.pairs(x, y)
        us[m] = passes_us(lambda: P.bayeslsh_exact_similarity(ctx, c, vecs, out))
    print("similarity sample %s: %s us" % (kind, us), flush=True)
    assert us[1000] < 4 * us[1]


@pytest.mark.parametrize("n", [8193, 65536, 65537, 8192 * 9, 8192 * 63 + 5, 8192 * 64 + 1])
def test_candidates_a_wave(ctx, n):
    """A wave a pair (256 CUs: up to 65,536 pairs), then 9 and up to 64 candidates to
    a wave, half of them in runs and half lone, the last wave's share cut short."""
    rng = np.random.default_rng(n)
    off, idx = csr_rows(rng, 300, 7, 140)
    x, y = rng.integers(0, 300, n), rng.integers(0, 300, n)
    x[: n // 2] = np.sort(x[: n // 2])
    member = np.zeros((300, 140), np.int32)
    np.put_along_axis(member, idx.astype(np.int64), 1, axis=1)
    common = (member @ member.T)[x, y]
    got = down(P.bayeslsh_exact_similarity(ctx, P.pairs(up(x.astype(np.uint32)), up(y.astype(np.uint32))),
                                           P.set_vectors(up(off), up(idx.reshape(-1)), 140)))[:n]
    P.bayeslsh_sync(ctx)
    np.testing.assert_array_equal(got, common / (14 - common))


@pytest.mark.parametrize("kind", ["csr", "sets"])
@pytest.mark.parametrize("spread", [900, 100_000])
def test_runs_of_one_x_over_odd_rows(ctx, kind, spread):
    """More pairs than go a wave each: the shapes above in runs of 64, 5 and 2 and one
    run across waves, bad ids among them."""
    rng = np.random.default_rng(spread + 1)
    rs = rows(rng, spread)
    n = len(rs)
    vs = [rng.normal(size=len(r)).astype(np.float32) for r in rs] if kind == "csr" else None
    off = np.zeros(n + 1, np.int64)
    np.cumsum([len(r) for r in rs], out=off[1:])
    idx = np.concatenate(rs).astype(np.uint32)
    vecs = (P.csr_vectors(up(off), up(idx), up(np.concatenate(vs)), 1 << 32) if kind == "csr"
            else P.set_vectors(up(off), up(idx), 1 << 32))
    ax, ay = (v.reshape(-1) for v in np.indices((n, n)))
    table = reference(rs, vs, ax, ay).reshape(n, n)
    m = 70_000
    x = np.concatenate([np.repeat(rng.integers(0, n, m // r + 1), r)[: m // 4] for r in (64, 5, 2, m)])
    y = rng.integers(0, n, len(x))
    bad = rng.choice(len(x), 50, replace=False)
    y[bad[:25]], x[bad[25:]] = n, n + 3
    got = down(P.bayeslsh_exact_similarity(ctx, P.pairs(up(x.astype(np.uint32)), up(y.astype(np.uint32))), vecs))[:len(x)]
    with pytest.raises(P.BayesLSHError):
        P.bayeslsh_sync(ctx)
    ok = np.ones(len(x), bool)
    ok[bad] = False
    assert np.isnan(got[bad]).all()
    np.testing.assert_allclose(got[ok], table[x[ok], y[ok]], rtol=0, atol=1e-12)


@pytest.mark.parametrize("kind", ["csr", "sets"])
def test_rows_longer_than_the_table(ctx, kind):
    """Rows of one piece, of several and of parts of one against short rows, rows
    of their own kind, rows that end before a piece does and rows far longer."""
    rng = np.random.default_rng(17)
    sizes = [0, 1, 30, 64, 65, 300, 383, 384, 385, 386, 500, 767, 768, 769, 1024, 1025, 1200, 1536, 2000, 5000, 17_000, 40_000]
    rs = [np.sort(rng.choice(60_000, size=n, replace=False)).astype(np.int64) for n in sizes]
    rs += [np.arange(400), np.arange(50_000, 51_000), np.arange(0, 60_000, 90), np.arange(59_000, 60_000)]
    for i in range(5, len(rs), 3):
        rs[i][-1] = TOP
    n = len(rs)
    vs = [rng.normal(size=len(r)).astype(np.float32) for r in rs] if kind == "csr" else None
    off = np.zeros(n + 1, np.int64)
    np.cumsum([len(r) for r in rs], out=off[1:])
    idx = np.concatenate(rs).astype(np.uint32)
    vecs = (P.csr_vectors(up(off), up(idx), up(np.concatenate(vs)), 1 << 32) if kind == "csr"
            else P.set_vectors(up(off), up(idx), 1 << 32))
    x, y = (v.reshape(-1) for v in np.indices((n, n)))
    want = reference(rs, vs, x, y)
    many = np.tile(np.arange(n * n), 65536 // (n * n) + 2)
    for order in (np.arange(n * n), many, rng.permutation(many)):   # a wave a pair, runs of one x, lone pairs
        got = down(P.bayeslsh_exact_similarity(ctx, P.pairs(up(x[order].astype(np.uint32)), up(y[order].astype(np.uint32))),
                                               vecs))[:len(order)]
        P.bayeslsh_sync(ctx)
        np.testing.assert_allclose(got, want[order], rtol=0, atol=1e-12)


@pytest.mark.parametrize("kind,long", [("csr", 500), ("sets", 100_000)])
def test_long_rows_take_no_longer_than_their_entries(ctx, kind, long):
    """Pairs of a row of 100 terms and a long one, 64 of them, against 64 pairs of
    rows of 100: a set of 100,000 is searched, not read; rows past the table's
    size are not one pair after another in a wave."""
    rng = np.random.default_rng(4)
    short, sidx = csr_rows(rng, 64, 100, 1 << 20)
    _, lidx = csr_rows(rng, 64, long, 1 << 20)
    off = np.concatenate([short, short[-1] + long * np.arange(1, 65, dtype=np.int64)])
    idx = np.concatenate([sidx.reshape(-1), lidx.reshape(-1)])
    vecs = (P.csr_vectors(up(off), up(idx), up(rng.normal(size=idx.size).astype(np.float32)), 1 << 20)
            if kind == "csr" else P.set_vectors(up(off), up(idx), 1 << 20))
    i, out = np.arange(64, dtype=np.uint32), torch.empty(64, dtype=torch.float64, device="cuda")
    us = []
    for x, y in ((i, i[::-1]), (i, i + 64), (i + 64, i)):
        c = P.pairs(up(np.ascontiguousarray(x)), up(np.ascontiguousarray(y)))
        us.append(passes_us(lambda: P.bayeslsh_exact_similarity(ctx, c, vecs, out)))
    print("similarity of long rows %s %d: %s us" % (kind, long, us), flush=True)
    assert max(us[1:]) < 6 * us[0]
