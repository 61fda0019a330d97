"""How the lists of a batch are shared out over the waves: every candidate decided
once whatever the lists' lengths, and lists of one length read in step."""
import numpy as np
import pytest
import torch

import paper_1110_1328_amd as P

pytestmark = pytest.mark.gpu

EPS, DELTA, GAMMA = 0.03, 0.05, 0.03


@pytest.fixture(scope="module")
def ctx():
    c = P.bayeslsh_create(0)
    yield c
    c.close()


def words(g, n, bits):
    a = torch.randint(-2 ** 31, 2 ** 31 - 1, (n, bits // 32), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    a[1::2] = torch.where(torch.rand(n // 2, bits // 32, generator=g, device="cuda") < 0.8, a[::2], a[1::2])
    return a


def lengths(kind, rng):
    if kind == "one length":
        return np.full(96, 40_000)
    if kind == "short":
        return rng.integers(0, 40, 3000)
    if kind == "one long":
        return np.concatenate([rng.integers(0, 700, 50), [3_000_000], rng.integers(0, 700, 50)])
    if kind == "several long":
        return np.array([700_001, 0, 5, 1_200_000, 255, 256, 257, 900_000])
    return np.exp(rng.uniform(0, np.log(60_000), 300)).astype(np.int64)


@pytest.mark.parametrize("kind", ["one length", "short", "one long", "several long", "mixed"])
@pytest.mark.parametrize("blocks", [0, 3, 7])
def test_every_candidate_once(ctx, kind, blocks):
    """The comparator's decisions, over lists of both measures; the codes start as 0xEE,
    which no decision is."""
    print("batched shares %s, %d blocks a CU" % (kind, blocks), flush=True)
    g, rng, n = torch.Generator(device="cuda").manual_seed(5), np.random.default_rng(5), 3000
    S = P.Signatures(words(g, n, 256).reshape(-1).view(torch.uint32), P.COSINE, P.OBJECT_MAJOR, n, 256)
    mh = torch.randint(0, 3, (n, 128), generator=g, device="cuda", dtype=torch.int32)
    J = P.Signatures(mh.reshape(-1).view(torch.uint32), P.JACCARD, P.OBJECT_MAJOR, n, 128)
    ln = lengths(kind, rng).astype(np.int64)
    m = int(ln.sum())
    off = np.concatenate([[0], np.cumsum(ln)])[:-1]
    q = rng.integers(0, n, len(ln))
    me = np.where(np.arange(len(ln)) % 3 == 0, P.JACCARD, P.COSINE)
    cand = torch.randint(0, n, (m,), generator=g, device="cuda", dtype=torch.int32).view(torch.uint32)
    d = P.list_descs(me, np.full(len(ln), 0.7), q, off, ln)
    got, want = P.make_result(m, m, m_debug=True), P.make_result(m, m, m_debug=True)
    got.code.fill_(0xEE)
    P.bayeslsh_set_tuning(ctx, batch_blocks_per_cu=blocks)
    try:
        P.bayeslsh_verify_batched(ctx, d, cand, J, S, EPS, DELTA, GAMMA, (1.0, 1.0), 32, got)
        P.bayeslsh_exhaustive_batched(ctx, d, cand, J, S, EPS, DELTA, GAMMA, (1.0, 1.0), 32, want)
        P.bayeslsh_sync(ctx)
    finally:
        P.bayeslsh_set_tuning(ctx)
    assert torch.equal(got.code[:m], want.code[:m])
    assert int(got.n_accepted.item()) == int(want.n_accepted.item()) > 0
    (gi, gv), (wi, wv) = got.accepted(), want.accepted()
    np.testing.assert_array_equal(gi, wi)
    np.testing.assert_array_equal(gv, wv)


@pytest.mark.parametrize("lists,length", [(512, 100_000), (1024, 40_000)])
def test_lists_of_one_length_keep_in_step(ctx, lists, length):
    """Sorted ids of an index larger than the L2s: the default shares take no more than
    1.4 times the best of 4 and 8 blocks a CU (parts that start at another place of
    every list took over 1.5 times)."""
    g, n = torch.Generator(device="cuda").manual_seed(6), 1_000_000
    S = P.Signatures(words(g, n, 1024).reshape(-1).view(torch.uint32), P.COSINE, P.OBJECT_MAJOR, n, 1024)
    m = lists * length
    of = torch.arange(lists, device="cuda").repeat_interleave(length)
    cand = ((torch.randint(0, n, (m,), generator=g, device="cuda") + (of << 32)).sort()[0] & 0xFFFFFFFF).to(torch.int32).view(torch.uint32)
    d = P.list_descs(np.full(lists, P.COSINE), np.full(lists, 0.7), np.random.default_rng(6).integers(0, n, lists),
                     np.arange(lists) * length, np.full(lists, length))
    res, us = P.make_result(m, 1000), {}
    try:
        for blocks in (0, 4, 8):
            P.bayeslsh_set_tuning(ctx, batch_blocks_per_cu=blocks)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            runs = []
            for _ in range(6):
                a.record()
                P.bayeslsh_verify_batched(ctx, d, cand, None, S, EPS, DELTA, GAMMA, (1.0, 1.0), 32, res)
                b.record()
                torch.cuda.synchronize()
                runs.append(a.elapsed_time(b) * 1e3)
            us[blocks] = min(runs)
    finally:
        P.bayeslsh_set_tuning(ctx)
    print("batched %d lists of %d: %s us" % (lists, length, us), flush=True)
    assert us[0] < 1.4 * min(us.values())


@pytest.mark.parametrize("k", [16, 32, 64])
def test_default_blocks_are_resident(ctx, k):
    """Lists of all lengths: the comparator's and phase 1's default grids take no more than
    1.2 times the best of 4 to 8 blocks a CU (blocks that a CU cannot hold at once wait for
    others to end: up to 1.27 times), and any grid gives the same codes."""
    g, n = torch.Generator(device="cuda").manual_seed(7), 100_000
    mh = torch.randint(0, 1 << 30, (n, 256), generator=g, device="cuda", dtype=torch.int32)
    mh[1::2] = torch.where(torch.rand(n // 2, 256, generator=g, device="cuda") < 0.6, mh[::2], mh[1::2])
    J = P.Signatures(mh.reshape(-1).view(torch.uint32), P.JACCARD, P.OBJECT_MAJOR, n, 256)
    rng = np.random.default_rng(7)
    ln = np.exp(rng.uniform(np.log(100), np.log(300_000), 1000)).astype(np.int64)
    m = int(ln.sum())
    of = torch.arange(len(ln), device="cuda").repeat_interleave(torch.from_numpy(ln).cuda())
    cand = ((torch.randint(0, n, (m,), generator=g, device="cuda") + (of << 32)).sort()[0] & 0xFFFFFFFF).to(torch.int32).view(torch.uint32)
    d = P.list_descs(np.full(len(ln), P.JACCARD), np.full(len(ln), 0.7), rng.integers(0, n, len(ln)),
                     np.concatenate([[0], np.cumsum(ln)])[:-1], ln)
    for f in (P.bayeslsh_verify_batched, P.bayeslsh_exhaustive_batched):
        res, us, codes = P.make_result(m, m // 10), {}, None
        try:
            for blocks in (0, 4, 5, 6, 8):
                P.bayeslsh_set_tuning(ctx, batch_blocks_per_cu=blocks)
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                runs = []
                for _ in range(5):
                    a.record()
                    f(ctx, d, cand, J, None, EPS, DELTA, GAMMA, (1.0, 1.0), k, res)
                    b.record()
                    torch.cuda.synchronize()
                    runs.append(a.elapsed_time(b) * 1e3)
                us[blocks] = min(runs)
                assert codes is None or torch.equal(codes, res.code[:m])
                codes = res.code[:m].clone()
        finally:
            P.bayeslsh_set_tuning(ctx)
        print("batched %s, k %d, %d candidates: %s us" % (f.__name__, k, m, us), flush=True)
        assert us[0] < 1.2 * min(us.values())
