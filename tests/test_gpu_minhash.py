"""Minhash signatures at the edges of their arithmetic: every hashes-per-lane
variant, set sizes around the 64 elements taken at a time, elements and
coefficients up to 2^32 - 1 (residues 0 and P - 1 among them)."""
import numpy as np
import pytest
import torch

import paper_1110_1328_amd as P

from gpu_util import down, up

pytestmark = pytest.mark.gpu

PRIME = (1 << 31) - 1


@pytest.mark.parametrize("n_hashes", [1, 64, 130, 192, 300, 360, 448, 512, 600, 768, 1024])
def test_minhash_edges(n_hashes):
    print("minhash edges: %d hashes" % n_hashes, flush=True)
    rng = np.random.default_rng(n_hashes)
    sizes = np.array([1, 2, 3, 4, 5, 63, 64, 65, 67, 68, 127, 128, 129, 200, 1000])
    off = np.zeros(len(sizes) + 1, np.int64)
    np.cumsum(sizes, out=off[1:])
    elems = rng.integers(0, 1 << 32, size=int(off[-1]), dtype=np.uint64).astype(np.uint32)
    elems[::7] = rng.choice(np.array([0, 1, PRIME - 1, PRIME, PRIME + 1, 2 * PRIME, 2 * PRIME + 1, 1 << 31], np.uint64),
                            size=len(elems[::7])).astype(np.uint32)
    a = rng.integers(1, PRIME, size=n_hashes, dtype=np.uint64)
    b = rng.integers(0, PRIME, size=n_hashes, dtype=np.uint64)
    a[::5] = rng.choice(np.array([1, PRIME - 1, PRIME, (1 << 32) - 1], np.uint64), size=len(a[::5]))
    b[::3] = rng.choice(np.array([0, PRIME - 1, PRIME, (1 << 32) - 1], np.uint64), size=len(b[::3]))
    ctx = P.bayeslsh_create(0)
    try:
        out = torch.empty(len(sizes) * n_hashes, dtype=torch.int32, device="cuda").view(torch.uint32)
        P.bayeslsh_minhash_sigs(ctx, P.set_vectors(up(off), up(elems), 1 << 32), up(a.astype(np.uint32)),
                                up(b.astype(np.uint32)), out)
        P.bayeslsh_sync(ctx)
        got = down(out).reshape(len(sizes), n_hashes)
    finally:
        ctx.close()
    h = (a[None, :] * elems.astype(np.uint64)[:, None] + b[None, :]) % np.uint64(PRIME)   # below 2^64
    want = np.minimum.reduceat(h, off[:-1], axis=0).astype(np.uint32)
    np.testing.assert_array_equal(got, want)


def test_decided_pairs_are_not_read_on():
    """Algorithm 1 over 4M id pairs of many x, one in ten similar: the levels past
    the first read the rows of what is left, so the call takes under 4 times one
    level of it (every pair's x row read at every level of its wave: over 5)."""
    n, H, m, k = 200_000, 256, 4_000_000, 16
    g = torch.Generator(device="cuda").manual_seed(9)
    sig = torch.randint(0, 1 << 30, (n, H), generator=g, device="cuda", dtype=torch.int32)
    keep = torch.rand(n // 2, H, generator=g, device="cuda") < torch.rand(n // 2, 1, generator=g, device="cuda")
    sig[1::2] = torch.where(keep, sig[::2], sig[1::2])
    x = torch.randint(0, n, (m,), generator=g, device="cuda", dtype=torch.int32)
    y = torch.where(torch.rand(m, generator=g, device="cuda") < 0.1, x ^ 1,
                    torch.randint(0, n, (m,), generator=g, device="cuda", dtype=torch.int32))
    ctx, cand, res = P.bayeslsh_create(0), P.pairs(x.view(torch.uint32), y.view(torch.uint32)), P.make_result(m, m)
    us = {}
    try:
        for n_max in (k, H):
            S = P.Signatures(sig.reshape(-1).view(torch.uint32), P.JACCARD, P.OBJECT_MAJOR, n, H, n_max)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            runs = []
            for _ in range(5):
                a.record()
                for _ in range(5):
                    P.bayeslsh_verify(ctx, cand, S, 0.7, 0.03, 0.05, 0.03, (1, 1), k, res)
                b.record()
                torch.cuda.synchronize()
                runs.append(a.elapsed_time(b) * 200)
            us[n_max] = min(runs)
        print("minhash pairs: %s us" % us, flush=True)
        assert us[H] < 4 * us[k]
    finally:
        ctx.close()


@pytest.mark.parametrize("n_sets", [32_767, 32_768, 32_769, 70_001])
@pytest.mark.parametrize("n_hashes", [32, 100])
def test_more_sets_than_waves(n_sets, n_hashes):
    """A wave that takes one, two or three sets (32,768 waves on 256 CUs), some of them
    empty, the last ones of different lengths."""
    rng = np.random.default_rng(n_sets)
    ln = rng.integers(0, 70, n_sets) * (rng.random(n_sets) < 0.3)
    off = np.concatenate([[0], np.cumsum(ln)]).astype(np.int64)
    el = rng.integers(0, 1 << 31, int(off[-1]), dtype=np.uint32)
    a, b = rng.integers(1, PRIME, n_hashes).astype(np.uint32), rng.integers(0, PRIME, n_hashes).astype(np.uint32)
    out = torch.empty(n_sets * n_hashes, dtype=torch.int32, device="cuda").view(torch.uint32)
    ctx = P.bayeslsh_create(0)
    try:
        P.bayeslsh_minhash_sigs(ctx, P.set_vectors(up(off), up(el), 1 << 31), up(a), up(b), out)
        with pytest.raises(P.BayesLSHError):   # the empty sets
            P.bayeslsh_sync(ctx)
    finally:
        ctx.close()
    got = down(out).reshape(n_sets, n_hashes)
    want = np.full((n_sets, n_hashes), 0xFFFFFFFF, np.uint64)
    for h in range(n_hashes):
        v = (el.astype(np.uint64) * np.uint64(a[h]) + np.uint64(b[h])) % np.uint64(PRIME)
        full = ln > 0
        want[full, h] = np.minimum.reduceat(v, off[:-1][full])
    np.testing.assert_array_equal(got, want.astype(np.uint32))
