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
