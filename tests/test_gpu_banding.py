"""GPU parity of LSH banding candidate generation (bayeslsh_band_candidates)
against the oracle's plain banding: the same pairs in the same order."""
import numpy as np
import pytest
import torch

import paper_1110_1328_amd as P
from oracle import reference as R
from synth import generators as G

from gpu_util import down, sigs_tensor, up

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available()
    c = P.bayeslsh_create(0)
    yield c
    c.close()


@pytest.fixture(scope="module")
def bits():
    """Sign bits of a clustered point set (64 bits): buckets of uneven size."""
    mix = G.dense_mixture(n=3000, d=64, n_comp=30, seed=G.SEED_BASE + 61)
    planes = G.gaussian_planes(64, 64, G.SEED_BASE + 62)
    return G.pack_bits((mix.x.astype(np.float64) @ planes >= 0).astype(np.uint8))


def run(ctx, S, nb, b, cap, max_bucket=0, tile=0):
    x, y, n, trunc = P.bayeslsh_band_candidates(ctx, S, nb, b, cap, max_bucket=max_bucket, order_tile=tile)
    k = min(n, cap)
    return down(x)[:k], down(y)[:k], n, trunc


@pytest.mark.parametrize("tile", [0, 16])
@pytest.mark.parametrize("nb,b,max_bucket", [(8, 8, 0), (5, 11, 0), (8, 8, 5), (4, 16, 0), (3, 5, 40), (20, 3, 40)])
def test_banding_matches_oracle(ctx, bits, nb, b, max_bucket, tile):
    """Both layouts; band keys that straddle a 32-bit word (b = 11); bucket
    caps (a single tile per bucket, and caps that are not a multiple of the
    tile); row-major and tiled orders; 20 bands of 3 bits (many pairs seen
    again in later bands, so the earlier-band test drops most of them)."""
    print("banding nb=%d b=%d max_bucket=%d tile=%d" % (nb, b, max_bucket, tile), flush=True)
    wx, wy = R.band_candidates(bits, nb, b, max_bucket, tile=tile)
    assert len(wx) > 1000
    for layout in (P.OBJECT_MAJOR, P.WORD_MAJOR):
        S = sigs_tensor(bits, P.COSINE, layout)
        gx, gy, n, trunc = run(ctx, S, nb, b, len(wx) + 100, max_bucket, tile)
        assert n == len(wx) and not trunc
        np.testing.assert_array_equal(gx, wx)
        np.testing.assert_array_equal(gy, wy)


@pytest.mark.parametrize("tile", [0, 16])
def test_banding_truncation_empty_and_invalid(ctx, bits, tile):
    print("banding truncation tile=%d" % tile, flush=True)
    wx, wy = R.band_candidates(bits, 8, 8, tile=tile)
    S = sigs_tensor(bits, P.COSINE, P.OBJECT_MAJOR)
    half = len(wx) // 2
    gx, gy, n, trunc = run(ctx, S, 8, 8, half, tile=tile)
    assert trunc and n == len(wx)
    np.testing.assert_array_equal(gx, wx[:half])
    np.testing.assert_array_equal(gy, wy[:half])
    with pytest.raises(P.BayesLSHError) as e:
        run(ctx, S, 8, 8, 16, tile=8)
    assert e.value.code == -1
    # distinct random 32-bit keys in a single band: no pair
    rnd = np.random.default_rng(3).integers(0, 2 ** 32, size=(500, 1), dtype=np.uint64).astype(np.uint32)
    _, _, n0, _ = run(ctx, sigs_tensor(rnd, P.COSINE, P.OBJECT_MAJOR), 1, 32, 16)
    assert n0 == len(R.band_candidates(rnd, 1, 32)[0])
    for nb, b in ((0, 8), (8, 0), (8, 33), (9, 8)):     # 9 x 8 bits > 64 stored bits
        with pytest.raises(P.BayesLSHError) as e:
            run(ctx, S, nb, b, 16)
        assert e.value.code == -1
    mh = sigs_tensor(np.zeros((10, 64), np.uint32), P.JACCARD, P.OBJECT_MAJOR)
    with pytest.raises(P.BayesLSHError):
        run(ctx, mh, 4, 8, 16)


@pytest.mark.parametrize("nb,b,n,max_bucket,fixed", [
    (17, 16, 1500, 0, False),    # two keys to a word, an odd number of them, one more word than the registers hold
    (16, 16, 1500, 33, False),   # the last word in registers; a bucket cap of two tiles and one member
    (9, 17, 1500, 0, False),     # keys of more than 16 bits, eight words of earlier bands
    (12, 20, 1500, 0, False),    # the same, more words than the registers hold
    (64, 2, 300, 0, False),      # the most bands
    (1, 1, 257, 0, False),       # one band, two buckets
    (3, 32, 1500, 0, False),     # full-word keys: one band at a time
    (8, 8, 3000, 0, True),       # a workspace that holds some of the bands at a time
])
def test_banding_key_rows_and_groups(ctx, nb, b, n, max_bucket, fixed):
    """The earlier-band test over every row shape, and the bands in one group
    or several: pairs in both orders and the tile descriptors, against the
    oracle's pairs."""
    print("banding rows nb=%d b=%d n=%d cap=%d" % (nb, b, n, max_bucket), flush=True)
    rng = np.random.default_rng(G.SEED_BASE + 63 + nb * b)
    words = (nb * b + 31) // 32
    base = rng.integers(0, 2, size=(n // 60 + 1, words * 32), dtype=np.uint8)
    flip = rng.random((n, words * 32)) < 0.02
    bits = G.pack_bits((base[rng.integers(0, len(base), n)] ^ flip).astype(np.uint8))
    S = sigs_tensor(bits, P.COSINE, P.OBJECT_MAJOR)
    own = P.bayeslsh_create(0) if fixed else ctx
    try:
        if fixed:
            P.bayeslsh_reserve_workspace(own, 8 * n * (nb + 6) + (128 << 10), fixed=True)
        for tile in (0, 16):
            wx, wy = R.band_candidates(bits, nb, b, max_bucket, tile=tile)
            assert len(wx) > 100
            gx, gy, got, trunc = run(own, S, nb, b, len(wx) + 7, max_bucket, tile)
            assert got == len(wx) and not trunc
            np.testing.assert_array_equal(gx, wx)
            np.testing.assert_array_equal(gy, wy)
        # the descriptors list the tiled order's pairs; a short buffer gets its first tiles
        buf, nt, got, trunc = P.bayeslsh_band_tiles(own, S, nb, b, 1 << 16, max_bucket=max_bucket)
        assert got == len(wx) and not trunc
        t = down(buf)[:24 * nt].reshape(nt, 24)
        first, keep, ids = t[:, 0], np.ascontiguousarray(t[:, 2:6]), np.ascontiguousarray(t[:, 6:22]).view(np.uint32)
        on = np.unpackbits(keep.view(np.uint8), axis=1, bitorder="little").astype(bool)
        np.testing.assert_array_equal(first, np.cumsum(on.sum(1)) - on.sum(1))
        tile_of, pos = np.nonzero(on)
        np.testing.assert_array_equal(ids[tile_of, pos // 16], wx)
        np.testing.assert_array_equal(ids[tile_of, 16 + pos % 16], wy)
        assert not t[:, 22:].any()
        short = torch.full((24 * nt,), -1, dtype=torch.int64, device="cuda")
        _, nt2, got2, trunc = P.bayeslsh_band_tiles(own, S, nb, b, nt // 2, max_bucket=max_bucket, tiles_out=short)
        assert trunc == (nt > nt // 2) and nt2 == nt and got2 == got
        s = down(short).reshape(nt, 24)
        np.testing.assert_array_equal(s[:nt // 2], t[:nt // 2])
        assert (s[nt // 2:] == -1).all()
    finally:
        if fixed:
            own.close()


@pytest.mark.parametrize("tile", [0, 16])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1024, 1025, 2049, 4097])
def test_buckets_across_chunks(ctx, n, tile):
    """Buckets found some hundred positions to a wave: one bucket for all, buckets that end
    with a wave's step or chunk, of one member, and over several whole chunks."""
    rng = np.random.default_rng(n)
    keys = np.zeros((n, 4), np.uint32)                     # 8-bit band keys: band 0 all equal
    keys[:, 1] = np.minimum(np.arange(n) // 64, 255)       # whole steps
    keys[:, 2] = np.where(rng.random(n) < 0.02, rng.integers(0, 255, n), 255)
    keys[:, 3] = rng.integers(0, 256, n)
    words = (keys[:, 0] | keys[:, 1] << 8 | keys[:, 2] << 16 | keys[:, 3] << 24).astype(np.uint32).reshape(n, 1)
    S = sigs_tensor(words, P.COSINE, P.OBJECT_MAJOR)
    for max_bucket in (40, 0):
        if max_bucket == 0 and n > 1100:
            continue
        for order in ([0, 1, 2, 3], [3, 2, 1, 0]):
            w = sum(keys[:, b].astype(np.uint32) << np.uint32(8 * i) for i, b in enumerate(order)).astype(np.uint32).reshape(n, 1)
            S = sigs_tensor(w, P.COSINE, P.OBJECT_MAJOR)
            wx, wy = R.band_candidates(w, 4, 8, max_bucket, tile=tile)
            gx, gy, m, trunc = run(ctx, S, 4, 8, len(wx) + 10, max_bucket, tile)
            assert m == len(wx) and not trunc
            np.testing.assert_array_equal(gx, wx)
            np.testing.assert_array_equal(gy, wy)


@pytest.mark.parametrize("nb,b", [(5, 30), (5, 31), (3, 32), (7, 29), (33, 26)])
def test_groups_of_wide_keys(ctx, nb, b):
    """Keys too wide to sort all bands together: groups of bands, the last one
    smaller, at sizes where the library's sort changes its method."""
    rng = np.random.default_rng(nb * b)
    n_words = (nb * b + 31) // 32
    for n in (1, 300, 1500, 5000, 20_000, 70_000):
        rows = rng.integers(0, 1 << 32, (max(n // 3, 1), n_words), dtype=np.uint32)
        sig = rows[rng.integers(0, len(rows), n)]
        flip = rng.random((n, n_words)) < 0.5
        sig = np.where(flip, sig ^ (np.uint32(1) << rng.integers(0, 32, (n, n_words)).astype(np.uint32)), sig)
        S = sigs_tensor(sig, P.COSINE, P.OBJECT_MAJOR)
        wx, wy = R.band_candidates(sig, nb, b, 0, tile=16)
        gx, gy, m, trunc = run(ctx, S, nb, b, len(wx) + 10, 0, 16)
        assert m == len(wx) and not trunc
        np.testing.assert_array_equal(gx, wx)
        np.testing.assert_array_equal(gy, wy)
