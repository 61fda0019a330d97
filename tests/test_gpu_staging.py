"""Algorithm 1 calls of more candidates than run in one launch: the accepted pairs'
staging slices overflowing to the caller's list, a list too short for them, and ids
out of range, in every kernel that stages -- rows of 256 and of more hashes, rows at 4
bytes, word-major with and without a prefix, minhash."""
import numpy as np
import pytest
import torch

import paper_1110_1328_amd as P
from oracle import reference as R
from synth import generators as G

from gpu_util import assert_same_as_oracle, decode_result, sigs_tensor, up

pytestmark = pytest.mark.gpu

T, EPS, DELTA, GAMMA, K = 0.7, 0.03, 0.05, 0.03, 32
N = 65536 + 4096 + 7
N_OBJ = 4001
SLICES = 256


@pytest.fixture(scope="module")
def ctx():
    c = P.bayeslsh_create(0)
    yield c
    c.close()


def signatures(measure, n_hashes, seed):
    s = np.random.default_rng(seed).uniform(0.5, 1.0, (N_OBJ + 1) // 2)
    if measure == P.JACCARD:
        return G.calibration_minhash(len(s), n_hashes, s, seed)[:N_OBJ]
    return G.pack_bits(G.calibration_bits(len(s), n_hashes, s, seed))[:N_OBJ]


def form_of(name, sig, n_hashes):
    if name == "minhash":
        return sigs_tensor(sig, P.JACCARD, P.OBJECT_MAJOR)
    om, wm = sigs_tensor(sig, P.COSINE, P.OBJECT_MAJOR), sigs_tensor(sig, P.COSINE, P.WORD_MAJOR)
    pfx = up(np.ascontiguousarray(sig[:, :4]))
    buf = torch.zeros(om.data.numel() + 1, dtype=torch.int32, device="cuda")
    buf[1:] = om.data.reshape(-1).view(torch.int32)
    at4 = buf[1:].view(torch.uint32)
    return {"rows": om, "words": wm,
            "words, prefix": P.Signatures(wm.data, P.COSINE, P.WORD_MAJOR, N_OBJ, n_hashes, prefix=pfx),
            "rows at 4 bytes": P.Signatures(at4, P.COSINE, P.OBJECT_MAJOR, N_OBJ, n_hashes),
            "rows at 4 bytes, prefix": P.Signatures(at4, P.COSINE, P.OBJECT_MAJOR, N_OBJ, n_hashes, prefix=pfx)}[name]


@pytest.mark.parametrize("name,n_hashes", [("rows", 256), ("rows", 512), ("rows", 1024), ("rows at 4 bytes", 1024),
                                           ("rows at 4 bytes, prefix", 512), ("words", 512), ("words, prefix", 1024),
                                           ("minhash", 256)])
def test_staging_overflow_short_lists_and_bad_ids(ctx, name, n_hashes):
    print("staging %s %d hashes" % (name, n_hashes), flush=True)
    measure = P.JACCARD if name == "minhash" else P.COSINE
    sig = signatures(measure, n_hashes, 91 + n_hashes)
    S = form_of(name, sig, n_hashes)
    rng = np.random.default_rng(n_hashes)
    x = rng.integers(0, N_OBJ - 1, N).astype(np.uint32)
    y = np.where(rng.random(N) < 0.6, x ^ 1, rng.integers(0, N_OBJ, N)).astype(np.uint32)
    want = R.verify(x, y, measure, sig, K, n_hashes // K, T, EPS, DELTA, GAMMA)
    n_acc = int(((want["decision"] == R.DEC_CONC) | (want["decision"] == R.DEC_NMAX)).sum())
    assert n_acc > 20 * SLICES
    bad = np.array([0, 63, 64, 700, N // 2, N - 2, N - 1])
    bx, by = x.copy(), y.copy()
    bx[bad[::2]], by[bad[1::2]] = N_OBJ, 0xFFFFFFFF
    ok = np.ones(N, bool)
    ok[bad] = False
    try:
        for stage in (SLICES, 16 * SLICES, 0):   # one entry a slice: nearly all direct; 16: staged and direct; all staged
            P.bayeslsh_set_tuning(ctx, acc_stage_cap=stage)
            for xs, ys, cap, code in ((x, y, N, None), (x, y, n_acc // 3, -4), (bx, by, N, -5), (x, y, N, None)):
                res = P.make_result(N, cap, m_debug=True)
                P.bayeslsh_verify(ctx, P.pairs(up(xs), up(ys)), S, T, EPS, DELTA, GAMMA, (1, 1), K, res)
                if code is None:
                    P.bayeslsh_sync(ctx)
                    assert_same_as_oracle(decode_result(res, N), want)
                    continue
                with pytest.raises(P.BayesLSHError) as e:
                    P.bayeslsh_sync(ctx)
                assert e.value.code == code
                got = res.code.cpu().numpy()[:N]
                if code == -4:
                    np.testing.assert_array_equal(got >> 6, want["decision"])
                    assert int(res.n_accepted.item()) == n_acc
                else:
                    assert (got[bad] == 0xFF).all()
                    np.testing.assert_array_equal((got >> 6)[ok], want["decision"][ok])
                    np.testing.assert_array_equal((got & 63)[ok], want["level"][ok])
                    idx, _ = res.accepted()
                    acc = np.flatnonzero(ok & ((want["decision"] == R.DEC_CONC) | (want["decision"] == R.DEC_NMAX)))
                    np.testing.assert_array_equal(idx, acc)
    finally:
        P.bayeslsh_set_tuning(ctx)


@pytest.mark.parametrize("name,n_hashes", [("rows", 512), ("words, prefix", 1024), ("minhash", 256)])
def test_short_lists_and_bad_ids_of_few_candidates(ctx, name, n_hashes):
    """The same of calls that run in one launch, at its last size and a small one."""
    measure = P.JACCARD if name == "minhash" else P.COSINE
    sig = signatures(measure, n_hashes, 17 + n_hashes)
    S = form_of(name, sig, n_hashes)
    rng = np.random.default_rng(n_hashes)
    for n in (40, 65536):
        x = rng.integers(0, N_OBJ - 1, n).astype(np.uint32)
        y = np.where(rng.random(n) < 0.9, x ^ 1, rng.integers(0, N_OBJ, n)).astype(np.uint32)
        want = R.verify(x, y, measure, sig, K, n_hashes // K, T, EPS, DELTA, GAMMA)
        acc = (want["decision"] == R.DEC_CONC) | (want["decision"] == R.DEC_NMAX)
        bx, by = x.copy(), y.copy()
        bx[3], by[n - 1] = N_OBJ, 1 << 31
        ok = np.ones(n, bool)
        ok[[3, n - 1]] = False
        for xs, ys, cap, code in ((x, y, int(acc.sum()) - 1, -4), (bx, by, n, -5), (x, y, n, None)):
            res = P.make_result(n, cap, m_debug=True)
            P.bayeslsh_verify(ctx, P.pairs(up(xs), up(ys)), S, T, EPS, DELTA, GAMMA, (1, 1), K, res)
            if code is None:
                P.bayeslsh_sync(ctx)
                assert_same_as_oracle(decode_result(res, n), want)
                continue
            with pytest.raises(P.BayesLSHError) as e:
                P.bayeslsh_sync(ctx)
            assert e.value.code == code
            if code == -4:
                assert int(res.n_accepted.item()) == int(acc.sum())
            else:
                got = res.code.cpu().numpy()[:n]
                assert (got[~ok] == 0xFF).all()
                np.testing.assert_array_equal((got >> 6)[ok], want["decision"][ok])
                np.testing.assert_array_equal(res.accepted()[0], np.flatnonzero(ok & acc))
