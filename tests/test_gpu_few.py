"""Algorithm 1 of few candidates (one launch, up to 65536) and of more (queue and
flush): the oracle's decisions, levels, m and S_hat on both sides of the limit
and of a block, for every layout and k, rows of one x and of many, in calls
that follow one another on one context."""
import numpy as np
import pytest
import torch

import paper_1110_1328_amd as P
from oracle import reference as R
from synth import generators as G

from gpu_util import assert_same_as_oracle, decode_result, sigs_tensor, up

pytestmark = pytest.mark.gpu

T, EPS, DELTA, GAMMA = 0.7, 0.03, 0.05, 0.03
N_OBJ = 3001
FEW = 65536


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


def ids(n, seed, one_x=False):
    """Pairs of which about half are the generator's similar ones."""
    rng = np.random.default_rng(seed)
    x = rng.integers(0, N_OBJ - 1, n).astype(np.uint32)
    if one_x:
        x[:] = 10
    y = np.where(rng.random(n) < 0.5, x ^ 1, rng.integers(0, N_OBJ, n)).astype(np.uint32)
    y[-1] = N_OBJ - 1   # the last row ends the buffer
    return x, y


def variants(sig, measure, n_hashes):
    om = sigs_tensor(sig, measure, P.OBJECT_MAJOR)
    out = {"rows": om}
    if measure == P.COSINE:
        buf = torch.zeros(om.data.numel() + 1, dtype=torch.int32, device="cuda")
        buf[1:] = om.data.reshape(-1).view(torch.int32)
        pfx = up(np.ascontiguousarray(sig[:, :4])) if n_hashes >= 128 else None
        wm = sigs_tensor(sig, measure, P.WORD_MAJOR)
        out["words"] = wm
        out["rows at 4 bytes"] = P.Signatures(buf[1:].view(torch.uint32), measure, P.OBJECT_MAJOR, N_OBJ, n_hashes)
        if pfx is not None:
            out["words, prefix"] = P.Signatures(wm.data, measure, P.WORD_MAJOR, N_OBJ, n_hashes, prefix=pfx)
            out["rows at 4 bytes, prefix"] = P.Signatures(buf[1:].view(torch.uint32), measure, P.OBJECT_MAJOR, N_OBJ,
                                                          n_hashes, prefix=pfx)
    return out


@pytest.mark.parametrize("measure,n_hashes,k", [(P.COSINE, 1024, 16), (P.COSINE, 1024, 32), (P.COSINE, 1024, 64),
                                                (P.COSINE, 416, 32), (P.COSINE, 96, 32), (P.COSINE, 128, 64),
                                                (P.JACCARD, 256, 16), (P.JACCARD, 256, 32), (P.JACCARD, 192, 64)])
def test_few_and_many_candidates(ctx, measure, n_hashes, k):
    sig = signatures(measure, n_hashes, 31 + n_hashes + k)
    S = variants(sig, measure, n_hashes)
    for n in (1, 255, 256, 257, FEW, FEW + 1, 64):
        for one_x in (False, True):
            x, y = ids(n, n + k, one_x)
            want = R.verify(x, y, measure, sig, k, n_hashes // k, T, EPS, DELTA, GAMMA)
            for name, s in S.items():
                print("few measure %d hashes %d k %d n %d one x %d %s" % (measure, n_hashes, k, n, one_x, name), flush=True)
                cands = [P.pairs(up(x), up(y))]
                if one_x:
                    cands.append(P.query_lists(up(x[:1]), up(np.array([0, n], np.int64)), up(y)))
                for c in cands:
                    res = P.make_result(n, n, m_debug=True)
                    P.bayeslsh_verify(ctx, c, s, T, EPS, DELTA, GAMMA, (1, 1), k, res)
                    P.bayeslsh_sync(ctx)
                    assert_same_as_oracle(decode_result(res, n), want)


@pytest.mark.parametrize("measure", [P.COSINE, P.JACCARD])
def test_few_candidates_refused_ids_and_short_lists(ctx, measure):
    """An id out of range, then a list too short for the accepted pairs: each is
    reported, the count is the true one, and the next call starts from zero."""
    sig = signatures(measure, 256, 5)
    S = sigs_tensor(sig, measure, P.OBJECT_MAJOR)
    x, y = ids(1000, 6)
    want = R.verify(x, y, measure, sig, 32, 8, T, EPS, DELTA, GAMMA)
    n_acc = int(((want["decision"] == R.DEC_CONC) | (want["decision"] == R.DEC_NMAX)).sum())
    assert n_acc > 100
    bad = y.copy()
    bad[700] = N_OBJ
    for ys, cap, code, count in ((bad, 1000, -5, None), (y, 50, -4, n_acc), (y, 1000, None, n_acc)):
        res = P.make_result(1000, cap, m_debug=True)
        P.bayeslsh_verify(ctx, P.pairs(up(x), up(ys)), S, T, EPS, DELTA, GAMMA, (1, 1), 32, res)
        if code is None:
            P.bayeslsh_sync(ctx)
            assert_same_as_oracle(decode_result(res, 1000), want)
        else:
            with pytest.raises(P.BayesLSHError) as e:
                P.bayeslsh_sync(ctx)
            assert e.value.code == code
        got = res.code.cpu().numpy()
        keep = np.arange(1000) != 700 if ys is bad else np.ones(1000, bool)
        np.testing.assert_array_equal((got >> 6)[keep], want["decision"][keep])
        assert ys is not bad or got[700] == 0xFF
        assert count is None or int(res.n_accepted.item()) == count
