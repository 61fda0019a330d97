"""Query lists whose survivors are bunched: thousands of neighbouring related
candidates in one list beside lists with none, with the survivor queue long
enough, too short, and off; the oracle's decisions, levels, m and S_hat, and
the same again from the next batch (the accepted counts start from zero)."""
import numpy as np
import pytest

import paper_1110_1328_amd as P
from oracle import reference as R
from synth import generators as G

from gpu_util import assert_same_as_oracle, decode_result, sigs_tensor, up

pytestmark = pytest.mark.gpu

EPS, DELTA, GAMMA = 0.03, 0.05, 0.03
N_OBJ = 4000
LISTS = [(30_000, 12_000), (1, 1), (9_001, 0), (700, 700), (64, 5), (5_000, 3_000)]   # (length, related run)


@pytest.fixture(scope="module")
def ctx():
    c = P.bayeslsh_create(0)
    yield c
    c.close()


def signatures(measure, n_hashes, seed):
    """Objects 2 i and 2 i + 1 alike, similarities over (0.3, 1)."""
    s = np.random.default_rng(seed).uniform(0.3, 1.0, N_OBJ // 2)
    if measure == P.JACCARD:
        return G.calibration_minhash(len(s), n_hashes, s, seed)
    return G.pack_bits(G.calibration_bits(len(s), n_hashes, s, seed))


def check(ctx, lists, kj, kc, layout, tuning):
    rng = np.random.default_rng(kj + kc)
    jac, cos = signatures(P.JACCARD, 256, 5), signatures(P.COSINE, 512, 6)
    meas, ts, query, ids = [], [], [], []
    for i, (n, run) in enumerate(lists * 2):
        me = (P.JACCARD, P.COSINE)[i >= len(lists)]
        q = int(rng.integers(0, N_OBJ))
        own = rng.integers(0, N_OBJ, n)
        at = int(rng.integers(0, n - run + 1))
        own[at:at + run] = q ^ 1
        meas.append(me); ts.append((0.5, 0.7)[i % 2]); query.append(q); ids.append(own)
    length = np.array([len(v) for v in ids], np.int64)
    offset = np.cumsum(length) - length
    n = int(length.sum())
    want = dict(decision=np.zeros(n, int), level=np.zeros(n, int), m=np.zeros(n, int), shat=np.zeros(n))
    for i, y in enumerate(ids):
        sig, k, h = (jac, kj, 256) if meas[i] == P.JACCARD else (cos, kc, 512)
        w = R.verify(np.full(len(y), query[i], np.uint32), y.astype(np.uint32), meas[i], sig, k, h // k, ts[i], EPS, DELTA,
                     GAMMA)
        for name in want:
            want[name][offset[i]:offset[i] + length[i]] = w[name]
    descs = P.list_descs(np.array(meas, np.int32), np.array(ts), np.array(query, np.uint32), offset, length)
    cand = up(np.concatenate(ids).astype(np.uint32))
    J, C = sigs_tensor(jac, P.JACCARD, P.OBJECT_MAJOR), sigs_tensor(cos, P.COSINE, layout)
    P.bayeslsh_set_tuning(ctx, **tuning)
    try:
        for _ in range(2):
            res = P.make_result(n, n, m_debug=True)
            P.bayeslsh_verify_batched(ctx, descs, cand, J, C, EPS, DELTA, GAMMA, (1.0, 1.0), (kj, kc), res)
            P.bayeslsh_sync(ctx)
            assert_same_as_oracle(decode_result(res, n), want)
    finally:
        P.bayeslsh_set_tuning(ctx)


@pytest.mark.parametrize("kj,kc,layout", [(16, 64, P.WORD_MAJOR), (32, 32, P.OBJECT_MAJOR), (64, 16, P.WORD_MAJOR)])
@pytest.mark.parametrize("tuning", [{}, {"batch_spill_cap": 4096}, {"batch_inreg": 1}, {"batch_inreg": 64},
                                    {"batch_inreg": 1, "batch_blocks_per_cu": 1, "acc_stage_cap": 512}])
def test_bunched_survivors(ctx, kj, kc, layout, tuning):
    print("bunched survivors k %d/%d layout %d %s" % (kj, kc, layout, tuning), flush=True)
    check(ctx, LISTS, kj, kc, layout, tuning)


@pytest.mark.parametrize("lengths", [[250_007], [100, 90_017, 0, 33, 120_000, 1], [70_001, 64, 70_016, 512, 70_000]])
def test_lists_over_several_waves(ctx, lengths):
    """Lists long enough that waves of a small grid run several tiles each and
    share a list by turns, between lists that begin and end inside a wave."""
    print("lists over several waves %s" % lengths, flush=True)
    check(ctx, [(n, n // 50) for n in lengths], 16, 64, P.WORD_MAJOR,
          {"batch_blocks_per_cu": 1, "batch_srp_tile": 128, "batch_mh_tile": 64})
