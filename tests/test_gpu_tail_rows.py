"""Undecided SRP pairs finished by groups of lanes over 16-byte-aligned rows:
row lengths around a pass of the group (4 or 8 lanes, 512 or 1024 hashes), a
last pass that is nearly empty, n_max below the stored hashes, every k; the
oracle's decisions, levels, m and S_hat."""
import numpy as np
import pytest

import paper_1110_1328_amd as P
from oracle import reference as R
from synth import generators as G

from gpu_util import assert_same_as_oracle, decode_result, sigs_tensor, up

pytestmark = pytest.mark.gpu

N_OBJ = 2002
N = 65536 + 77   # past the calls that run in one launch


@pytest.fixture(scope="module")
def ctx():
    c = P.bayeslsh_create(0)
    yield c
    c.close()


@pytest.mark.parametrize("stored,n_max,k", [(256, 256, 16), (256, 192, 64), (384, 384, 32), (512, 512, 64), (512, 512, 16),
                                            (640, 544, 32), (640, 640, 64), (1024, 1024, 16), (1024, 992, 32),
                                            (1152, 1088, 64), (1152, 1056, 32), (2048, 2048, 32), (2048, 2048, 64),
                                            (3072, 2112, 64)])
@pytest.mark.parametrize("t,prefix", [(0.7, False), (0.8, True)])
def test_rows_tail(ctx, stored, n_max, k, t, prefix):
    print("rows tail stored %d n_max %d k %d t %.1f prefix %d" % (stored, n_max, k, t, prefix), flush=True)
    rng = np.random.default_rng(stored + n_max + k)
    s = rng.uniform(0.6, 0.95, N_OBJ // 2)
    sig = G.pack_bits(G.calibration_bits(len(s), stored, s, stored + k))
    x = rng.integers(0, N_OBJ, N).astype(np.uint32)
    y = np.where(rng.random(N) < 0.7, x ^ 1, rng.integers(0, N_OBJ, N)).astype(np.uint32)
    want = R.verify(x, y, P.COSINE, sig, k, n_max // k, t, 0.03, 0.05, 0.03)
    assert np.sum(want["level"] >= 128 // k) > 1000   # the tail has work
    S = sigs_tensor(sig, P.COSINE, P.OBJECT_MAJOR, n_max)
    if prefix:
        S = P.Signatures(S.data, P.COSINE, P.OBJECT_MAJOR, N_OBJ, stored, n_max, prefix=up(np.ascontiguousarray(sig[:, :4])))
    res = P.make_result(N, N, m_debug=True)
    P.bayeslsh_verify(ctx, P.pairs(up(x), up(y)), S, t, 0.03, 0.05, 0.03, (1, 1), k, res)
    P.bayeslsh_sync(ctx)
    assert_same_as_oracle(decode_result(res, N), want)
