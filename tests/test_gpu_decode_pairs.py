"""Decode of a batch by blocks that share a CU two and two (rings of two
stages) against the same requests one by one and under a table so wide that
the blocks keep rings of three: the ring depth changes no result bit, and the
oracle's tolerance holds: 2e-3, plus 2^-11 |o| for
the rounding of the fp16 output itself (a window of one or a few positions has
outputs as large as the outlier channels, |o| ~ 20).  Lengths around a row (32), the
rows of one ring turn of a block (8 or 4 waves), a page, and two requests of
very different lengths."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_cases import build, check_tol, log  # noqa: E402
from test_gpu_decode import _q, decode_gpu, decode_oracle  # noqa: E402


@pytest.mark.parametrize("P,hkv,hq,d,G,lens", [
    (256, 2, 8, 128, 64, (1, 31, 33, 257)),
    (64, 1, 8, 128, 32, (4097, 63)),
    (256, 1, 4, 128, 128, (2049, 511, 768)),
    (256, 4, 24, 256, 64, (1500, 256)),
    (64, 1, 4, 256, 32, (129, 2000, 5)),
])
def test_pairs_equal_single_requests(P, hkv, hq, d, G, lens):
    log("decode pairs P=%d hkv=%d hq=%d d=%d G=%d lens=%s" % (P, hkv, hq, d, G, lens))
    case = build(P=P, hkv=hkv, d=d, G=G, hq=hq, lens=lens, seed=sum(lens))
    q = _q(3, len(lens), hq, d)
    got = decode_gpu(case, q)
    check_tol(got, decode_oracle(case, q), atol=2e-3, rel_elem=2.0 ** -11, what="pairs")
    for b, n in enumerate(lens):
        alone = decode_gpu(case, q[b:b + 1], lens=[n], tables=case.tables[b:b + 1])
        assert np.array_equal(alone[0], got[b])
    # one split covers more than 4,096 positions of this table
    wide = np.full((len(lens), 256 * 4096 // P + 300), -1, np.int32)
    wide[:, :case.tables.shape[1]] = case.tables
    assert np.array_equal(decode_gpu(case, q, tables=wide), got)
