"""Decode of a batch by blocks that share a CU two and two (rings of two
stages) against the same requests one by one and, at head_dim 128, under a
table so wide that the blocks keep rings of three: the ring depth changes no
result bit, and the oracle's tolerance holds: 2e-3, plus 2^-11 |o| for
the rounding of the fp16 output itself (a window of one or a few positions has
outputs as large as the outlier channels, |o| ~ 20).  Lengths around a row (32), the
rows of one ring turn of a block (8 or 4 waves), a page, and two requests of
very different lengths; the fused step over several ring turns.  Each case
states that the launch it means to test is paired, and that the ones it is
compared with are not."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from gpu_cases import build, check_tol, log  # noqa: E402
from test_gpu_decode import _q, decode_gpu, decode_oracle  # noqa: E402
from test_gpu_decode_step import _run_steps  # noqa: E402


def paired(P, hkv, hq, d, G, B, max_pages, max_splits=64):
    """Whether the launch pairs its blocks: one column set, more blocks than CUs
    and, at head_dim 128, tables of at most 4,096 positions per split."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    gq = hq // hkv
    slots = 4 if d == 256 or G == 32 else 8  # query heads of a column set
    if d == 64 or (d == 128 and gq > slots):
        return False
    chunks = -(-gq // slots)
    splits = max(1, min(max_splits, cus // (hkv * chunks)))
    blocks = splits * hkv if chunks == 1 else -(-splits * hkv // 8) * 8 * chunks
    return blocks * B > cus and (d == 256 or max_pages * P <= 4096 * splits)


@pytest.mark.parametrize("P,hkv,hq,d,G,lens", [
    (256, 2, 8, 128, 64, (1, 31, 33, 257)),
    (64, 2, 8, 128, 32, (4097, 63, 700)),
    (256, 2, 8, 128, 128, (2049, 511, 768)),
    (256, 4, 24, 256, 64, (1500, 256)),    # two head chunks
    (64, 2, 8, 256, 32, (129, 2000, 5)),
    (64, 2, 6, 256, 128, (900, 33, 65)),
])
def test_pairs_equal_single_requests(P, hkv, hq, d, G, lens):
    log("decode pairs P=%d hkv=%d hq=%d d=%d G=%d lens=%s" % (P, hkv, hq, d, G, lens))
    case = build(P=P, hkv=hkv, d=d, G=G, hq=hq, lens=lens, seed=sum(lens))
    B, width = case.tables.shape
    assert paired(P, hkv, hq, d, G, B, width) and not paired(P, hkv, hq, d, G, 1, width)
    q = _q(3, len(lens), hq, d)
    got = decode_gpu(case, q)
    check_tol(got, decode_oracle(case, q), atol=2e-3, rel_elem=2.0 ** -11, what="pairs")
    for b, n in enumerate(lens):
        alone = decode_gpu(case, q[b:b + 1], lens=[n], tables=case.tables[b:b + 1])
        assert np.array_equal(alone[0], got[b])
    if d == 256:  # (paired whatever the width)
        return
    # one split covers more than 4,096 positions of this table
    wide = np.full((len(lens), 256 * 4096 // P + 300), -1, np.int32)
    wide[:, :width] = case.tables
    assert not paired(P, hkv, hq, d, G, B, wide.shape[1])
    assert np.array_equal(decode_gpu(case, q, tables=wide), got)


@pytest.mark.parametrize("hq,d,G", [(32, 128, 32), (32, 128, 64), (64, 128, 128), (32, 256, 32),
                                    (24, 256, 64), (32, 256, 128)])
def test_paired_steps_over_several_ring_turns(hq, d, G):
    """Fused steps of five requests over seven splits: ~1,290 positions per split,
    five rows per wave of 8 and ten of 4, so the two-stage rings turn over
    several times; the new rows fall into different waves and stages.  Pool
    bytes and outputs as in test_gpu_decode_step."""
    P, hkv, lens = 64, 8, (9000, 8970, 4097, 9023, 130)
    assert paired(P, hkv, hq, d, G, len(lens), -(-9025 // P), max_splits=7)
    _run_steps(P, hkv, d, G, hq, lens, 2, seed=d + G, max_splits=7)
