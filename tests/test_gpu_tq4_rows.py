"""GPU TQ4 encoder and reconstruction where a wave's four vectors meet an edge:
head counts that do not divide a batch (each vector then looks its row up by
itself), a last batch that is not full, more batches than the grid's waves
take at once, and pages shorter than the run of positions a wave rebuilds.
Oracle, bounds and poison checks are those of test_gpu_tq4 and
test_gpu_reconstruct."""
import pytest

pytestmark = pytest.mark.gpu

from test_gpu_reconstruct import test_tq4_reconstruct_matches_oracle as check_reconstruct  # noqa: E402
from test_gpu_tq4 import run_case  # noqa: E402


@pytest.mark.parametrize("P,hkv,lens,starts,NP", [
    (64, 1, (37, 1, 130), (5, 63, 0), 8),   # four rows, of several requests, in a batch
    (20, 3, (61, 30), (3, 0), 8),           # batches across rows; pages of 20
    (64, 6, (75,), (0,), 3),                # both kinds of batch in turn; a last one of two
    (256, 8, (6000,), (100,), 25),          # 12,000 batches: several per wave
])
def test_encode_batches(P, hkv, lens, starts, NP):
    run_case(P, hkv, lens, starts, NP, seed=P + hkv)


@pytest.mark.parametrize("P,hkv,L,n,kv0,g", [
    (20, 2, 150, 141, 0, 2),    # a wave's 16 positions span pages
    (24, 1, 100, 99, 0, 1),
    (48, 3, 200, 161, 1, 2),    # whole waves per page, a last one of one position
])
def test_reconstruct_short_pages(P, hkv, L, n, kv0, g):
    check_reconstruct(P, hkv, L, n, kv0, g)
