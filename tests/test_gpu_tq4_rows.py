"""GPU TQ4 encoder and reconstruction where a wave's four vectors meet an edge:
head counts that do not divide a batch (each vector then looks its row up by
itself), a last batch that is not full, more batches than the grid's waves
take at once, and pages shorter than the run of positions a wave rebuilds.
Oracle, bounds and poison checks are those of test_gpu_tq4 and
test_gpu_reconstruct."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from gpu_cases import log  # noqa: E402
from oracle import tq4  # noqa: E402
from paper_2609_17475_amd import jfkv  # noqa: E402
from test_gpu_tq4_decode import Case  # noqa: E402
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


@pytest.mark.parametrize("index", [1, 14])  # a negative and a positive centroid
def test_cancelled_sums_are_positive_zeros(index):
    """A vector of one centroid transforms to 256 c in element 0 and sums that
    cancel elsewhere: +0 in fp32 (x - x), whatever lane holds them, so that the
    fp16 result there is a zero with the sign of its element's sign (to the bit)."""
    log("tq4 cancelled sums, index %d" % index)
    P, L = 64, 70
    c = Case(P, 1, (L,), seed=index)
    for pool in (c.k_pool, c.v_pool):
        pool.words.fill_(index * 0x11111111 - (1 << 32 if index > 7 else 0))
        pool.norms.fill_(1.0)
    k, v = (torch.full((1, L, 256), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2))
    jfkv.jf_tq4_reconstruct(c.k_pool, c.v_pool, c.dev["sk"], c.dev["sv"], c.dev["c"],
                            torch.from_numpy(c.tables[0]).to("cuda"), L, 0, 1, k, v)
    o = c.gpu(np.zeros((1, 4, 256), np.float16), lens=[1])
    for what, got, s in (("K", k, c.sk), ("V", v, c.sv), ("decode", torch.from_numpy(o), c.sv)):
        got = got.cpu().numpy().reshape(-1, 256)
        assert np.all(np.abs(got[:, 0] - s[0] * 16 * np.float64(c.c[index])) <= 2e-3 * 16 * abs(c.c[index]))
        assert not np.any(got[:, 1:]), what
        assert np.array_equal(np.signbit(got[:, 1:]), np.broadcast_to(s[1:] < 0, got[:, 1:].shape)), what


@pytest.mark.parametrize("index", [None, 1, 14])
def test_zero_norm_gives_zeros_of_the_vector_s_signs(index):
    """A norm of 0 (a zero vector; all indices equal, as the encoder stores it, or
    any) times the transform: zeros with the signs of the products, sums that
    cancel counting as +0."""
    log("tq4 zero norms, index %s" % index)
    P, L = 64, 37
    c = Case(P, 1, (L,), seed=5)
    for pool in (c.k_pool, c.v_pool):
        if index is not None:
            pool.words.fill_(index * 0x11111111 - (1 << 32 if index > 7 else 0))
        pool.norms.fill_(0.0)
    k, v = (torch.full((1, L, 256), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2))
    jfkv.jf_tq4_reconstruct(c.k_pool, c.v_pool, c.dev["sk"], c.dev["sv"], c.dev["c"],
                            torch.from_numpy(c.tables[0]).to("cuda"), L, 0, 1, k, v)
    for what, got, pool, s in (("K", k, c.k_pool, c.sk), ("V", v, c.v_pool, c.sv)):
        got = got.cpu().numpy()[0]
        assert not np.any(got), what
        words, _ = tq4.gather(pool.words.cpu().numpy().view(np.uint32), c.kn, c.tables[0], L)
        x = tq4.reconstruct(tq4.unpack(words[:, 0]), np.ones(L, np.float16), s, c.c)
        # sums near zero may have either sign in fp32 (2^-20 of the largest is far
        # above their rounding, 8 * 2^-24); exact ones are +0, times the sign
        sure = np.abs(x) > 2.0 ** -20 * np.abs(x).max()
        assert np.array_equal(np.signbit(got)[sure], (x < 0)[sure]), what
        if index is not None:
            assert np.array_equal(np.signbit(got[:, 1:]), np.broadcast_to(s[1:] < 0, (L, 255))), what


def test_nan_rows_keep_the_norm_s_bits():
    """The norm of a row with a NaN is that NaN, quiet, with its sign (the signs of
    the transform do not enter the squares)."""
    log("tq4 NaN rows")
    lay = jfkv.layout(64, 4, 256, 64, 2)
    x = torch.randn((16, 4, 256), generator=torch.Generator().manual_seed(1)).half()
    for i in range(16):
        x[i, :, 16 * i + i % 5] = float("nan")
    pool = jfkv.TQ4Pool(lay, fill=0)
    i32 = dict(dtype=torch.int32, device="cuda")
    signs = torch.where(torch.arange(256) % 3 == 0, -1.0, 1.0).cuda()
    jfkv.jf_tq4_encode_append(pool, x.cuda(), signs, Case(64, 1, (1,), 1).dev["c"],
                              torch.tensor([0, 16], **i32), torch.tensor([0], **i32),
                              torch.tensor([[1]], **i32))
    bits = pool.norms.view(torch.int16)[1, :, :16].cpu().numpy().view(np.uint16)
    assert np.all(bits == 0x7E00), bits
